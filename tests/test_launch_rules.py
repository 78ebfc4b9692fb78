"""Host-side launch arithmetic of the unit kernels (moe_internal.h), compiled
into a small host program: the LDS that limits resident wavefronts, and the
token ranges of batches with more units than one launch takes."""
import os
import subprocess

import pytest

from paper_2607_26444_amd import build as lib_build

PROGRAM = r"""
#include <cstdio>
#include "moe_internal.h"
extern "C" hipError_t hipGetLastError() { return hipSuccess; }   // nothing is launched here
int main() {
  for (int wpb : {1, 2, 4})
    for (int waves = 1; waves <= 64; ++waves)
      std::printf("lds %d %d %u\n", wpb, waves, moe::wave_limit_lds(waves, wpb));
  for (long long tokens : {0ll, 1ll, 16777215ll, 16777216ll, 16777221ll, 50000000ll})
    for (int slices : {1, 3, 14, 16777216, 20000000}) {
      std::printf("batch %lld %d\n", tokens, slices);
      if (tokens > 1000 && slices > 1000) continue;
      (void)moe::launch_token_ranges(tokens, slices, [](int first, int units) {
        std::printf("range %d %d\n", first, units);
      });
    }
}
"""


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = os.path.join(d, "rules.hip"), os.path.join(d, "rules")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run([lib_build.hipcc(), *lib_build.FLAGS, src, "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return [ln.split() for ln in out.splitlines()]


def test_wave_limit(lines):
    rows = [tuple(map(int, ln[1:])) for ln in lines if ln[0] == "lds"]
    assert len(rows) == 3 * 64
    for wpb, waves, lds in rows:
        blocks = max(1, waves // wpb)
        if lds == 0:     # no limit asked for, or none that LDS can give
            assert 128 // (128 // blocks) * wpb >= 32, (wpb, waves)
            continue
        assert lds % 1280 == 0 and lds <= 160 * 1024
        fit = 128 // (lds // 1280)
        assert blocks <= fit and fit * wpb < 32, (wpb, waves)
        if lds // 1280 < 128:   # one granule more would let in too few
            assert 128 // (lds // 1280 + 1) < blocks, (wpb, waves)


def test_token_ranges(lines):
    batch, got, seen = None, [], 0

    def check():
        tokens, slices = batch
        if tokens > 1000 and slices > 1000:
            return
        at = 0
        for first, units in got:
            assert first == at and units > 0 and units % slices == 0, batch
            assert units <= 1 << 24 or units == slices, batch   # a token is never split
            at += units // slices
        assert at == tokens, batch

    for ln in lines:
        if ln[0] == "batch":
            if batch:
                check()
            batch, got, seen = (int(ln[1]), int(ln[2])), [], seen + 1
        elif ln[0] == "range":
            got.append((int(ln[1]), int(ln[2])))
    check()
    assert seen == 30
