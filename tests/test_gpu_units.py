"""The (token, slice) unit kernels of the default split: edges of slices and
slot groups, against the oracle and, bit for bit, against the persistent
split of the same library (MOE_POLICY_STATIC)."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_26444_amd import moe
    moe.lib()


# T, H, E, R, k, payload, mask, short: row widths one 16-byte piece around
# 1, 2 and 4 KiB (a slice, and the widths from which k = 2 and k = 1 take two
# and four slices per wavefront); k around the groups of 8 gathers; one token.
CASES = [
    (1, 7168, 256, 64, 8, wl.BF16, 0.0, False),
    (3, 8, 4, 2, 1, wl.BF16, 0.0, False),
    (65, 504, 16, 4, 1, wl.BF16, 0.1, True),
    (65, 512, 16, 4, 2, wl.BF16, 0.1, False),
    (65, 520, 16, 4, 2, wl.BF16, 0.0, True),
    (63, 1016, 16, 8, 1, wl.BF16, 0.2, False),
    (63, 1032, 16, 8, 1, wl.BF16, 0.0, True),
    (63, 2056, 16, 8, 1, wl.BF16, 0.2, False),
    (130, 3080, 32, 8, 3, wl.BF16, 0.1, True),
    (130, 1544, 32, 32, 5, wl.BF16, 0.3, False),
    (130, 1032, 64, 16, 7, wl.BF16, 0.3, True),
    (130, 1032, 64, 16, 9, wl.BF16, 0.3, True),
    (70, 520, 64, 16, 16, wl.BF16, 0.5, False),
    (70, 520, 64, 16, 17, wl.BF16, 0.5, True),
    (70, 520, 1024, 1024, 32, wl.BF16, 0.5, True),
    (1, 128, 8, 2, 8, wl.FP8_E4M3, 0.0, False),
    (130, 1152, 32, 8, 3, wl.FP8_E4M3, 0.2, True),      # 36-byte scale rows, pitch 128
    (130, 7168, 64, 16, 8, wl.FP8_E4M3, 0.1, True),     # 224-byte scale rows, pitch 256
    (40, 33280, 16, 4, 4, wl.FP8_E4M3, 0.1, False),     # scale rows of more than 1 KiB
    (65, 56, 16, 4, 3, wl.BF16, 0.1, True),             # rows of less than a line: not units
    (63, 1024, 16, 8, 1, wl.BF16, 0.1, False),          # k = 1: slices of 2 KiB
    (63, 1536, 16, 8, 1, wl.BF16, 0.1, True),           # ... and a last one of 1 KiB
    # 96 to 300 MiB of x and rows: ordinary stores, slices of 2 KiB
    (4100, 2048, 64, 16, 8, wl.BF16, 0.0, True),
    (16000, 1536, 64, 16, 3, wl.BF16, 0.1, False),
    (6000, 1544, 64, 16, 8, wl.BF16, 0.1, True),        # off the line
    (7000, 2048, 64, 16, 8, wl.FP8_E4M3, 0.1, True),
]


# fp8 scale rows at the harness's pitch (whole 128-byte lines) and packed
PACKED = [c + (p,) for p in (False, True) for c in CASES if not p or c[5] == wl.FP8_E4M3]


@pytest.mark.parametrize("T,H,E,R,k,payload,mask,short,packed", PACKED)
def test_units_match_oracle_and_persistent_split(T, H, E, R, k, payload, mask, short, packed):
    import gpu_harness as h
    from paper_2607_26444_amd import moe
    from test_gpu_parity import _full_parity
    cfg = wl.custom(T, H, E, R, k, payload=payload, zipf_s=1.2, seed=T + H + k)
    inp = wl.make_inputs(cfg)
    idx = wl.mask_slots(inp["topk_idx"], mask, seed=k) if mask else None
    delta = [-(r % 2) for r in range(R)] if short else None
    pitch = 0 if packed else None
    kw = dict(idx=idx, spare_rows=0 if short else 1, cap_delta=delta, scale_pitch=pitch)
    run, _ = _full_parity(cfg, inp, **kw)
    again = h.GpuRun(cfg, inp, topk_idx=idx, spare_rows=kw["spare_rows"], cap_delta=delta,
                     scale_pitch=pitch, policy=moe.MOE_POLICY_STATIC,
                     combine_policy=moe.MOE_POLICY_STATIC)
    assert np.array_equal(run.y, again.y)
    assert run.layout["status"] == again.layout["status"]


@pytest.mark.parametrize("T,H,E,R,k", [
    (32768, 8, 16, 4, 2), (32768, 512, 16, 4, 2), (32767, 512, 16, 4, 2), (32768, 256, 16, 4, 4),
    (65536, 64, 16, 8, 1), (65600, 256, 16, 4, 3)])
def test_many_narrow_rows(T, H, E, R, k):
    """Sizes from which combine and the source-side sum leave the units for
    the persistent split, and one token short of them."""
    from test_gpu_dedup import _dedup_parity
    from test_gpu_parity import _full_parity
    cfg = wl.custom(T, H, E, R, k, zipf_s=1.2, seed=T + H + k)
    inp = wl.make_inputs(cfg)
    idx = wl.mask_slots(inp["topk_idx"], 0.1, seed=k)
    delta = [-(r % 2) for r in range(R)]
    _full_parity(cfg, inp, idx=idx, spare_rows=0, cap_delta=delta)
    _dedup_parity(cfg, inp, idx=idx, spare_rows=0, pcap_delta=delta)


# row widths of whole lines (fitting the last slice exactly, or not), of odd
# multiples of 64 bytes and off the line; region bases by bytes past a line,
# one after another over the regions
OFF_BASES = [(0,), (16,), (64,), (112, 0, 48)]
OFF_CASES = [
    (65, 64, 8, 4, 1, wl.BF16),        # one line
    (65, 512, 16, 4, 2, wl.BF16),      # 1 KiB: the whole last slice
    (65, 520, 16, 4, 2, wl.BF16),      # 1 KiB + 16 B
    (65, 568, 16, 4, 3, wl.BF16),      # 1 KiB + 112 B
    (65, 544, 16, 8, 8, wl.BF16),      # 1 KiB + 64 B
    (65, 1016, 16, 4, 1, wl.BF16),     # 2 KiB - 16 B
    (65, 1024, 16, 4, 1, wl.BF16),
    (40, 2048, 64, 16, 9, wl.BF16),    # 4 KiB
    (40, 2056, 64, 16, 17, wl.BF16),
    (30, 7168, 64, 16, 8, wl.BF16),
    (30, 7176, 64, 16, 4, wl.BF16),
    (65, 128, 16, 4, 2, wl.FP8_E4M3),
    (65, 1024, 16, 4, 3, wl.FP8_E4M3),
    (30, 7168, 64, 16, 8, wl.FP8_E4M3),
]


@pytest.fixture(params=OFF_BASES, ids=str)
def off_bases(request, monkeypatch):
    """Regions whose bases lie the given bytes past a 4 KiB boundary."""
    from paper_2607_26444_amd import moe

    class Shifted(moe.Regions):
        def __init__(self, rows, row_bytes, **kw):
            super().__init__(rows, row_bytes, **kw)   # guards are wider than the shift
            by = [request.param[r % len(request.param)] for r in range(len(self.rows))]
            self.offsets = [o + b for o, b in zip(self.offsets, by)]
            self.table += torch.tensor(by, device=self.table.device)

    monkeypatch.setattr(moe, "Regions", Shifted)


@pytest.mark.parametrize("T,H,E,R,k,payload", OFF_CASES)
def test_rows_that_start_inside_a_line(T, H, E, R, k, payload, off_bases):
    """Dispatch, and the per-peer chain, into destination rows that start
    anywhere in a 128-byte line, every byte of the regions and around them."""
    from test_gpu_dedup import _dedup_parity
    from test_gpu_parity import _full_parity
    cfg = wl.custom(T, H, E, R, k, payload=payload, zipf_s=1.2, seed=T + H + k)
    inp = wl.make_inputs(cfg)
    idx = wl.mask_slots(inp["topk_idx"], 0.1, seed=k)
    _full_parity(cfg, inp, idx=idx, spare_rows=1)
    _dedup_parity(cfg, inp, idx=idx)


def _rows_equal(regions, x, src, k):
    """Every region row is x's row of its slot, compared a few million at a time."""
    at = 0
    for r, n in enumerate(regions.rows):
        rows = regions.region(r).view(torch.bfloat16)
        for i in range(0, n, 1 << 22):
            m = min(n - i, 1 << 22)
            want = x[(src[at + i: at + i + m] // k).long()]
            if not torch.equal(rows[i: i + m], want):
                return False
        at += n
    return True


def test_more_units_than_one_launch():
    """2^24 + 300 one-slice tokens: the units of every copy kernel go out in
    two launches, the second one long enough for combine's XCD groups.  x holds
    small integers and every weight is 1, so y is k * x and all sums are exact."""
    from paper_2607_26444_amd import moe
    T, H, E, R, k = (1 << 24) + 300, 64, 8, 4, 5
    t = torch.arange(T, device="cuda", dtype=torch.int32)[:, None]
    j = torch.arange(k, device="cuda", dtype=torch.int32)[None, :]
    idx = ((t * 3 + t // 7 + j) % E).contiguous()
    del t
    x = torch.randint(-2, 3, (T, H), device="cuda", dtype=torch.int8).to(torch.bfloat16)
    w = torch.ones(T, k, device="cuda")
    lay, dl = moe.Layout(T, k, E, R), moe.DedupLayout(T, k, E, R)
    lay.run(idx)
    dl.run(idx)
    src = lay.row_src
    at = (moe.MOE_DTYPE_BF16, H, E, R, idx)

    reg = moe.Regions(lay.rank_count.tolist(), 2 * H, fill=0)
    moe.moe_dispatch(x, None, *at, lay.pos, lay.rank_offset, reg.table, None, reg.cap,
                     lay.workspace, lay.status)
    assert _rows_equal(reg, x, src, k)
    y = torch.zeros_like(x)
    moe.moe_combine(reg.table, w, H, E, R, idx, lay.pos, lay.rank_offset, reg.cap, y,
                    lay.workspace, lay.status)
    assert torch.equal(y, k * x)

    pairs = moe.Regions(dl.tok_count.tolist(), 2 * H, fill=0)
    moe.moe_dispatch_dedup(x, None, *at, dl.tok_pos, dl.tok_offset, pairs.table, None, pairs.cap,
                           dl.workspace, dl.status)
    assert _rows_equal(pairs, x, dl.tok_src, k)
    reg.buf.zero_()
    moe.moe_expand(pairs.table, None, *at, lay.pos, lay.rank_offset, dl.tok_pos, dl.tok_offset,
                   pairs.cap, reg.table, None, reg.cap, lay.workspace, lay.status)
    assert _rows_equal(reg, x, src, k)
    pairs.buf.zero_()
    moe.moe_combine_local(reg.table, w, H, E, R, idx, lay.pos, lay.rank_offset, reg.cap,
                          dl.tok_pos, dl.tok_offset, pairs.cap, pairs.table, lay.workspace,
                          lay.status)
    y.zero_()
    moe.moe_combine_dedup(pairs.table, H, E, R, idx, dl.tok_pos, dl.tok_offset, pairs.cap, y,
                          dl.workspace, dl.status)
    assert torch.equal(y, k * x)
    assert int(lay.status) == 0 and int(dl.status) == 0
