"""Run the HIP path end to end through the C ABI and the oracle beside it.

Used by the GPU parity tests and the smoke check.  Inputs come from
`workloads`; the oracle chain (layout -> dispatch -> expert -> combine) is
computed from the same inputs only, never from GPU results.
"""
from __future__ import annotations

import sys

import numpy as np
import torch

import oracle
import workloads as wl
from paper_2607_26444_amd import moe

SENTINEL = 0xA5
GUARD = 4096


def log(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def to_dev(a: np.ndarray) -> torch.Tensor:
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint16:
        a = a.view(np.int16)
    return torch.from_numpy(a).to("cuda")


def u8_rows(a: np.ndarray) -> np.ndarray:
    a = np.ascontiguousarray(a)
    return a.view(np.uint8).reshape(a.shape[0], int(np.prod(a.shape[1:])) * a.itemsize)


class GpuRun:
    """One pass of layout -> dispatch -> expert -> combine on the GPU."""

    def __init__(self, cfg, inp, topk_idx=None, topk_w=None, spare_rows=0,
                 cap_delta=None, identity=None, combine_on_dispatch=False, scale_pitch=None,
                 policy=0, trace=False, combine_policy=0, repeat=1, capacity=None, waves=0):
        self.cfg = cfg
        T, H, E, R = cfg["T"], cfg["H"], cfg["E"], cfg["R"]
        idx = inp["topk_idx"] if topk_idx is None else topk_idx
        w = inp["topk_w"] if topk_w is None else topk_w
        k = idx.shape[1]
        fp8 = cfg["payload"] == wl.FP8_E4M3
        dtype = moe.MOE_DTYPE_FP8_E4M3 if fp8 else moe.MOE_DTYPE_BF16
        ident = (cfg["expert"] == "identity") if identity is None else identity
        self.idx, self.w, self.k = idx, w, k

        idx_d = to_dev(idx.astype(np.int32))
        w_d = to_dev(w.astype(np.float32))
        lay = moe.Layout(T, k, E, R, capacity=capacity)
        lay.run(idx_d)
        torch.cuda.synchronize()
        counts = lay.rank_count.cpu().numpy()
        if capacity is None:
            caps = counts.astype(np.int64) + spare_rows
        else:   # whole expert windows, no count needed
            caps = np.full(R, (E // R) * capacity, np.int64)
        if cap_delta is not None:
            caps = np.maximum(0, caps + np.asarray(cap_delta))
        self.caps = caps.astype(np.int32)
        rows = [int(c) for c in self.caps]

        rb, sb = wl.row_bytes(cfg), wl.scale_row_bytes(cfg)
        # default scale pitch: rows rounded up to whole 128-byte lines
        self.scale_pitch = (sb + 127) // 128 * 128 if scale_pitch is None else (scale_pitch or sb)
        self.regions = moe.Regions(rows, rb, guard_bytes=GUARD, fill=SENTINEL)
        cap_d = to_dev(self.caps)
        self.sregions = None
        x_d = to_dev(u8_rows(inp["x"]))
        xs_d = None
        if fp8:
            self.sregions = moe.Regions(rows, self.scale_pitch, guard_bytes=GUARD,
                                        fill=SENTINEL)
            xs_d = to_dev(inp["x_scales"]).view(torch.float32)
        self.dtrace = torch.zeros(2 * moe.MOE_PLAN_PARTS, dtype=torch.int64,
                                  device="cuda") if trace else None
        self.ctrace = torch.zeros_like(self.dtrace) if trace else None
        # Repeats reuse one layout and so its work tickets: before every
        # repeat the outputs go back to the sentinel, so a call that skipped
        # parts (a ticket counter left non-zero by the call before it) would
        # leave sentinel bytes behind; after every call all tickets are zero.
        for i in range(repeat):
            if i > 0:
                self.regions.buf.fill_(SENTINEL)
                if fp8:
                    self.sregions.buf.fill_(SENTINEL)
            moe.moe_dispatch_ex(x_d, xs_d, dtype, H, E, R, idx_d, lay.pos, lay.rank_offset,
                                lay.row_src, self.regions.table,
                                self.sregions.table if fp8 else None, cap_d, lay.workspace,
                                lay.status, policy=policy, trace=self.dtrace,
                                scale_pitch=self.scale_pitch, waves=waves)
            check_tickets_zero(lay.workspace, f"dispatch call {i}")

        y = torch.empty((max(1, T), H), dtype=torch.int16, device="cuda")
        y.fill_(0x5A5A)
        if combine_on_dispatch:
            assert not fp8
            ey_table = self.regions.table
            self.eregions = None
        else:
            self.eregions = moe.Regions(rows, 2 * H, guard_bytes=GUARD, fill=SENTINEL)
            moe.moe_expert_scale(self.regions.table,
                                 self.sregions.table if fp8 else None, dtype, H, E, R,
                                 ident, lay.expert_offset, lay.rank_offset, cap_d,
                                 self.eregions.table,
                                 max(1, T * k if capacity is None else E * capacity),
                                 scale_pitch=self.scale_pitch)
            ey_table = self.eregions.table
        for i in range(repeat):
            if i > 0:
                y.fill_(0x5A5A)
            moe.moe_combine_ex(ey_table, w_d, H, E, R, idx_d, lay.pos, lay.rank_offset, cap_d,
                               y, lay.workspace, lay.status, policy=combine_policy,
                               trace=self.ctrace, waves=waves)
            check_tickets_zero(lay.workspace, f"combine call {i}")
        torch.cuda.synchronize()

        nrows = T * k if capacity is None else E * capacity
        self.layout = dict(
            expert_count=lay.expert_count.cpu().numpy(),
            expert_offset=lay.expert_offset.cpu().numpy(),
            rank_count=counts,
            rank_offset=lay.rank_offset.cpu().numpy(),
            pos=lay.pos.cpu().numpy()[: T * k],
            row_src=lay.row_src.cpu().numpy()[:nrows],
            status=int(lay.status.cpu().numpy()[0]))
        self.plan = lay.plan().cpu().numpy()
        self.y = y.cpu().numpy().view(np.uint16)[:T]
        self._lay = lay

    def region_bytes(self, regions):
        return regions.buf.cpu().numpy(), regions.offsets


# The work tickets sit right after the plan, which is bound[MOE_PLAN_PARTS +
# 1] padded to 256 bytes (the library's internal workspace layout): two groups
# (dispatch, combine) of 16 shards, each shard {next claim, wavefronts done} at
# the start of its own 128-byte line.
TICKET_OFFSET = ((moe.MOE_PLAN_PARTS + 1) * 4 + 255) // 256 * 256
TICKET_LINES = 2 * 16
TICKET_BYTES = TICKET_LINES * 128


def ticket_words(raw: np.ndarray) -> np.ndarray:
    """{next, done} of every shard from the raw int32 ticket block."""
    return raw[: TICKET_LINES * 32].reshape(TICKET_LINES, 32)[:, :2].ravel()


def tickets(workspace) -> np.ndarray:
    torch.cuda.synchronize()
    raw = workspace[TICKET_OFFSET: TICKET_OFFSET + TICKET_BYTES].view(torch.int32).cpu().numpy()
    return ticket_words(raw)


def check_tickets_zero(workspace, what):
    t = tickets(workspace)
    assert not t.any(), f"{what}: work tickets not reset: {t.tolist()}"


def oracle_chain(cfg, inp, topk_idx=None, topk_w=None, caps=None, identity=None,
                 combine_on_dispatch=False, scale_pitch=0, capacity=None):
    E, R, H = cfg["E"], cfg["R"], cfg["H"]
    idx = inp["topk_idx"] if topk_idx is None else topk_idx
    w = inp["topk_w"] if topk_w is None else topk_w
    fp8 = cfg["payload"] == wl.FP8_E4M3
    ident = (cfg["expert"] == "identity") if identity is None else identity
    lay = oracle.layout(idx, E, R) if capacity is None else \
        oracle.layout_fixed(idx, E, R, capacity)
    cap = lay["rank_count"] if caps is None else caps
    xs = u8_rows(inp["x_scales"]) if fp8 else None
    regs, sregs, st_d = oracle.dispatch(u8_rows(inp["x"]), xs, idx, lay["pos"],
                                        lay["rank_offset"], E, R, cap, SENTINEL,
                                        scale_pitch=scale_pitch)
    if combine_on_dispatch:
        ey = [r.view(np.uint16).reshape(r.shape[0], H) for r in regs]
    else:
        ey = oracle.expert_scale(regs, sregs, fp8, H, E, R, ident, lay["expert_offset"],
                                 lay["rank_offset"], cap)
    y, st_c = oracle.combine(ey, w, idx, lay["pos"], lay["rank_offset"], cap, E, R, H)
    return dict(layout=lay, regs=regs, sregs=sregs, ey=ey, y=y, status=st_d | st_c)


def bf16_to_f64(a):
    return (a.astype(np.uint32) << 16).view(np.float32).astype(np.float64)


def combine_close(y, y_ref, rtol=8e-3, atol=1e-3):
    """|y - y_ref| <= rtol*|y_ref| + atol, element-wise (NaN must match)."""
    a, b = bf16_to_f64(y), bf16_to_f64(y_ref)
    nan = np.isnan(b)
    if not np.array_equal(np.isnan(a), nan):
        return False, "NaN mismatch"
    err = np.abs(a[~nan] - b[~nan])
    bound = rtol * np.abs(b[~nan]) + atol
    bad = err > bound
    if bad.any():
        i = int(np.argmax(err - bound))
        return False, f"{int(bad.sum())} elements out of tolerance; worst err {err[i]} " \
                      f"bound {bound[i]}"
    return True, f"max err/bound {float((err / bound).max()) if err.size else 0:.3f}"


def check_regions(run, regions, oracle_regs, rows_written=None):
    """Region bytes equal the oracle's (only the first rows_written[r] rows of
    region r when given; the rest must keep the sentinel); guard bands and
    gaps between regions keep the sentinel."""
    buf = regions.buf.cpu().numpy()
    mask = np.ones(buf.shape[0], bool)
    for r, off in enumerate(regions.offsets):
        n_cap = regions.rows[r]
        got = buf[off: off + n_cap * regions.row_bytes].reshape(n_cap, regions.row_bytes)
        want = oracle_regs[r]
        if rows_written is not None:
            n = int(rows_written[r])
            assert np.all(got[n:] == SENTINEL), f"region {r}: rows past {n} written"
            got, want = got[:n], want[:n]
        assert got.shape == want.shape, (r, got.shape, want.shape)
        if not np.array_equal(got, want):
            bad = np.nonzero((got != want).any(1))[0]
            raise AssertionError(f"region {r}: {len(bad)} rows differ, first {bad[:5]}")
        mask[off: off + n_cap * regions.row_bytes] = False
    outside = buf[mask]
    assert np.all(outside == SENTINEL), "bytes outside the regions were written"


def f32_bits_to_bf16_rne(f32: np.ndarray) -> np.ndarray:
    """bf16 bit patterns of float32 values via torch's CPU cast (RNE)."""
    t = torch.from_numpy(np.ascontiguousarray(f32, np.float32)).to(torch.bfloat16)
    return t.view(torch.int16).numpy().view(np.uint16)


class DedupRun:
    """The per-peer deduplicated chain on the GPU: both layouts, dispatch of
    pair rows, expansion into expert order, stand-in expert, partial combine
    per pair and the source-side sum."""

    def __init__(self, cfg, inp, topk_idx=None, topk_w=None, spare_rows=1, dcap_delta=None,
                 pcap_delta=None, identity=None, scale_pitch=None):
        T, H, E, R = cfg["T"], cfg["H"], cfg["E"], cfg["R"]
        idx = inp["topk_idx"] if topk_idx is None else topk_idx
        w = inp["topk_w"] if topk_w is None else topk_w
        k = idx.shape[1]
        fp8 = cfg["payload"] == wl.FP8_E4M3
        dtype = moe.MOE_DTYPE_FP8_E4M3 if fp8 else moe.MOE_DTYPE_BF16
        ident = (cfg["expert"] == "identity") if identity is None else identity
        self.idx, self.w, self.k = idx, w, k
        idx_d = to_dev(idx.astype(np.int32))
        w_d = to_dev(w.astype(np.float32))
        lay = moe.Layout(T, k, E, R)
        lay.run(idx_d)
        dl = moe.DedupLayout(T, k, E, R)
        dl.run(idx_d)
        torch.cuda.synchronize()

        def caps(counts, delta):
            c = counts.astype(np.int64) + spare_rows
            if delta is not None:
                c = np.maximum(0, c + np.asarray(delta))
            return c.astype(np.int32)
        self.caps = caps(lay.rank_count.cpu().numpy(), None)
        self.dcaps = caps(dl.tok_count.cpu().numpy(), dcap_delta)
        self.pcaps = caps(dl.tok_count.cpu().numpy(), pcap_delta)
        rb, sb = wl.row_bytes(cfg), wl.scale_row_bytes(cfg)
        self.scale_pitch = (sb + 127) // 128 * 128 if scale_pitch is None else (scale_pitch or sb)
        sp = self.scale_pitch

        def regions(rows, width):
            return moe.Regions([int(c) for c in rows], width, guard_bytes=GUARD, fill=SENTINEL)
        self.dregions = regions(self.dcaps, rb)
        self.dsregions = regions(self.dcaps, sp) if fp8 else None
        x_d = to_dev(u8_rows(inp["x"]))
        xs_d = to_dev(inp["x_scales"]).view(torch.float32) if fp8 else None
        self.st_dispatch = torch.zeros(1, dtype=torch.int32, device="cuda")
        moe.moe_dispatch_dedup(x_d, xs_d, dtype, H, E, R, idx_d, dl.tok_pos, dl.tok_offset,
                               self.dregions.table,
                               self.dsregions.table if fp8 else None, self.dregions.cap,
                               dl.workspace, self.st_dispatch, scale_pitch=sp)
        self.regions = regions(self.caps, rb)
        self.sregions = regions(self.caps, sp) if fp8 else None
        self.st_expand = torch.zeros(1, dtype=torch.int32, device="cuda")
        moe.moe_expand(self.dregions.table, self.dsregions.table if fp8 else None, dtype, H, E,
                       R, idx_d, lay.pos, lay.rank_offset, dl.tok_pos, dl.tok_offset,
                       self.dregions.cap, self.regions.table,
                       self.sregions.table if fp8 else None, self.regions.cap, lay.workspace,
                       self.st_expand, scale_pitch=sp)
        self.eregions = regions(self.caps, 2 * H)
        moe.moe_expert_scale(self.regions.table, self.sregions.table if fp8 else None, dtype, H,
                             E, R, ident, lay.expert_offset, lay.rank_offset, self.regions.cap,
                             self.eregions.table, max(1, T * k), scale_pitch=sp)
        self.pregions = regions(self.pcaps, 2 * H)
        self.st_local = torch.zeros(1, dtype=torch.int32, device="cuda")
        moe.moe_combine_local(self.eregions.table, w_d, H, E, R, idx_d, lay.pos,
                              lay.rank_offset, self.eregions.cap, dl.tok_pos, dl.tok_offset,
                              self.pregions.cap, self.pregions.table, lay.workspace,
                              self.st_local)
        y = torch.empty((max(1, T), H), dtype=torch.int16, device="cuda")
        y.fill_(0x5A5A)
        self.st_sum = torch.zeros(1, dtype=torch.int32, device="cuda")
        moe.moe_combine_dedup(self.pregions.table, H, E, R, idx_d, dl.tok_pos, dl.tok_offset,
                              self.pregions.cap, y, dl.workspace, self.st_sum)
        torch.cuda.synchronize()
        self.dedup = dict(tok_count=dl.tok_count.cpu().numpy(),
                          tok_offset=dl.tok_offset.cpu().numpy(),
                          tok_pos=dl.tok_pos.cpu().numpy()[: T * k],
                          tok_src=dl.tok_src.cpu().numpy()[: T * k],
                          status=int(dl.status.cpu().numpy()[0]))
        self.plan = dl.plan().cpu().numpy()
        self.status = {n: int(getattr(self, "st_" + n).cpu().numpy()[0])
                       for n in ("dispatch", "expand", "local", "sum")}
        self.y = y.cpu().numpy().view(np.uint16)[:T]


def oracle_dedup_chain(cfg, inp, run, topk_idx=None, topk_w=None, identity=None):
    """The oracle's deduplicated chain on the same inputs and region sizes."""
    E, R, H = cfg["E"], cfg["R"], cfg["H"]
    idx = inp["topk_idx"] if topk_idx is None else topk_idx
    w = inp["topk_w"] if topk_w is None else topk_w
    fp8 = cfg["payload"] == wl.FP8_E4M3
    ident = (cfg["expert"] == "identity") if identity is None else identity
    lay = oracle.layout(idx, E, R)
    d = oracle.layout_dedup(idx, E, R)
    xs = u8_rows(inp["x_scales"]) if fp8 else None
    dregs, dsregs, st_d = oracle.dispatch_dedup(u8_rows(inp["x"]), xs, idx, d["tok_pos"],
                                                d["tok_offset"], E, R, run.dcaps, SENTINEL,
                                                scale_pitch=run.scale_pitch if fp8 else 0)
    srb = xs.shape[1] if fp8 else 0
    regs, sregs, st_e = oracle.expand(dregs, dsregs, srb, idx, lay["pos"], lay["rank_offset"],
                                      d["tok_pos"], d["tok_offset"], run.dcaps, E, R, run.caps,
                                      SENTINEL)
    ey = oracle.expert_scale(regs, sregs, fp8, H, E, R, ident, lay["expert_offset"],
                             lay["rank_offset"], run.caps)
    parts, st_l = oracle.combine_local(ey, w, idx, lay["pos"], lay["rank_offset"], run.caps,
                                       d["tok_pos"], d["tok_offset"], run.pcaps, E, R, H,
                                       sentinel=SENTINEL * 0x101)
    y, st_y = oracle.combine_dedup(parts, idx, d["tok_pos"], d["tok_offset"], run.pcaps, E, R,
                                   H)
    return dict(layout=lay, dedup=d, dregs=dregs, dsregs=dsregs, regs=regs, sregs=sregs,
                ey=ey, parts=parts, y=y,
                status=dict(dispatch=st_d, expand=st_e, local=st_l, sum=st_y))
