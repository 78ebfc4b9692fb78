"""Per-peer deduplicated path on the GPU against the oracle.

Pair-row layout, its plan, the pair regions, the expanded expert regions and
every status word are compared exactly.  Partial rows and y are bf16 sums
computed in float32 on the GPU and in double in the oracle: partials within
8e-3*|ref| + 1e-3 (one rounding of a float32 sum, as for moe_combine), y
within 1.6e-2*|ref| + 1e-3 -- a partial that lands on the other side of a
rounding boundary moves by up to 2^-7 of itself, and with the stand-in
experts' positive scales and the positive softmax weights every partial of
a token has y's sign, so those moves add up to at most 2^-7 |y| on top of
the 2^-7 |y| of y's own rounding.
"""
import numpy as np
import pytest

import workloads as wl
from paper_2607_26444_amd import moe

pytestmark = pytest.mark.gpu


def _h():
    import gpu_harness
    return gpu_harness


def _close(h, got_u16, want_u16, rtol, what):
    ok, msg = h.combine_close(got_u16, want_u16, rtol=rtol)
    assert ok, f"{what}: {msg}"


def _dedup_parity(cfg, inp=None, idx=None, w=None, **kw):
    h = _h()
    inp = wl.make_inputs(cfg) if inp is None else inp
    idx = inp["topk_idx"] if idx is None else idx
    h.log(f"[dedup] {cfg['name']} T={cfg['T']} H={cfg['H']} E={cfg['E']} R={cfg['R']} "
          f"k={idx.shape[1]} {kw}")
    run = h.DedupRun(cfg, inp, topk_idx=idx, topk_w=w, **kw)
    ref = h.oracle_dedup_chain(cfg, inp, run, topk_idx=idx, topk_w=w)
    T, k = idx.shape
    for key in ("tok_count", "tok_offset", "tok_pos", "tok_src", "status"):
        assert np.array_equal(np.asarray(run.dedup[key]), np.asarray(ref["dedup"][key])), key
    assert np.array_equal(run.plan, oracle_plan(ref["dedup"]["tok_pos"], T, k)), "plan"
    assert run.status == ref["status"], (run.status, ref["status"])
    h.check_regions(None, run.dregions, ref["dregs"])
    if run.dsregions is not None:
        h.check_regions(None, run.dsregions, ref["dsregs"])
    h.check_regions(None, run.regions, ref["regs"])
    if run.sregions is not None:
        h.check_regions(None, run.sregions, ref["sregs"])
    # partial rows: written rows within tolerance, the rest keep the sentinel
    buf = run.pregions.buf.cpu().numpy()
    H = cfg["H"]
    for r, off in enumerate(run.pregions.offsets):
        n_cap = run.pregions.rows[r]
        got = buf[off: off + n_cap * 2 * H].view(np.uint16).reshape(n_cap, H)
        want = ref["parts"][r]
        n = min(int(ref["dedup"]["tok_count"][r]), n_cap)
        assert np.all(got[n:] == h.SENTINEL * 0x101), f"partial region {r}: rows past {n}"
        _close(h, got[:n], want[:n], 8e-3, f"partial region {r}")
    _close(h, run.y, ref["y"], 1.6e-2, "y")
    return run, ref


def oracle_plan(tok_pos, T, k):
    import oracle
    return oracle.plan(tok_pos, T, k, moe.MOE_PLAN_PARTS)


@pytest.mark.parametrize("T,H,E,R,k,payload,mask,zipf", [
    (1000, 1032, 24, 6, 3, wl.BF16, 0.1, 0.0),
    (700, 640, 32, 8, 5, wl.FP8_E4M3, 0.05, 0.0),
    (2049, 7168, 256, 64, 8, wl.BF16, 0.0, 1.2),
    (400, 6152, 64, 16, 8, wl.BF16, 0.1, 1.2),     # 12 KiB + 16 B source-sum rows
    (513, 4096, 128, 32, 8, wl.FP8_E4M3, 0.0, 1.2),
    (300, 256, 16, 4, 1, wl.BF16, 0.0, 0.0),       # k = 1: every slot is a pair
    (200, 512, 16, 16, 4, wl.BF16, 0.0, 0.0),      # one expert per peer
    (150, 256, 8, 1, 4, wl.BF16, 0.0, 0.0),        # one peer
    (300, 256, 8, 2, 6, wl.BF16, 0.1, 0.0),        # k > R: many slots per pair
    (257, 2048, 64, 8, 16, wl.BF16, 0.0, 1.2),
    (100, 512, 64, 8, 32, wl.BF16, 0.05, 0.0),     # 32 slots
    (333, 1024, 48, 12, 7, wl.FP8_E4M3, 0.0, 0.0), # scale rows of 32 bytes
    (2000, 256, 1024, 64, 8, wl.BF16, 0.05, 1.2),  # MOE_MAX_EXPERTS
    (300, 16384, 64, 8, 4, wl.BF16, 0.0, 0.0),     # 32 KiB rows: two passes
    (100, 20480, 32, 8, 2, wl.FP8_E4M3, 0.0, 0.0), # 640-byte scale rows
    (131072, 128, 256, 64, 8, wl.BF16, 0.0, 1.2),  # 1M slots
])
def test_dedup_chain_matches_oracle(T, H, E, R, k, payload, mask, zipf):
    cfg = wl.custom(T, H, E, R, k, payload=payload, zipf_s=zipf, seed=T + 7)
    inp = wl.make_inputs(cfg)
    idx = wl.mask_slots(inp["topk_idx"], mask, seed=T) if mask else None
    _dedup_parity(cfg, inp, idx=idx)


def test_dedup_expand_rebuilds_per_slot_dispatch():
    """The expanded expert regions are the per-slot dispatch's, byte for byte
    (run both on the GPU; each is also checked against the oracle)."""
    h = _h()
    cfg = wl.custom(900, 2048, 64, 16, 6, zipf_s=1.2, seed=5)
    inp = wl.make_inputs(cfg)
    run, _ = _dedup_parity(cfg, inp)
    ref = h.GpuRun(cfg, inp, spare_rows=1)
    a = run.regions.buf.cpu().numpy()
    b = ref.regions.buf.cpu().numpy()
    for r in range(cfg["R"]):
        n = run.regions.rows[r] * run.regions.row_bytes
        assert np.array_equal(a[run.regions.offsets[r]: run.regions.offsets[r] + n],
                              b[ref.regions.offsets[r]: ref.regions.offsets[r] + n]), r


def test_dedup_capacity_overflow():
    """Short pair and partial regions: rows past them are neither written
    nor read, every stage flags bit 4, and the oracle agrees row by row."""
    cfg = wl.custom(800, 1024, 32, 8, 6, zipf_s=1.2, seed=3)
    dd = [0] * 8
    dd[0] = -40
    pd = [0] * 8
    pd[2] = -7
    run, ref = _dedup_parity(cfg, spare_rows=0, dcap_delta=dd, pcap_delta=pd)
    assert run.status["dispatch"] == moe.MOE_STATUS_CAPACITY
    assert run.status["expand"] == moe.MOE_STATUS_CAPACITY
    assert run.status["local"] == moe.MOE_STATUS_CAPACITY


def test_dedup_bad_and_repeated_indices():
    cfg = wl.custom(400, 512, 32, 8, 5, seed=11)
    inp = wl.make_inputs(cfg)
    idx = inp["topk_idx"].copy()
    idx[3, 1] = 32          # out of range
    idx[5, 2] = -7          # out of range (negative)
    idx[7, 4] = idx[7, 0]   # repeat
    idx[9, :] = -1          # token with no routed slot
    run, _ = _dedup_parity(cfg, inp, idx=idx)
    assert run.dedup["status"] == moe.MOE_STATUS_BAD_INDEX | moe.MOE_STATUS_DUP_INDEX
    assert np.all(run.y[9] == 0)


def test_dedup_zero_tokens():
    cfg = wl.custom(0, 256, 16, 4, 2, seed=1)
    _dedup_parity(cfg)


@pytest.mark.parametrize("name", ["decode", "prefill"])
def test_dedup_full_size(name):
    cfg = wl.get(name)
    run, ref = _dedup_parity(cfg)
    n_pairs = int(ref["dedup"]["tok_offset"][-1])
    _h().log(f"[dedup] {name}: {n_pairs} pair rows for {cfg['T'] * cfg['k']} slots "
             f"({n_pairs / (cfg['T'] * cfg['k']):.3f})")


def test_dedup_large_batch():
    """24576 tokens of 14 KiB, the largest chain that is compared whole."""
    _dedup_parity(wl.custom(24576, 7168, 256, 64, 8, zipf_s=1.2, seed=24576))


@pytest.mark.parametrize("T,H,E,R,k,zipf,signed_w", [
    (1500, 2048, 64, 16, 8, 1.2, False),    # several experts per peer under skew
    (600, 7168, 32, 4, 8, 0.0, True),       # k > R: every pair sums slots; signed weights
])
def test_dedup_combine_signed_expert_outputs(T, H, E, R, k, zipf, signed_w):
    """Random signed expert outputs (and, in one case, signed weights), so a
    token's partials differ in sign and y can be much smaller than them.

    Each partial is one float32 sum rounded once to bf16 and may land one
    bf16 step (2^-7 of itself) from the oracle's; the source-side sum adds
    those moves and rounds once more.  So partials are held to
    8e-3*|P_ref| + 1e-3 and y to 8e-3*(sum over the token's pairs of
    |P_ref| + |y_ref|) + 1e-3: with cancelling partials the per-slot bound
    8e-3*|y_ref| + 1e-3 does not hold for this path in general."""
    import oracle
    import torch
    h = _h()
    cfg = wl.custom(T, H, E, R, k, zipf_s=zipf, seed=T + 31)
    inp = wl.make_inputs(cfg)
    idx = inp["topk_idx"]
    w = inp["topk_w"]
    if signed_w:
        rng = np.random.Generator(np.random.PCG64(T))
        w = rng.standard_normal(w.shape).astype(np.float32)
    h.log(f"[dedup-signed] T={T} H={H} E={E} R={R} k={k} signed weights {signed_w}")
    idx_d = h.to_dev(idx.astype(np.int32))
    w_d = h.to_dev(w)
    lay = moe.Layout(T, k, E, R)
    lay.run(idx_d)
    dl = moe.DedupLayout(T, k, E, R)
    dl.run(idx_d)
    torch.cuda.synchronize()
    caps = lay.rank_count.cpu().numpy().astype(np.int32) + 1
    pcaps = dl.tok_count.cpu().numpy().astype(np.int32) + 1
    # expert outputs: seeded signed bf16 rows, the same bytes on both sides
    ey = [wl.random_bf16_rows(int(c), H, seed=1000 + r) for r, c in enumerate(caps)]
    eregions = moe.Regions([int(c) for c in caps], 2 * H, guard_bytes=h.GUARD,
                           fill=h.SENTINEL)
    for r in range(R):
        eregions.region(r).copy_(torch.from_numpy(ey[r].view(np.uint8)).cuda())
    pregions = moe.Regions([int(c) for c in pcaps], 2 * H, guard_bytes=h.GUARD,
                           fill=h.SENTINEL)
    y = torch.full((T, H), 0x5A5A, dtype=torch.int16, device="cuda")
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    moe.moe_combine_local(eregions.table, w_d, H, E, R, idx_d, lay.pos, lay.rank_offset,
                          eregions.cap, dl.tok_pos, dl.tok_offset, pregions.cap,
                          pregions.table, lay.workspace, st)
    moe.moe_combine_dedup(pregions.table, H, E, R, idx_d, dl.tok_pos, dl.tok_offset,
                          pregions.cap, y, dl.workspace, st)
    torch.cuda.synchronize()
    assert int(st.item()) == 0

    ol = oracle.layout(idx, E, R)
    od = oracle.layout_dedup(idx, E, R)
    parts, st_l = oracle.combine_local(ey, w, idx, ol["pos"], ol["rank_offset"], caps,
                                       od["tok_pos"], od["tok_offset"], pcaps, E, R, H,
                                       sentinel=h.SENTINEL * 0x101)
    y_ref, st_y = oracle.combine_dedup(parts, idx, od["tok_pos"], od["tok_offset"], pcaps,
                                       E, R, H)
    assert st_l == 0 and st_y == 0
    buf = pregions.buf.cpu().numpy()
    for r, off in enumerate(pregions.offsets):
        n = int(od["tok_count"][r])
        got = buf[off: off + pregions.rows[r] * 2 * H].view(np.uint16).reshape(-1, H)
        _close(h, got[:n], parts[r][:n], 8e-3, f"partial region {r}")
    # sum over each token's pairs of |P_ref|
    L = E // R
    abs_sum = np.zeros((T, H))
    for s in np.nonzero(od["tok_pos"] >= 0)[0]:
        t, r = s // k, idx.ravel()[s] // L
        row = od["tok_pos"][s] - od["tok_offset"][r]
        abs_sum[t] += np.abs(h.bf16_to_f64(parts[r][row]))
    got = h.bf16_to_f64(y.cpu().numpy().view(np.uint16))
    want = h.bf16_to_f64(y_ref)
    err = np.abs(got - want)
    bound = 8e-3 * (abs_sum + np.abs(want)) + 1e-3
    assert np.all(err <= bound), (int((err > bound).sum()), float((err / bound).max()))
    plain = err > 8e-3 * np.abs(want) + 1e-3
    h.log(f"[dedup-signed] y within the two-rounding bound (max err/bound "
          f"{float((err / bound).max()):.3f}); {int(plain.sum())} of {err.size} elements "
          f"outside the per-slot bound 8e-3*|y|+1e-3")
