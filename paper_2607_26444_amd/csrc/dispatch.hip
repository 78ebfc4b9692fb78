// Dispatch: copy each routed token row into its rank's receive region.
//
// Default split (dispatch_unit_kernel): the batch is cut into (token, 1 or 2
// KiB slice of its row) units, one wavefront each, launched in token order.  A
// wavefront loads its slice once and stores it to the token's k destination
// rows, so x is read exactly once, and the hardware hands units out as
// wavefronts retire: every compute unit takes the next work when it is free,
// whatever the routing (a hot expert only changes where rows land), with no
// plan, no tickets and no metadata beyond the token's own k slots.  The
// fourteen slices of a 14 KiB row start together, so each destination row
// still reaches memory as one run, and a batch of a few tokens spreads over
// the chip by its slices.
//
// Explicit splits (dispatch_kernel; moe_dispatch_ex with a policy, a
// wavefront count or a trace), and rows of less than a line: persistent
// wavefronts over the byte-balanced plan (Section 6.2 with one memory tier,
// Appendix D third level).  moe_layout leaves MOE_PLAN_PARTS contiguous token
// ranges of equal byte cost; wavefront g of W takes parts g,
// g + W, g + 2W, ... or claims parts in plan order at run time.  A wavefront
// reads its token's whole row into registers and stores it to each of the k
// destinations; slot metadata for a batch of 64/k tokens is loaded once, one
// slot per lane, and parked in LDS.

#include "moe_internal.h"

namespace moe {
namespace {

// VPL: 1 KiB segments held per lane-set (row bytes up to VPL KiB per pass).
// FULL: row bytes == VPL KiB exactly (no per-lane tail test).
template <int VPL, bool FULL, bool SCALES, int MODE>
__global__ __launch_bounds__(kBlock) void dispatch_kernel(DispatchArgs a) {
  // Destination row (and scale row) of every slot of the current batch, one
  // entry per lane of each wavefront (0 = slot not dispatched), padded with
  // zeros so a token can read k entries without a bounds test.
  __shared__ uint64_t s_dst[kWavesPerBlock][kWave + MOE_MAX_K];
  __shared__ uint64_t s_sdst[kWavesPerBlock][SCALES ? kWave + MOE_MAX_K : 1];
  // Per-rank tables (first global row, capacity, region bases), staged once
  // per workgroup: a slot's destination is then an LDS lookup behind its pos
  // and expert loads rather than a second, dependent global load.  Measured
  // on MI355X in whole steps: fp8 dispatch 208.0 -> 206.8 us, large 443.9 ->
  // 443.2, prefill and decode unchanged.
  __shared__ int32_t s_roff[MOE_MAX_EXPERTS];
  __shared__ int32_t s_cap[MOE_MAX_EXPERTS];
  __shared__ uint64_t s_rx[MOE_MAX_EXPERTS];
  __shared__ uint64_t s_rs[SCALES ? MOE_MAX_EXPERTS : 1];
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = threadIdx.x / kWave;
  const int g = uniform(blockIdx.x * kWavesPerBlock + wv);
  const uint64_t t_start = a.trace ? (uint64_t)wall_clock64() : 0;
  for (int i = threadIdx.x; i < a.R; i += kBlock) {
    s_roff[i] = a.rank_offset[i];
    s_cap[i] = a.recv_cap[i];
    s_rx[i] = a.recv_x[i];
    if (SCALES) s_rs[i] = a.recv_scales[i];
  }
  __syncthreads();
  const int W = gridDim.x * kWavesPerBlock;
  const uint32_t rb = (uint32_t)a.row_bytes;
  const uint32_t sb = (uint32_t)a.scale_row_bytes;
  const uint32_t sp = (uint32_t)a.scale_pitch;
  const uint32_t l16 = lane * kVecBytes;
  const int k = a.k;
  const int tpb = kWave / k;        // tokens whose slots fit one lane each
  const int lt = lane / k;          // this lane's token within a batch
  const int lj = lane - lt * k;     // ... and its slot
  uint32_t st = 0;
  if (lane < MOE_MAX_K) {
    s_dst[wv][kWave + lane] = 0;
    if (SCALES) s_sdst[wv][kWave + lane] = 0;
  }
  // Rows that fit in one pass (row bytes <= VPL KiB) are loaded one token
  // ahead: the next token's row is requested before the current one is
  // stored, so its loads complete while the stores drain instead of after
  // them (loads and stores share one in-order completion counter).
  const bool one_pass = rb <= (uint32_t)(VPL * kWaveBytes);
  const bool s16 = SCALES && sb % kVecBytes == 0 && sp % kVecBytes == 0 && sp <= kWaveBytes;
  u32x4 vn[VPL];
  u32x4 svn = {0u, 0u, 0u, 0u};
  int pre_t = -1;   // token whose row vn holds (-1: none)
  auto load_row = [&](u32x4 (&v)[VPL], u32x4& sv, int t) {
    const uint8_t* src = a.x + (int64_t)t * rb;
#pragma unroll
    for (int c = 0; c < VPL; ++c) {
      const uint32_t off = c * kWaveBytes + l16;
      if (FULL || off < rb) v[c] = ld16(src + off);
    }
    if (s16 && l16 < sb) sv = ld16(a.x_scales + (int64_t)t * sb + l16);
  };

  const int T = (int)a.tokens;
  for_each_part<MODE, true>(a.bound, a.tickets, g, W, lane, [&](int t0, int t1, int next) {
  // Token ranges (and the token read ahead) stay inside the batch whatever
  // the plan holds: a layout whose barrier timed out leaves parts of it
  // unwritten.
  t0 = max(t0, 0);
  t1 = min(t1, T);
  if (next >= T) next = -1;
  for (int tb = t0; tb < t1; tb += tpb) {
    const int te = min(t1, tb + tpb);
    uint64_t dst = 0, sdst = 0;
    if (tb + lt < te) {
      const int64_t s = (int64_t)(tb + lt) * k + lj;
      const int p = a.pos[s];
      if (p >= 0) {
        const int r = a.topk_idx[s] / a.L;
        if ((unsigned)r >= (unsigned)a.R) {
          st |= MOE_STATUS_BAD_INDEX;   // pos and topk_idx disagree: not copied
        } else {
          const int local = p - s_roff[r];
          if (local >= 0 && local < s_cap[r]) {
            dst = s_rx[r] + (uint64_t)local * rb;
            if (SCALES) sdst = s_rs[r] + (uint64_t)local * sp;
          } else {
            st |= MOE_STATUS_CAPACITY;
          }
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
    s_dst[wv][lane] = dst;
    if (SCALES) s_sdst[wv][lane] = sdst;
    __builtin_amdgcn_wave_barrier();

    for (int t = tb; t < te; ++t) {
      const int l0 = (t - tb) * k;
      const uint8_t* src = a.x + (int64_t)t * rb;
      const uint8_t* ssrc = SCALES ? a.x_scales + (int64_t)t * sb : nullptr;
      // Scale rows (pitch up to 1 KiB, sizes in 16-byte multiples) move with
      // the row: lane l carries bytes [16 l, 16 l + 16) of the pitched row,
      // scales first, zeros after.
      if (one_pass) {
        u32x4 v[VPL];
        u32x4 sv = {0u, 0u, 0u, 0u};
        if (pre_t == t) {
#pragma unroll
          for (int c = 0; c < VPL; ++c) v[c] = vn[c];
          sv = svn;
        } else {
          load_row(v, sv, t);
        }
        pre_t = t + 1 < t1 ? t + 1 : next;
        if (pre_t >= 0) load_row(vn, svn, pre_t);
        for (int j = 0; j < k; ++j) {
          uint8_t* d = reinterpret_cast<uint8_t*>(readlane64(s_dst[wv][l0 + j], 0));
          if (!d) continue;
#pragma unroll
          for (int c = 0; c < VPL; ++c) {
            const uint32_t off = c * kWaveBytes + l16;
            if (FULL || off < rb) store_row16<VPL>(d + off, v[c]);
          }
          if (s16) {
            uint8_t* sd = reinterpret_cast<uint8_t*>(readlane64(s_sdst[wv][l0 + j], 0));
            if (l16 < sp) store_row16<VPL>(sd + l16, sv);
          }
        }
      } else {
      u32x4 sv = {0u, 0u, 0u, 0u};
      if (s16 && l16 < sb) sv = ld16(ssrc + l16);
      for (uint32_t seg = 0; seg < rb; seg += VPL * kWaveBytes) {
        u32x4 v[VPL];
#pragma unroll
        for (int c = 0; c < VPL; ++c) {
          const uint32_t off = seg + c * kWaveBytes + l16;
          if (FULL || off < rb) v[c] = ld16(src + off);
        }
        for (int j = 0; j < k; ++j) {
          uint8_t* d = reinterpret_cast<uint8_t*>(readlane64(s_dst[wv][l0 + j], 0));
          if (!d) continue;
#pragma unroll
          for (int c = 0; c < VPL; ++c) {
            const uint32_t off = seg + c * kWaveBytes + l16;
            if (FULL || off < rb) store_row16<VPL>(d + off, v[c]);
          }
          if (s16 && seg == 0) {
            uint8_t* sd = reinterpret_cast<uint8_t*>(readlane64(s_sdst[wv][l0 + j], 0));
            if (l16 < sp) store_row16<VPL>(sd + l16, sv);
          }
        }
      }
      }
      if (SCALES && !s16) {
        // Other scale-row sizes: one float32 per lane per pass.
        for (uint32_t o = 0; o < sp; o += kWave * 4) {
          const uint32_t off = o + lane * 4;
          uint32_t s4 = 0;
          if (off < sb) s4 = ld4(ssrc + off);
          for (int j = 0; j < k; ++j) {
            uint8_t* d = reinterpret_cast<uint8_t*>(readlane64(s_sdst[wv][l0 + j], 0));
            if (d && off < sp) st4(d + off, s4);
          }
        }
      }
    }
  }
  });
  finish_parts<MODE>(a.tickets, g, W, lane);
  st = wave_or(st);
  if (st && lane == 0) atomicOr(a.status, st);
  trace_wave(a.trace, a.trace_waves, g, t_start, lane);
}

// Lane l's value of lane (l - n) mod 64, n wavefront-uniform.
__device__ __forceinline__ u32x4 rotate_up(u32x4 v, int n, int lane) {
  const int from = ((lane - n) & (kWave - 1)) * 4;
  u32x4 r;
  r.x = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)v.x);
  r.y = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)v.y);
  r.z = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)v.z);
  r.w = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)v.w);
  return r;
}

template <bool NT>
__device__ __forceinline__ void store16(void* p, u32x4 v) {
  if constexpr (NT)
    st16_stream(p, v);
  else
    st16(p, v);
}

// One wavefront per (token, 1 KiB slice of its row).
//
// Bound by HBM writes (one read per k writes).  What sets the rate is how
// many row stores are in flight over the chip: too few leave HBM idle, too
// many open more destination rows than its pages serve well, so the launch
// limits the resident wavefronts (launch_unit).  S: slices of S KiB, one
// 16-byte store per lane, KiB and destination; 1 KiB holds the fewest bytes per
// wavefront.
// Metadata is the token's k slots, one lane each, read by every slice (one
// line, from the caches); the destinations are read back by lane, so neither
// LDS nor a barrier is needed.  Measured on MI355X against the persistent
// split below (us before -> after, GB/s of algorithmic bytes after):
//   16384 x 14 KiB, k = 8, Zipf 1.2 routing   380 -> 361  (5860)
//   16384 x 14 KiB, k = 8, uniform            401 -> 399  (5300)
//   32768 x 8 KiB, k = 8, Zipf 1.5            443 -> 411  (5870)
//   16384 x 8 KiB, k = 8, uniform             221 -> 223  (5410)
//   8192 x 14 KiB, k = 16, uniform            508 -> 398  (5020)
//   4096 x 14 KiB, k = 8, uniform, x in HBM / cached   104 -> 101 / 92 -> 93
//   16384 x 2 KiB, k = 8, uniform             58 -> 50  (6040)
//   32768 x 512 B, k = 8                      36.5 -> 27.9  (5410)
//   512 x 14 KiB, k = 8                       22.6 -> 12.7
//   16384 x 7 KiB fp8, k = 8, uniform / Zipf  209 / 197 -> 205 / 195
// Slower: batches with most slots unused, whose wavefronts are bound by their
// metadata chain and, at 32768 x 14 KiB, by the launch of so many of them
// (half of the slots unused 457 -> 503, nine tenths 190 -> 287; at 4096 tokens
// 34 -> 38), and batches whose x the Infinity Cache holds whole (16384 x 14
// KiB, k = 8: 343 -> 359).
// NT: non-temporal stores.  CUT_NT: the same for rows that start inside a line.
//
// SCALES: the wavefront of slice 0 also carries the token's scale row: sized
// in 16-byte multiples and at most 1 KiB, its pitched bytes are spread over
// groups of `pieces` lanes, one group per destination, so one store
// instruction writes 64 / pieces scale rows whole.
//
// Destination rows that start inside a 128-byte line (rows that are no
// multiple of a line, or a region whose base is not on one): the slices of
// such a row are cut at its lines, so that no line is written in part by two
// wavefronts except where two rows meet.  Each lane's piece moves up by `cut`
// lanes through the LDS crossbar and the last pieces of the slice before it
// (pv, one 7-lane load, from the caches) come in from below; the last slice
// also stores the row's end.  Rows on the line whose region starts at half a
// line are left as they are: writing half lines measured as fast.  pv is
// requested with the slice where the row width says that it is needed, else
// only once a destination asks for it.  us on MI355X, persistent split (a row
// per wavefront) / uncut slices / this:
//   16384 x 14 KiB, k = 8, bases 16 / 64 bytes off  431 602 413 / 406 436 422
//   4096 x 14 KiB, k = 8, bases 16 bytes off        115 154 108
//   16384 x 8 KiB, k = 8, bases 16 / 64 off         243 345 259 / 231 249 237
//   16384 x 4 KiB, k = 8, bases 16 / 64 off         142 168 135 / 134 118 117
// and with the rows themselves off the line, persistent split / a load of its
// own per destination / this:
//   16384 x 14352 B, k = 8 / 2 / 1    437 414 418 / 151 198 141 / 96 159 95
//   16384 x 8208 B, k = 9 / 6         312 324 293 / 202 197 198
//   4770 x 6752 B, k = 6              41 50 39
//   16384 x 14400 B, k = 8            442 435 424 (an odd multiple of 64 bytes)
template <bool SCALES, bool NT, bool CUT_NT, int S>
__global__ __launch_bounds__(kBlock) void dispatch_unit_kernel(DispatchArgs a, int first,
                                                               int slices, int units) {
  const int lane = threadIdx.x & (kWave - 1);
  const int u = uniform(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave);
  if (u >= units) return;
  const int q = u % slices, t = first + u / slices;
  const uint32_t rb = (uint32_t)a.row_bytes;
  const uint32_t sb = (uint32_t)a.scale_row_bytes;
  const uint32_t sp = (uint32_t)a.scale_pitch;
  const int k = a.k;
  const uint32_t off = (uint32_t)q * (S * kWaveBytes) + lane * kVecBytes;
  int p = -1, e = 0;
  if (lane < k) {
    p = a.pos[(int64_t)t * k + lane];
    e = a.topk_idx[(int64_t)t * k + lane];
  }
  // v: this lane's piece of the slice; pv: the last pieces of the slice
  // before it, in the same lanes
  const uint8_t* row = a.x + (int64_t)t * rb;
  u32x4 v[S], pv = {0u, 0u, 0u, 0u}, sv = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int c = 0; c < S; ++c) {
    v[c] = u32x4{0u, 0u, 0u, 0u};
    if (off + c * kWaveBytes < rb) v[c] = ld16(row + off + c * kWaveBytes);
  }
  const bool before = q > 0 && lane >= kWave - (int)(kLine / kVecBytes - 1);
  const bool off_line = rb % kLine != 0;
  if (off_line && before) pv = ld16(row + off - kWaveBytes);
  const uint8_t* ssrc = SCALES ? a.x_scales + (int64_t)t * sb : nullptr;
  const bool scales_here = SCALES && q == 0;
  const int pieces = (int)sp / kVecBytes;
  const bool s16 = a.scales16;
  int sj = 0;           // this lane's destination within a group store
  uint32_t soff = 0;    // ... and its bytes of the scale row
  if (scales_here && s16) {
    sj = lane / pieces;
    soff = (uint32_t)(lane - sj * pieces) * kVecBytes;
    if (soff < sb) sv = ld16(ssrc + soff);
  }
  uint64_t dst = 0, sdst = 0;
  uint32_t st = 0;
  if (p >= 0) {
    const int r = e / a.L;
    if ((unsigned)r >= (unsigned)a.R) {
      st |= MOE_STATUS_BAD_INDEX;   // pos and topk_idx disagree: not copied
    } else {
      const int local = p - a.rank_offset[r];
      const int cap = a.recv_cap[r];
      const uint64_t rx = a.recv_x[r];
      uint64_t rs = 0;
      if (scales_here) rs = a.recv_scales[r];
      if (local >= 0 && local < cap) {
        dst = rx + (uint64_t)local * rb;
        sdst = rs + (uint64_t)local * sp;
      } else {
        st |= MOE_STATUS_CAPACITY;
      }
    }
  }
  // Bytes by which each destination row starts past its line, as far as they
  // matter: half a line does as well as none where rows are whole lines.
  const uint32_t in_line = off_line ? kLine - 1 : kLine / 2 - 1;
  if (!off_line && __any(((uint32_t)dst & in_line) != 0) && before)
    pv = ld16(row + off - kWaveBytes);
  for (int j = 0; j < k; ++j) {
    uint8_t* d = reinterpret_cast<uint8_t*>(readlane64(dst, j));
    if (!d) continue;
    const uint32_t past = (uint32_t)(uintptr_t)d % kLine;
    const int cut = past & in_line ? (int)(past / kVecBytes) : 0;
    if (cut == 0) {
#pragma unroll
      for (int c = 0; c < S; ++c) {
        const uint32_t o = off + c * kWaveBytes;
        if (o < rb) store16<NT>(d + o, v[c]);
      }
      continue;
    }
    // every lane's piece moves up by `cut` lanes; the last ones of the KiB
    // before it come in from below
#pragma unroll
    for (int c = 0; c < S; ++c) {
      const u32x4 r = rotate_up(lane + cut < kWave ? v[c] : c > 0 ? v[c > 0 ? c - 1 : 0] : pv, cut,
                                lane);
      const uint32_t o = off + c * kWaveBytes - cut * kVecBytes;   // wraps before the row's start
      if (o < rb) store16<CUT_NT>(d + o, r);
    }
    const uint32_t o = off + (S - 1) * kWaveBytes;
    if (q == slices - 1 && lane + cut >= kWave && o < rb) store16<CUT_NT>(d + o, v[S - 1]);
    // the two kinds of store are not joined, which would drop the hint of both
    if constexpr (NT != CUT_NT) __builtin_amdgcn_wave_barrier();
  }
  if (scales_here) {
    if (s16) {
      const int per = kWave / pieces;
      for (int j0 = 0; j0 < k; j0 += per) {
        const int j = j0 + sj;
        uint8_t* d = reinterpret_cast<uint8_t*>(
            __shfl((unsigned long long)sdst, j & (kWave - 1), kWave));
        if (sj < per && j < k && d) store16<NT>(d + soff, sv);
      }
    } else {
      // other scale-row sizes: one float32 per lane per pass
      for (uint32_t o = 0; o < sp; o += kWave * 4) {
        const uint32_t so = o + lane * 4;
        uint32_t s4 = 0;
        if (so < sb) s4 = ld4(ssrc + so);
        for (int j = 0; j < k; ++j) {
          uint8_t* d = reinterpret_cast<uint8_t*>(readlane64(sdst, j));
          if (d && so < sp) st4(d + so, s4);
        }
      }
    }
  }
  if (q == 0) {   // one wavefront reports a token
    st = wave_or(st);
    if (st && lane == 0) atomicOr(a.status, st);
  }
}

template <bool SCALES, bool NT, int S, bool CUT_NT = NT>
hipError_t launch_unit_as(const DispatchArgs& a, int waves, int wpb, hipStream_t stream) {
  const int slices = (int)((row_slices(a.row_bytes) + S - 1) / S);
  const unsigned lds = wave_limit_lds(waves, wpb);
  return launch_token_ranges(a.tokens, slices, [&](int first, int units) {
    hipLaunchKernelGGL((dispatch_unit_kernel<SCALES, NT, CUT_NT, S>),
                       dim3((units + wpb - 1) / wpb), dim3(wpb * kWave), lds, stream, a, first,
                       slices, units);
  });
}

// Bytes of x and of the rows written that the 256 MiB Infinity Cache takes in:
// up to here ordinary stores end in it, and beyond non-temporal ones are the
// better choice; from kAbsorbedMin on they gain (below, a launch is too short,
// and a step of 777 x 4112 B, k = 6, 1 us longer for the write-back at its end).
constexpr int64_t kAbsorbedMin = 96ll << 20, kAbsorbedMax = 300ll << 20;

// How the units are launched.  What bounds a batch is, by size: launch latency
// and the metadata chain (small ones), the Infinity Cache (up to
// kAbsorbedMax), HBM writes (beyond).  All figures us on MI355X with x from
// HBM / re-read from the caches, "persistent" the split of launch_scales.
//
// 1. Rows under 1 KiB (a partly filled wavefront each): every wavefront
//    resident, workgroups of four.  32768 x 512 B, k = 8: persistent 37 / 27,
//    12 resident wavefronts 32 / 28, this 28 / 27; 65536 x 256 B, k = 8: 49 56
//    32.  Rows off the line take ordinary stores (rows that share a line meet
//    in L2: 32768 x 528 B, k = 8: persistent 43, non-temporal 49, this 36), and so
//    does every destination that starts inside a line.
// 2. Batches that the Infinity Cache absorbs, and smaller ones of rows under 2
//    KiB off the line (8192 x 1040 B, k = 8: 16 22 15): ordinary stores, slices
//    of 2 KiB, workgroups of four, 24 wavefronts (32 for fewer than 4 rows a
//    token and for rows off the line, whose lives are longer).  Against the
//    persistent split and non-temporal 1 KiB units:
//      16384 x 2 KiB, k = 8    57 / 64   58 / 54   50 / 51
//      4096 x 4 KiB, k = 8     26 / 25   28 / 27   26 / 24
//      4096 x 8 KiB, k = 8     50 / 51   57 / 52   49 / 50
//      32768 x 2 KiB, k = 2    36 / 33   42 / 33   35 / 32
//      16384 x 8 KiB, k = 1    46 / 45   54 / 47   44 / 41
//      8192 x 2 KiB fp8, k = 8 27 / 26   33 / 32   27 / 26
//      4096 x 7 KiB fp8, k = 8 45 / 46   52 / 50   45 / 47
//      4096 x 6752 B, k = 6    32 / 30   43 / 36   33 / 31
// 3. Other bf16 batches: non-temporal 1 KiB units (2 KiB for one row a token,
//    whose wavefronts hold least: 16384 x 14 KiB, k = 1: 91 / 81 -> 90 / 70).
//    About 112 KiB of stores in flight per compute unit for 8 rows a token (14
//    wavefronts), more wavefronts for fewer, in workgroups of two.  k = 8,
//    persistent / workgroups of one, 12 wavefronts / of two, 12 / of two, 14 /
//    of two, 16:
//      16384 x 14 KiB, uniform   399 408 390 398 407      Zipf  377 365 374 359 375
//      16384 x 10 KiB, uniform   285 289 277 276 286
//      16384 x 8 KiB, uniform    221 226 224 223 -        Zipf  216 209 216 208 -
//      16384 x 4 KiB, uniform    121 113 113 110 113      Zipf  121 107 110 107 110
//      4096 x 14 KiB, uniform    104 105 100 101 104      Zipf  98 95 97 94 95
//      with x re-read from the caches, 16384 x 14 KiB  344 364 359 358 358
//    k = 4, 14 KiB: persistent 231, 18 wavefronts 221, 14 237; k = 2: 145,
//    32 130, 14 163; k = 16 (8192 tokens): 506, 14 394.
//    Rows off the line want every wavefront (16384 x 8240 B, k = 4, at 32 /
//    20 / 12: 155 173 201), large batches of them in workgroups of one (16384 x
//    8256 B, k = 8: 239, of two 249).
// 4. fp8 rows, whose slice-0 wavefront lives longer, in workgroups of four (16384
//    x 4 KiB, k = 8: of one 131, of two 130, of four 118): rows of more than 4
//    KiB of an x that the Infinity Cache does not keep from the kernel that
//    wrote it (over 64 MiB) with ordinary stores and 16 wavefronts, else
//    non-temporal and 12.  k = 8, persistent / ordinary / non-temporal:
//      16384 x 7 KiB, uniform    209 205 209   (x cached 207 203 194)
//      16384 x 7 KiB, Zipf       197 195 192
//      16384 x 5 KiB, uniform    163 150 154   (162 150 139), Zipf 159 146 142
//      8192 x 7 KiB, uniform     111 107 110   (107 104 97), Zipf 103 100 97
//      16384 x 4 KiB, uniform    126 125 118   (125 124 104)
//      32768 x 7 KiB, uniform    425 414 417, Zipf 407 387 380
template <bool SCALES>
hipError_t launch_unit(const DispatchArgs& a, hipStream_t stream) {
  const int64_t rows = a.rows_hint > 0 ? a.rows_hint : a.k;   // pair rows: half the slots
  const int64_t x_bytes = a.tokens * a.row_bytes, touched = x_bytes * (a.k + 1);
  const bool off_line = a.row_bytes % kLine != 0;
  if (a.row_bytes < kWaveBytes)
    return off_line ? launch_unit_as<SCALES, false, 1>(a, 32, kWavesPerBlock, stream)
                    : launch_unit_as<SCALES, true, 1, false>(a, 32, kWavesPerBlock, stream);
  if (touched <= kAbsorbedMax &&
      (touched >= kAbsorbedMin || (off_line && a.row_bytes < 2 * kWaveBytes)))
    return launch_unit_as<SCALES, false, 2>(a, rows < 4 || off_line ? 32 : 24, kWavesPerBlock,
                                            stream);
  const int waves = off_line ? 32 : rows < 8 ? (int)(48 / rows) + 6 : SCALES ? 12 : 14;
  if (SCALES && rows >= 8 && a.row_bytes > 4 * kWaveBytes && x_bytes > (64ll << 20))
    return launch_unit_as<SCALES, false, 1>(a, 16, kWavesPerBlock, stream);
  const int wpb = SCALES ? kWavesPerBlock
                  : !off_line ? 2
                              : touched < kAbsorbedMin ? kWavesPerBlock : 1;
  if (rows == 1) return launch_unit_as<SCALES, true, 2>(a, 32, wpb, stream);
  return launch_unit_as<SCALES, true, 1>(a, waves, wpb, stream);
}

// Pull dispatch for the partitioning study: a wavefront walks a range of
// global (destination) rows and pulls each row's source token from x.
// POLICY MOE_POLICY_ROWS: the N routed rows are split evenly over the W
// wavefronts.  MOE_POLICY_BY_RANK: wavefronts form R fixed groups of W/R
// and group r splits rank r's rows (a per-peer core assignment that ignores
// how many rows each rank receives).  Per batch of 64 rows, lane l resolves
// row ib+l (source row, destination) into LDS, as the push kernel does.
template <int VPL, bool FULL, bool SCALES, int POLICY>
__global__ __launch_bounds__(kBlock) void dispatch_pull_kernel(DispatchArgs a) {
  __shared__ uint64_t s_src[kWavesPerBlock][kWave];
  __shared__ uint64_t s_dst[kWavesPerBlock][kWave];
  __shared__ uint64_t s_ssrc[kWavesPerBlock][SCALES ? kWave : 1];
  __shared__ uint64_t s_sdst[kWavesPerBlock][SCALES ? kWave : 1];
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = threadIdx.x / kWave;
  const int g = uniform(blockIdx.x * kWavesPerBlock + wv);
  const uint64_t t_start = a.trace ? (uint64_t)wall_clock64() : 0;
  const int W = gridDim.x * kWavesPerBlock;
  const uint32_t rb = (uint32_t)a.row_bytes;
  const uint32_t sb = (uint32_t)a.scale_row_bytes;
  const uint32_t sp = (uint32_t)a.scale_pitch;
  const uint32_t l16 = lane * kVecBytes;
  int64_t i0 = 0, i1 = 0;
  if (POLICY == MOE_POLICY_ROWS) {
    const int64_t n = a.rank_offset[a.R];
    i0 = n * g / W;
    i1 = n * (g + 1) / W;
  } else {
    const int G = W / a.R;  // the launch makes W a multiple of R
    const int r = g / G, q = g - r * G;
    if (r < a.R) {
      const int64_t b = a.rank_offset[r], n = a.rank_offset[r + 1] - b;
      i0 = b + n * q / G;
      i1 = b + n * (q + 1) / G;
    }
  }
  // rows and their sources stay inside the batch whatever the layout left
  const int64_t n_slots = a.tokens * a.k;
  i0 = max(i0, (int64_t)0);
  i1 = min(i1, n_slots);
  uint32_t st = 0;
  for (int64_t ib = i0; ib < i1; ib += kWave) {
    const int64_t ie = min(i1, ib + kWave);
    uint64_t src = 0, dst = 0, ssrc = 0, sdst = 0;
    if (ib + lane < ie) {
      const int64_t i = ib + lane;
      const int s = a.row_src[i];
      const bool known = s >= 0 && s < n_slots;
      const int t = known ? s / a.k : 0;
      const int r = known ? a.topk_idx[s] / a.L : -1;
      const int64_t local = (unsigned)r < (unsigned)a.R ? i - a.rank_offset[r] : -1;
      if (!known || (unsigned)r >= (unsigned)a.R) {
        st |= MOE_STATUS_BAD_INDEX;
      } else if (local >= 0 && local < a.recv_cap[r]) {
        src = reinterpret_cast<uint64_t>(a.x) + (uint64_t)t * rb;
        dst = a.recv_x[r] + (uint64_t)local * rb;
        if (SCALES) {
          ssrc = reinterpret_cast<uint64_t>(a.x_scales) + (uint64_t)t * sb;
          sdst = a.recv_scales[r] + (uint64_t)local * sp;
        }
      } else {
        st |= MOE_STATUS_CAPACITY;
      }
    }
    __builtin_amdgcn_wave_barrier();
    s_src[wv][lane] = src;
    s_dst[wv][lane] = dst;
    if (SCALES) {
      s_ssrc[wv][lane] = ssrc;
      s_sdst[wv][lane] = sdst;
    }
    __builtin_amdgcn_wave_barrier();
    for (int l = 0; l < (int)(ie - ib); ++l) {
      const uint8_t* sr = reinterpret_cast<const uint8_t*>(readlane64(s_src[wv][l], 0));
      uint8_t* d = reinterpret_cast<uint8_t*>(readlane64(s_dst[wv][l], 0));
      if (!d) continue;
      for (uint32_t seg = 0; seg < rb; seg += VPL * kWaveBytes) {
        u32x4 v[VPL];
#pragma unroll
        for (int c = 0; c < VPL; ++c) {
          const uint32_t off = seg + c * kWaveBytes + l16;
          if (FULL || off < rb) v[c] = ld16(sr + off);
        }
#pragma unroll
        for (int c = 0; c < VPL; ++c) {
          const uint32_t off = seg + c * kWaveBytes + l16;
          if (FULL || off < rb) st16(d + off, v[c]);
        }
      }
      if (SCALES) {
        const uint8_t* ss = reinterpret_cast<const uint8_t*>(readlane64(s_ssrc[wv][l], 0));
        uint8_t* sd = reinterpret_cast<uint8_t*>(readlane64(s_sdst[wv][l], 0));
        for (uint32_t o = 0; o < sp; o += kWave * 4) {
          const uint32_t off = o + lane * 4;
          uint32_t s4 = 0;
          if (off < sb) s4 = ld4(ss + off);
          if (off < sp) st4(sd + off, s4);
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  st = wave_or(st);
  if (st && lane == 0) atomicOr(a.status, st);
  trace_wave(a.trace, a.trace_waves, g, t_start, lane);
}

template <int VPL, bool FULL, bool SCALES, int POLICY>
hipError_t launch_pull(DispatchArgs a, hipStream_t stream) {
  const void* fn = reinterpret_cast<const void*>(&dispatch_pull_kernel<VPL, FULL, SCALES, POLICY>);
  int waves = a.launch_waves > 0 ? a.launch_waves : resident_waves(fn, 0);
  if (POLICY == MOE_POLICY_BY_RANK && a.launch_waves == 0) {
    // whole groups per rank, and whole workgroups
    waves = waves / a.R * a.R;
    while (waves > a.R && waves % kWavesPerBlock != 0) waves -= a.R;
    if (waves < a.R || waves % kWavesPerBlock != 0) waves = a.R * kWavesPerBlock;
  }
  hipLaunchKernelGGL((dispatch_pull_kernel<VPL, FULL, SCALES, POLICY>),
                     dim3(waves / kWavesPerBlock), dim3(kBlock), 0, stream, a);
  return hipGetLastError();
}

template <int VPL, bool SCALES, int MODE>
hipError_t launch_push_as(const DispatchArgs& a, int waves, bool full, hipStream_t stream) {
  const dim3 grid(waves / kWavesPerBlock), block(kBlock);
  if (full)
    hipLaunchKernelGGL((dispatch_kernel<VPL, true, SCALES, MODE>), grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL((dispatch_kernel<VPL, false, SCALES, MODE>), grid, block, 0, stream, a);
  return hipGetLastError();
}

template <int VPL, bool SCALES, int MODE>
hipError_t launch_push(DispatchArgs a, hipStream_t stream, bool all_static = false);

template <int VPL, bool SCALES>
hipError_t launch_vpl(DispatchArgs a, int policy, hipStream_t stream) {
  const bool full = a.row_bytes == (int64_t)VPL * kWaveBytes;
  if (policy == MOE_POLICY_ROWS)
    return full ? launch_pull<VPL, true, SCALES, MOE_POLICY_ROWS>(a, stream)
                : launch_pull<VPL, false, SCALES, MOE_POLICY_ROWS>(a, stream);
  if (policy == MOE_POLICY_BY_RANK)
    return full ? launch_pull<VPL, true, SCALES, MOE_POLICY_BY_RANK>(a, stream)
                : launch_pull<VPL, false, SCALES, MOE_POLICY_BY_RANK>(a, stream);
  const int64_t rows = a.rows_hint > 0 ? a.rows_hint : a.k;
  if (policy == MOE_POLICY_DYNAMIC ||
      (policy == MOE_POLICY_BALANCED &&
       claim_all_parts(a.tokens, a.row_bytes, rows, kClaimAllDispatchPartBytes)))
    return launch_push<VPL, SCALES, kPartsClaimed>(a, stream);
  return launch_push<VPL, SCALES, kPartsHybrid>(a, stream, policy == MOE_POLICY_STATIC);
}

template <int VPL, bool SCALES, int MODE>
hipError_t launch_push(DispatchArgs a, hipStream_t stream, bool all_static) {
  const bool full = a.row_bytes == (int64_t)VPL * kWaveBytes;
  const void* fn =
      full ? reinterpret_cast<const void*>(&dispatch_kernel<VPL, true, SCALES, MODE>)
           : reinterpret_cast<const void*>(&dispatch_kernel<VPL, false, SCALES, MODE>);
  const int64_t rows = a.rows_hint > 0 ? a.rows_hint : a.k;
  const int waves = a.launch_waves > 0
                        ? a.launch_waves
                        : copy_waves(fn, rows * a.row_bytes, kDispatchInFlight, 256);
  // The run-time share pays one serialized counter claim per two parts; it
  // only pays off while each wavefront owns several parts.
  if (MODE == kPartsHybrid && (all_static || MOE_PLAN_PARTS / waves < 8))
    return launch_push_as<VPL, SCALES, kPartsStatic>(a, waves, full, stream);
  return launch_push_as<VPL, SCALES, MODE>(a, waves, full, stream);
}

template <bool SCALES>
hipError_t launch_scales(const DispatchArgs& a, int policy, hipStream_t stream) {
  const int64_t segs = (a.row_bytes + kWaveBytes - 1) / kWaveBytes;
  switch (segs) {
    case 1: return launch_vpl<1, SCALES>(a, policy, stream);
    case 2: return launch_vpl<2, SCALES>(a, policy, stream);
    case 3: return launch_vpl<3, SCALES>(a, policy, stream);
    case 4: return launch_vpl<4, SCALES>(a, policy, stream);
    case 5: return launch_vpl<5, SCALES>(a, policy, stream);
    case 6: return launch_vpl<6, SCALES>(a, policy, stream);
    case 7: return launch_vpl<7, SCALES>(a, policy, stream);
    case 8: return launch_vpl<8, SCALES>(a, policy, stream);
    case 9: return launch_vpl<9, SCALES>(a, policy, stream);
    case 10: return launch_vpl<10, SCALES>(a, policy, stream);
    case 11: return launch_vpl<11, SCALES>(a, policy, stream);
    case 12: return launch_vpl<12, SCALES>(a, policy, stream);
    case 13: return launch_vpl<13, SCALES>(a, policy, stream);
    case 14: return launch_vpl<14, SCALES>(a, policy, stream);
    case 15: return launch_vpl<15, SCALES>(a, policy, stream);
    default: return launch_vpl<kMaxSegVecs, SCALES>(a, policy, stream);
  }
}

}  // namespace

// Rows of less than a line fill so little of a wavefront that the launch of one
// per token bounds the units: they keep the persistent split, static parts
// (262144 x 16 B, k = 1: units 66 us, persistent 40; 32768 x 16 B, k = 8: 18,
// 16.5; 131072 x 128 B, k = 8: 58, 72).
hipError_t launch_dispatch(const DispatchArgs& a, int policy, hipStream_t stream) {
  if (policy == MOE_POLICY_BALANCED && a.launch_waves == 0 && !a.trace) {
    if (a.row_bytes >= kLine)
      return a.x_scales ? launch_unit<true>(a, stream) : launch_unit<false>(a, stream);
    policy = MOE_POLICY_STATIC;
  }
  return a.x_scales ? launch_scales<true>(a, policy, stream)
                    : launch_scales<false>(a, policy, stream);
}

}  // namespace moe
