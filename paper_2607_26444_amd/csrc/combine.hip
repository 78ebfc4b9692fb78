// Combine: y[t] = bf16( sum_j w[t,j] * Y(row of slot j) ).
//
// Default split (combine_unit_kernel): one wavefront per (token, 1 KiB slice
// of its row) unit, launched in token order; the hardware hands units out as
// wavefronts retire.  A wavefront resolves its token's k slots one per lane,
// issues the k gathers of its slice together, multiplies and adds in float32
// in slot order and stores the slice of y.  Each output byte has exactly one
// writer, so the reduction needs no atomics (Section 6.1 accumulates on chip
// and writes back once).  Gathers and stores are non-temporal: every byte is
// touched once.
//
// Explicit splits (combine_kernel; moe_combine_ex with a policy, a wavefront
// count or a trace), and large batches of few narrow rows: persistent
// wavefronts over the byte-balanced plan (wavefront g of W takes parts g,
// g + W, ... or claims them at run time).  Slot metadata for a batch of 64/k
// tokens is resolved once, one slot per lane, and parked in LDS; for each token
// the wavefront walks the output row in 1 KiB segments, the next segment's
// gathers issued before the current one is reduced.  Output rows of 8-16 KiB
// are kept in registers and stored as one burst per token.  Unused and
// capacity-dropped slots are redirected to a routed row of the same token,
// their data is zeroed bitwise and their weight is 0 (a plain multiply
// by 0 would turn an Inf in that row into NaN).

#include "moe_internal.h"

namespace moe {
namespace {

template <int KW>
__device__ __forceinline__ void gather(u32x4 (&v)[KW], const uint8_t* const (&src)[KW],
                                       uint32_t off) {
#pragma unroll
  for (int j = 0; j < KW; ++j) v[j] = ld16_stream(src[j] + off);
}

// Weighted sum of one 1 KiB segment.  MASKED: unused slots read a routed
// row of the same token; their data is zeroed (bitwise, so an Inf or NaN
// there cannot leak) and their weight is 0.
template <int KW, bool MASKED>
__device__ __forceinline__ u32x4 reduce(const u32x4 (&v)[KW], const float (&wt)[KW],
                                        const uint32_t (&keep)[KW]) {
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < KW; ++j) {
    u32x4 x = v[j];
    if (MASKED) {
      x.x &= keep[j];
      x.y &= keep[j];
      x.z &= keep[j];
      x.w &= keep[j];
    }
    fma8(acc, x, wt[j]);
  }
  return pack8(acc);
}

// One token's output row: full 1 KiB segments two at a time, then the
// ragged tail.  The gathers of the next segment are issued before the
// current one is reduced and stored, so waiting for them never waits for a
// store (vector memory operations complete in issue order on this counter).
template <int KW, bool MASKED>
__device__ __forceinline__ void combine_row(uint8_t* dst, const uint8_t* const (&src)[KW],
                                            const float (&wt)[KW],
                                            const uint32_t (&keep)[KW], uint32_t rb,
                                            uint32_t l16) {
  const uint32_t nf = rb / kWaveBytes, tail = rb % kWaveBytes;
  u32x4 a[KW], b[KW];
  uint32_t o = l16;
  if (nf > 0) gather<KW>(a, src, o);
  for (uint32_t s = 0; s + 2 <= nf; s += 2) {
    gather<KW>(b, src, o + kWaveBytes);
    st16_stream(dst + o, reduce<KW, MASKED>(a, wt, keep));
    if (s + 2 < nf) gather<KW>(a, src, o + 2 * kWaveBytes);
    st16_stream(dst + o + kWaveBytes, reduce<KW, MASKED>(b, wt, keep));
    o += 2 * kWaveBytes;
  }
  if (nf & 1u) {
    st16_stream(dst + o, reduce<KW, MASKED>(a, wt, keep));
    o += kWaveBytes;
  }
  if (l16 < tail) {
    gather<KW>(a, src, o);
    st16_stream(dst + o, reduce<KW, MASKED>(a, wt, keep));
  }
}

// Stores of one output row held in registers (segment s at byte
// l16 + s KiB; lanes past the row end store nothing).
template <int NSEG>
__device__ __forceinline__ void store_row(uint8_t* dst, const u32x4 (&yr)[NSEG], uint32_t rb,
                                          uint32_t l16) {
#pragma unroll
  for (int s = 0; s < NSEG; ++s) {
    const uint32_t o = l16 + (uint32_t)s * kWaveBytes;
    if (o < rb) st16_stream(dst + o, yr[s]);
  }
}

// One token's output row of at most NSEG KiB, reduced into registers
// (ceil(rb / 1 KiB) segments, the last one partial when rb is not a
// multiple of 1 KiB) with the gathers two segments ahead as in combine_row,
// then stored as one burst.  Always masked: the unrolled row is large, and the
// mask is four ANDs per slot and segment (all ones for routed slots).
template <int KW, int NSEG>
__device__ __forceinline__ void combine_row_burst(uint8_t* dst, const uint8_t* const (&src)[KW],
                                                  const float (&wt)[KW],
                                                  const uint32_t (&keep)[KW], uint32_t rb,
                                                  uint32_t l16) {
  const uint32_t ns = (rb + kWaveBytes - 1) / kWaveBytes;
  u32x4 v[2][KW], yr[NSEG];
  if (l16 < rb) gather<KW>(v[0], src, l16);
#pragma unroll
  for (int s = 0; s < NSEG; ++s) {
    if ((uint32_t)s < ns) {
      const uint32_t on = l16 + (uint32_t)(s + 1) * kWaveBytes;
      if (on < rb) gather<KW>(v[(s + 1) & 1], src, on);
      yr[s] = reduce<KW, true>(v[s & 1], wt, keep);
    }
  }
  store_row<NSEG>(dst, yr, rb, l16);
}

// KW: slots resolved per token (>= k).  NSEG > 0: rows of at most NSEG KiB,
// each held in registers and stored as one burst (combine_row_burst).
template <int KW, bool DYN, int NSEG>
__global__ __launch_bounds__(kBlock) void combine_kernel(CombineArgs a) {
  // Per-slot source row and weight of the current batch, one entry per lane
  // of each wavefront (0 = slot not combined), padded with zeros so a token
  // can read KW entries without a bounds test.
  __shared__ uint64_t s_src[kWavesPerBlock][kWave + MOE_MAX_K];
  __shared__ float s_w[kWavesPerBlock][kWave + MOE_MAX_K];
  // Under run-time claiming (large parts) the per-rank tables (first global
  // row, capacity, region base) are staged in LDS once per workgroup, so a
  // slot's source row is an LDS lookup behind its pos and expert loads.
  // Measured on MI355X in whole steps: combine 0.25-0.3% faster at prefill,
  // fp8 and large; 0.3-0.6 us slower at decode (static split, 2048
  // wavefronts), which keeps the global loads.
  __shared__ int32_t s_roff[DYN ? MOE_MAX_EXPERTS : 1];
  __shared__ int32_t s_cap[DYN ? MOE_MAX_EXPERTS : 1];
  __shared__ uint64_t s_ry[DYN ? MOE_MAX_EXPERTS : 1];
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = threadIdx.x / kWave;
  const int g = uniform(blockIdx.x * kWavesPerBlock + wv);
  const uint64_t t_start = a.trace ? (uint64_t)wall_clock64() : 0;
  if constexpr (DYN) {
    for (int i = threadIdx.x; i < a.R; i += kBlock) {
      s_roff[i] = a.rank_offset[i];
      s_cap[i] = a.recv_cap[i];
      s_ry[i] = a.expert_y[i];
    }
    __syncthreads();
  }
  const int W = gridDim.x * kWavesPerBlock;
  const uint32_t rb = (uint32_t)a.row_bytes;
  const uint32_t l16 = lane * kVecBytes;
  const int k = a.k;
  const int tpb = kWave / k;        // tokens whose slots fit one lane each
  const int lt = lane / k;          // this lane's token within a batch
  const int lj = lane - lt * k;     // ... and its slot
  uint32_t st = 0;
  if (lane < MOE_MAX_K) {
    s_src[wv][kWave + lane] = 0;
    s_w[wv][kWave + lane] = 0.0f;
  }

  const int T = (int)a.tokens;
  for_each_part<DYN ? kPartsClaimed : kPartsStatic>(a.bound, a.tickets, g, W, lane,
                                                     [&](int t0, int t1) {
  // token ranges stay inside the batch whatever the plan holds (a layout
  // whose barrier timed out leaves parts of it unwritten)
  t0 = max(t0, 0);
  t1 = min(t1, T);
  for (int tb = t0; tb < t1; tb += tpb) {
    const int te = min(t1, tb + tpb);
    uint64_t srow = 0;
    float wl = 0.0f;
    if (tb + lt < te) {
      const int64_t s = (int64_t)(tb + lt) * k + lj;
      const int p = a.pos[s];
      if (p >= 0) {
        const int r = a.topk_idx[s] / a.L;
        if ((unsigned)r >= (unsigned)a.R) {
          st |= MOE_STATUS_BAD_INDEX;   // pos and topk_idx disagree: weight 0
        } else {
          const int local = p - (DYN ? s_roff[r] : a.rank_offset[r]);
          if (local >= 0 && local < (DYN ? s_cap[r] : a.recv_cap[r])) {
            srow = (DYN ? s_ry[r] : a.expert_y[r]) + (uint64_t)local * (uint64_t)rb;
            wl = a.topk_w ? a.topk_w[s] : 1.0f;   // null: unit weights
          } else {
            st |= MOE_STATUS_CAPACITY;
          }
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
    s_src[wv][lane] = srow;
    s_w[wv][lane] = wl;
    __builtin_amdgcn_wave_barrier();

    for (int t = tb; t < te; ++t) {
      const int l0 = (t - tb) * k;
      const uint8_t* src[KW];
      float wt[KW];
      uint32_t keep[KW];
      uint64_t first = 0;
      bool all = true;
#pragma unroll
      for (int j = KW - 1; j >= 0; --j) {
        uint64_t sp = readlane64(s_src[wv][l0 + j], 0);
        const float w = readlane_f32(s_w[wv][l0 + j], 0);
        sp = (j < k) ? sp : 0;
        src[j] = reinterpret_cast<const uint8_t*>(sp);
        wt[j] = sp ? w : 0.0f;
        keep[j] = sp ? 0xFFFFFFFFu : 0u;
        all = all && sp;
        first = sp ? sp : first;
      }
      uint8_t* dst = reinterpret_cast<uint8_t*>(a.y) + (int64_t)t * rb;
      if (!first) {  // no routed slot: y = +0
        for (uint32_t off = l16; off < rb; off += kWaveBytes)
          st16_stream(dst + off, u32x4{0u, 0u, 0u, 0u});
        continue;
      }
      if (!all) {
#pragma unroll
        for (int j = 0; j < KW; ++j)
          if (!keep[j]) src[j] = reinterpret_cast<const uint8_t*>(first);
      }
      if constexpr (NSEG > 0) {
        combine_row_burst<KW, NSEG>(dst, src, wt, keep, rb, l16);
      } else if (all) {
        combine_row<KW, false>(dst, src, wt, keep, rb, l16);
      } else {
        combine_row<KW, true>(dst, src, wt, keep, rb, l16);
      }
    }
  }
  });
  finish_parts<DYN ? kPartsClaimed : kPartsStatic>(a.tickets, g, W, lane);
  st = wave_or(st);
  if (st && lane == 0) atomicOr(a.status, st);
  trace_wave(a.trace, a.trace_waves, g, t_start, lane);
}

template <int KW, bool DYN, int NSEG>
hipError_t launch_kw(CombineArgs a, int64_t in_flight, hipStream_t stream) {
  const void* fn = reinterpret_cast<const void*>(&combine_kernel<KW, DYN, NSEG>);
  // KW gathers of 1 KiB for each of the two segments in flight
  const int waves = a.launch_waves > 0
                        ? a.launch_waves
                        : copy_waves(fn, 2ll * KW * kWaveBytes, in_flight, 512);
  hipLaunchKernelGGL((combine_kernel<KW, DYN, NSEG>), dim3(waves / kWavesPerBlock),
                     dim3(kBlock), 0, stream, a);
  return hipGetLastError();
}

// Output rows of 8 to 16 KiB (4096 <= H <= 8192 bf16) are stored as one
// burst from registers: on MI355X this measured 2-6% faster at H = 7168 and
// ~1% faster at H = 4096 (where parts are claimed at run time); narrower
// rows, wider rows and slot widths above 8 (whose gathers already fill the
// registers) store each segment as it is reduced.
constexpr int kBurstSegs = 16;

template <int KW, bool DYN>
hipError_t launch_rows(const CombineArgs& a, int64_t in_flight, hipStream_t stream) {
  if (KW <= 8 && a.row_bytes >= 8ll * kWaveBytes &&
      a.row_bytes <= (int64_t)kBurstSegs * kWaveBytes)
    return launch_kw<KW, DYN, (KW <= 8 ? kBurstSegs : 0)>(a, in_flight, stream);
  return launch_kw<KW, DYN, 0>(a, in_flight, stream);
}

template <bool DYN>
hipError_t launch_dyn(const CombineArgs& a, int64_t in_flight, hipStream_t stream) {
  switch (slot_width(a.k)) {
    case 2: return launch_rows<2, DYN>(a, in_flight, stream);
    case 4: return launch_rows<4, DYN>(a, in_flight, stream);
    case 8: return launch_rows<8, DYN>(a, in_flight, stream);
    case 16: return launch_rows<16, DYN>(a, in_flight, stream);
    default: return launch_rows<32, DYN>(a, in_flight, stream);
  }
}

// One wavefront per (token, slice of S KiB of its row); KB: slots gathered
// together (k when k <= 8, else 8 at a time).
//
// Bound by HBM reads (k gathers per store).  As in dispatch the number of
// bytes in flight over the chip sets the rate, from both sides, so the launch
// limits the resident wavefronts (gather_unit_waves) and a slice is as
// narrow as keeps a few gathers in flight per wavefront: S = 1 from k = 3,
// at most 2 for k = 2 and 4 for k = 1 (16384 x 14 KiB on MI355X, us at S = 1 / 2 / 4:
// k = 1 120 87 84, k = 2 133 118 119, k = 4 192 196 201, k = 8 340 360 360).
// Slots are read through buffer resources: an unused or capacity-dropped
// slot's resource has an empty range, so its load returns +0 without touching
// memory, and so does the part of a slice past the row's end.  Measured on
// MI355X against the persistent split below (us before -> after, GB/s of
// algorithmic bytes after):
//   16384 x 14 KiB, k = 8, Zipf 1.2 routing   366 -> 334  (6330)
//   32768 x 8 KiB, k = 8, Zipf 1.5            431 -> 392  (6160)
//   8192 x 14 KiB, k = 16, uniform            444 -> 338  (5900)
//   16384 x 10 KiB, k = 6, uniform            221 -> 196  (5990)
//   4096 x 14 KiB, k = 8, uniform             90.3 -> 88.0 (6010)
//   32768 x 512 B, k = 8                      44.4 -> 28.3 (5340)
//   16384 x 14 KiB, k = 1, uniform            104 -> 80  (5850)
//   512 x 14 KiB, k = 8                       25.7 -> 13.0
//
// group > 0: tokens go to the XCDs in groups of that many neighbours
// (workgroups are placed on the eight XCDs in turn), so one XCD's L2 fetches
// a group's slot metadata once, instead of every XCD fetching the line for
// its few slices.  Groups of 4 (k = 8: one 128-byte line of each array)
// measured 16384 x 14 KiB Zipf 342 -> 334 us, uniform 358 -> 352, 32768 x 8
// KiB Zipf 405 -> 392, 4096 x 14 KiB 88.2 -> 87.9; 1 and 2 gain half to two
// thirds of that.  Dispatch, whose rows want to be written by all XCDs at
// once, got 2-16% slower that way and the partial combine did not change.
constexpr int kXcds = 8;
constexpr int kXcdGroup = 4;
template <int KB, int S>
__global__ __launch_bounds__(kBlock) void combine_unit_kernel(CombineArgs a, int first,
                                                              int slices, int units,
                                                              int group) {
  const int lane = threadIdx.x & (kWave - 1);
  int q, t;
  if (group > 0) {
    // workgroup b runs on XCD b % kXcds: unit `u` of that XCD's own sequence
    const int x = blockIdx.x % kXcds;
    const int u = uniform(blockIdx.x / kXcds * kWavesPerBlock + threadIdx.x / kWave);
    const int n = u / slices;   // n-th token of this XCD
    q = u % slices;
    t = (n / group * kXcds + x) * group + n % group;
    if (t >= units / slices) return;
  } else {
    const int u = uniform(blockIdx.x * kWavesPerBlock + threadIdx.x / kWave);
    if (u >= units) return;
    q = u % slices;
    t = u / slices;
  }
  t += first;
  const uint32_t rb = (uint32_t)a.row_bytes;
  const int k = a.k;
  const uint32_t o0 = (uint32_t)q * (S * kWaveBytes) + lane * kVecBytes;
  int p = -1, e = 0;
  float w = 1.0f;   // null weights: unit weights
  if (lane < k) {
    const int64_t s = (int64_t)t * k + lane;
    p = a.pos[s];
    e = a.topk_idx[s];
    if (a.topk_w) w = a.topk_w[s];
  }
  uint64_t srow = 0;
  float wl = 0.0f;
  uint32_t st = 0;
  if (p >= 0) {
    const int r = e / a.L;
    if ((unsigned)r >= (unsigned)a.R) {
      st |= MOE_STATUS_BAD_INDEX;   // pos and topk_idx disagree: weight 0
    } else {
      const int local = p - a.rank_offset[r];
      const int cap = a.recv_cap[r];
      const uint64_t ry = a.expert_y[r];
      if (local >= 0 && local < cap) {
        srow = ry + (uint64_t)local * (uint64_t)rb;
        wl = w;
      } else {
        st |= MOE_STATUS_CAPACITY;
      }
    }
  }
  float acc[S][8];
#pragma unroll
  for (int c = 0; c < S; ++c)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[c][i] = 0.0f;
  // lanes past k hold no slot, so the last group of 8 may be partly empty
  for (int j0 = 0; j0 < k; j0 += KB) {
    u32x4 v[KB][S];
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      const uint64_t base = readlane64(srow, j0 + j);
      const Rsrc rs = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<uint8_t*>(base),
                                                        (short)0, base ? (int)rb : 0, kRsrcWord3);
#pragma unroll
      for (int c = 0; c < S; ++c)
        v[j][c] = __builtin_amdgcn_raw_buffer_load_b128(rs, o0 + c * kWaveBytes, 0,
                                                        kLoadNonTemporal);
    }
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      const float wj = readlane_f32(wl, j0 + j);
#pragma unroll
      for (int c = 0; c < S; ++c) fma8(acc[c], v[j][c], wj);
    }
  }
  uint8_t* dst = reinterpret_cast<uint8_t*>(a.y) + (int64_t)t * rb;
#pragma unroll
  for (int c = 0; c < S; ++c) {
    const uint32_t off = o0 + c * kWaveBytes;
    if (off < rb) st16_stream(dst + off, pack8(acc[c]));
  }
  if (q == 0) {   // one wavefront reports a token
    st = wave_or(st);
    if (st && lane == 0) atomicOr(a.status, st);
  }
}

template <int KB, int S>
hipError_t launch_unit_as(const CombineArgs& a, hipStream_t stream) {
  const int slices = (int)((row_slices(a.row_bytes) + S - 1) / S);
  const int64_t width = a.row_bytes < S * kWaveBytes ? a.row_bytes : S * kWaveBytes;
  const unsigned lds = wave_limit_lds(gather_unit_waves(a.k * width), kWavesPerBlock);
  return launch_token_ranges(a.tokens, slices, [&](int first, int units) {
    // Batches of a few tokens spread every token's slices over the XCDs.
    const int tokens = units / slices, round = kXcds * kXcdGroup;
    const int group = tokens >= 8 * round ? kXcdGroup : 0;
    const int64_t launched = group ? (int64_t)(tokens + round - 1) / round * round * slices : units;
    hipLaunchKernelGGL((combine_unit_kernel<KB, S>),
                       dim3((launched + kWavesPerBlock - 1) / kWavesPerBlock), dim3(kBlock), lds,
                       stream, a, first, slices, units, group);
  });
}

template <int KB>
hipError_t launch_unit(const CombineArgs& a, hipStream_t stream) {
  if (KB == 1 && a.row_bytes > 2 * kWaveBytes)
    return launch_unit_as<KB, KB == 1 ? 4 : 1>(a, stream);
  if (KB <= 2 && a.row_bytes > kWaveBytes) return launch_unit_as<KB, KB <= 2 ? 2 : 1>(a, stream);
  return launch_unit_as<KB, 1>(a, stream);
}

hipError_t launch_units(const CombineArgs& a, hipStream_t stream) {
  switch (a.k) {
    case 1: return launch_unit<1>(a, stream);
    case 2: return launch_unit<2>(a, stream);
    case 3: return launch_unit<3>(a, stream);
    case 4: return launch_unit<4>(a, stream);
    case 5: return launch_unit<5>(a, stream);
    case 6: return launch_unit<6>(a, stream);
    case 7: return launch_unit<7>(a, stream);
    default: return launch_unit<8>(a, stream);
  }
}

// Large batches of few, narrow rows per token: a unit is then a fraction of a
// wavefront's lanes and a chain of three loads, and the launch of one per token
// bounds the batch.  They keep the persistent split, static parts, whose
// wavefronts resolve 64 / k tokens at once.  us, persistent / units at 32768,
// 65536 and 131072 tokens:
//   k = 1, 16 B    11.8 / 11.0  22.6 / 24.5  39.5 / 47.0     512 B  17.3 / 16.9  30.6 / 31.4  55.7 / 60.7
//   k = 2, 128 B   14.6 / 17.5  23.1 / 32.6  45.0 / 62.8    1 KiB   22.4 / 24.2  39.1 / 44.8  73.6 / 87.1
//   k = 3, 512 B   22.9 / 21.9  38.9 / 41.0  69.5 / 79.2    1 KiB   27.5 / 26.5  51.4 / 50.7  -
//   k = 4, 128 B   18.5 / 19.9  31.4 / 36.7  55.1 / 70.5    1 KiB   31.4 / 30.3  60.7 / 56.7  -
//   k = 6, 512 B   44.0 / 24.5  76.6 / 46.0  - (its slots are padded to 8)
bool many_narrow_rows(const CombineArgs& a) {
  if (a.k > 4 || a.row_bytes > (a.k <= 2 ? 1024 : 512)) return false;
  return a.tokens >= (a.k % 2 == 0 ? 32768 : 65536);
}

}  // namespace

hipError_t launch_combine(const CombineArgs& a, int policy, hipStream_t stream) {
  if (policy == MOE_POLICY_BALANCED && a.launch_waves == 0 && !a.trace) {
    if (!many_narrow_rows(a)) return launch_units(a, stream);
    policy = MOE_POLICY_STATIC;
  }
  const bool large = claim_all_parts(a.tokens, a.row_bytes, a.k);
  const bool claim = policy == MOE_POLICY_DYNAMIC || (policy == MOE_POLICY_BALANCED && large);
  // Small parts (decode-sized batches) measured 2% faster for combine, and
  // the dispatch after it too, with twice the gathers in flight; large
  // parts 6% slower.
  const int64_t in_flight = large ? kCombineInFlight : 2 * kCombineInFlight;
  return claim ? launch_dyn<true>(a, in_flight, stream)
               : launch_dyn<false>(a, in_flight, stream);
}

}  // namespace moe
