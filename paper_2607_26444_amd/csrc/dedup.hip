// Per-peer deduplicated dispatch and combine.
//
// The peer windows of Appendix D hold one row per routed (token, expert)
// pair; a token with several experts on one peer then crosses to that peer
// several times.  This path sends it once per peer instead (the traffic per
// peer that Section 6.2 balances shrinks by the duplicates):
//
//   moe_layout_dedup   one row per (token, peer) pair, token order per peer
//                      (the layout kernels over peers: each slot reads as
//                      its peer if it is the token's first slot on it, as
//                      unrouted otherwise);
//   moe_dispatch_dedup the dispatch kernel over the pair rows;
//   moe_expand         on the receiving peer: pair rows -> expert-ordered
//                      rows, the layout a per-slot dispatch would have left;
//   moe_combine_local  on the receiving peer: each pair's weighted sum of its
//                      expert outputs, one bf16 row per pair;
//   moe_combine_dedup  on the source: the combine kernel with unit weights
//                      over the pair rows.
//
// The two receiver-side kernels take one wavefront per (token, slice of its
// row) unit, launched in token order (as dispatch and combine do); each
// resolves the token's k slots one per lane.

#include "dedup.h"

namespace moe {
namespace {

constexpr int kNoKey = 0x7FFFFFFF;   // sort key of an unrouted slot (last)

// The pair row of this lane's slot: the first non-negative tok_pos among the
// token's slots (lanes below k) with the same peer, -1 if none.
__device__ __forceinline__ int run_row(int key, int tok_pos, int k) {
  int row = -1;
  for (int j = 0; j < k; ++j) {
    const int kk = __builtin_amdgcn_readlane(key, j), qq = __builtin_amdgcn_readlane(tok_pos, j);
    if (kk == key && row < 0 && qq >= 0) row = qq;
  }
  return row;
}

// One wavefront per (token, slice of S KiB of its row): the expansion.  Bound by
// HBM (k writes and up to k reads per slice).  Each slot's pair-row slice is
// requested before the first store (KB slots at a time, through buffer
// resources: a slot without a source reads nothing), so a token's k loads
// overlap; slots that share a pair row read it again from the cache, which is
// cheaper than walking the runs of a peer one load after another.  Measured on
// MI355X against persistent wavefronts that did that over whole rows (us
// before -> after, GB/s of algorithmic bytes after):
//   16384 x 14 KiB, k = 8, Zipf 1.2     546 -> 502  (5710)
//   32768 x 8 KiB, k = 8, Zipf 1.5      624 -> 551  (5730)
//   16384 x 10 KiB, k = 6, uniform      401 -> 388
//   16384 x 7 KiB fp8, k = 8, uniform   397 -> 394
//   4096 x 14 KiB, k = 8, uniform       190 -> 185  (4990)
//   8192 x 8 KiB, k = 16, uniform       406 -> 411
//   16384 x 2 KiB, k = 1                16.9 -> 14.1
template <bool SCALES, int KB, int S>
__global__ __launch_bounds__(kBlock) void expand_unit_kernel(ExpandArgs a, int first, int slices,
                                                             int units) {
  const int lane = threadIdx.x & (kWave - 1);
  const int u = uniform(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave);
  if (u >= units) return;
  const int q = u % slices, t = first + u / slices;
  const uint32_t rb = (uint32_t)a.row_bytes;
  const uint32_t sb = (uint32_t)a.scale_row_bytes;
  const uint32_t sp = (uint32_t)a.scale_pitch;
  const int k = a.k;
  const uint32_t o0 = (uint32_t)q * (S * kWaveBytes) + lane * kVecBytes;
  const bool scales_here = SCALES && q == 0;
  int p = -1, e = 0, tp = -1;
  if (lane < k) {
    const int64_t s = (int64_t)t * k + lane;
    p = a.pos[s];
    e = a.topk_idx[s];
    tp = a.tok_pos[s];
  }
  int key = kNoKey;
  uint32_t st = 0;
  uint64_t src = 0, dst = 0, ssrc = 0, sdst = 0;
  if (p >= 0) {
    const int r = e / a.L;
    if ((unsigned)r < (unsigned)a.R) key = r;
    else st |= MOE_STATUS_BAD_INDEX;   // pos and topk_idx disagree: not copied
  }
  const int pair = run_row(key, tp, k);
  if (key != kNoKey) {
    const int r = key;
    const int dl = pair - a.tok_offset[r], ol = p - a.rank_offset[r];
    const int dcap = a.dedup_cap[r], ocap = a.recv_cap[r];
    const uint64_t dx = a.dedup_x[r], rx = a.recv_x[r];
    uint64_t ds = 0, rs = 0;
    if (scales_here) {
      ds = a.dedup_scales[r];
      rs = a.recv_scales[r];
    }
    if (pair >= 0 && dl >= 0 && dl < dcap) {
      src = dx + (uint64_t)dl * rb;
      ssrc = ds + (uint64_t)dl * sp;
    } else {
      st |= MOE_STATUS_CAPACITY;
    }
    if (ol >= 0 && ol < ocap) {
      dst = rx + (uint64_t)ol * rb;
      sdst = rs + (uint64_t)ol * sp;
    } else {
      st |= MOE_STATUS_CAPACITY;
    }
    if (!src || !dst) src = dst = 0;
  }
  // a slice of each destination row is cut at that row's own 128-byte lines:
  // it starts `cut` bytes early, and the last slice ends with the row (16384 x
  // 14 KiB, k = 8, region bases 16 bytes off the line: 752 us for whole rows
  // per wavefront, 804 with uncut slices, 731 now)
  for (int j0 = 0; j0 < k; j0 += KB) {
    u32x4 v[KB][S];
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      const uint64_t base = readlane64(src, j0 + j);
      const uint32_t cut = (uint32_t)readlane64(dst, j0 + j) % kLine;
      const Rsrc rs = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<uint8_t*>(base),
                                                        (short)0, base ? (int)rb : 0, kRsrcWord3);
#pragma unroll
      for (int c = 0; c < S; ++c)
        v[j][c] = __builtin_amdgcn_raw_buffer_load_b128(rs, o0 - cut + c * kWaveBytes, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      uint8_t* d = reinterpret_cast<uint8_t*>(readlane64(dst, j0 + j));
      if (!d) continue;
      const uint32_t cut = (uint32_t)(uintptr_t)d % kLine;
#pragma unroll
      for (int c = 0; c < S; ++c) {
        const uint32_t off = o0 - cut + c * kWaveBytes;   // wraps before the row's start
        if (off < rb) st16_stream(d + off, v[j][c]);
      }
      if (cut && q == slices - 1) {
        const uint32_t off = o0 + (S - 1) * kWaveBytes;
        const uint8_t* from = reinterpret_cast<const uint8_t*>(readlane64(src, j0 + j));
        if (lane * kVecBytes + cut >= kWaveBytes && off < rb)
          st16_stream(d + off, ld16(from + off));
      }
    }
  }
  if (scales_here) {
    if (!src) sdst = 0;
    if (a.scales16) {
      // groups of `pieces` lanes carry one destination's scale row each
      const int pieces = (int)sp / kVecBytes, per = kWave / pieces;
      const int sj = lane / pieces;
      const uint32_t soff = (uint32_t)(lane - sj * pieces) * kVecBytes;
      for (int j0 = 0; j0 < k; j0 += per) {
        const int j = j0 + sj;
        const uint64_t from = __shfl((unsigned long long)ssrc, j & (kWave - 1), kWave);
        const uint64_t to = __shfl((unsigned long long)sdst, j & (kWave - 1), kWave);
        if (sj < per && j < k && to) {
          u32x4 sv = {0u, 0u, 0u, 0u};
          if (soff < sb) sv = ld16(reinterpret_cast<const uint8_t*>(from) + soff);
          st16_stream(reinterpret_cast<uint8_t*>(to) + soff, sv);
        }
      }
    } else {
      // other scale-row sizes: one float32 per lane per pass
      for (int j = 0; j < k; ++j) {
        const uint8_t* from = reinterpret_cast<const uint8_t*>(readlane64(ssrc, j));
        uint8_t* to = reinterpret_cast<uint8_t*>(readlane64(sdst, j));
        if (!to) continue;
        for (uint32_t o = lane * 4; o < sp; o += kWave * 4)
          st4(to + o, o < sb ? ld4(from + o) : 0u);
      }
    }
  }
  if (q == 0) {   // one wavefront reports a token
    st = wave_or(st);
    if (st && lane == 0) atomicOr(a.status, st);
  }
}

// Resident wavefronts per compute unit of the expansion for wave_bytes of
// loads and as many of stores per wavefront.  The range of unmasked batches is
// flat from 12 to 20 wavefronts (16384 x 14 KiB, k = 8, Zipf, us at 32 / 20 /
// 16 / 12 / 8: 517 505 502 499 518; uniform 736 736 736 735 721); batches with
// unused slots, whose wavefronts move little each, want more (32768 x 14 KiB,
// k = 8, half / three quarters / nine tenths unused: 12 wavefronts 770 585 417,
// 16 750 527 347, one persistent wavefront per row 745 384 157).
int expand_unit_waves(int64_t wave_bytes) {
  const int64_t w = 48 * kWaveBytes / wave_bytes + 6;
  return w < 16 ? 16 : w > 32 ? 32 : (int)w;
}

// One wavefront per (token, slice of S KiB of its row): the partial combine.
// Bound by HBM reads (k gathers and one store per run).  The slots are taken
// in (peer, slot) order, KB gathers at a time; a run's sum restarts from +0
// and is stored at the run's last slot (no destination: the pair row is past
// its region, nothing is stored).  A slot without an expert row reads nothing
// and adds +0.  Measured on MI355X against persistent wavefronts over whole
// rows, us of this kernel before -> after:
//   16384 x 14 KiB, k = 8, Zipf 1.2     556 -> 489  (5900 GB/s)
//   4096 x 14 KiB, k = 8, uniform       196 -> 187
template <int KB, int S>
__global__ __launch_bounds__(kBlock) void combine_local_unit_kernel(LocalArgs a, int first,
                                                                    int slices, int units) {
  const int lane = threadIdx.x & (kWave - 1);
  const int u = uniform(blockIdx.x * kWavesPerBlock + threadIdx.x / kWave);
  if (u >= units) return;
  const int q = u % slices, t = first + u / slices;
  const uint32_t rb = (uint32_t)a.row_bytes;
  const int k = a.k;
  const uint32_t o0 = (uint32_t)q * (S * kWaveBytes) + lane * kVecBytes;
  int p = -1, e = 0, tp = -1;
  float w = 0.0f;
  if (lane < k) {
    const int64_t s = (int64_t)t * k + lane;
    p = a.pos[s];
    e = a.topk_idx[s];
    tp = a.tok_pos[s];
    w = a.topk_w[s];
  }
  int key = kNoKey;
  uint32_t st = 0;
  if (p >= 0) {
    const int r = e / a.L;
    if ((unsigned)r < (unsigned)a.R) key = r;
    else st |= MOE_STATUS_BAD_INDEX;   // pos and topk_idx disagree: not combined
  }
  const int pair = run_row(key, tp, k);
  // position of this lane's slot after ordering the slots by (peer, slot),
  // and whether it closes its run; lanes past k keep their place
  int spos = lane < k ? 0 : lane;
  bool last = key != kNoKey;
  for (int j = 0; j < k; ++j) {
    const int kk = __builtin_amdgcn_readlane(key, j);
    if (lane < k) {
      spos += (kk < key || (kk == key && j < lane)) ? 1 : 0;
      last = last && !(kk == key && j > lane);
    }
  }
  uint64_t src = 0, dst = 0;
  float wl = 0.0f;
  if (key != kNoKey) {
    const int r = key;
    const int il = p - a.rank_offset[r], pl = pair - a.tok_offset[r];
    const int icap = a.recv_cap[r], pcap = a.part_cap[r];
    const uint64_t ey = a.expert_y[r], pt = a.partial[r];
    if (il >= 0 && il < icap) {
      src = ey + (uint64_t)il * rb;
      wl = w;
    } else {
      st |= MOE_STATUS_CAPACITY;
    }
    if (last) {
      if (pair >= 0 && pl >= 0 && pl < pcap) dst = pt + (uint64_t)pl * rb;
      else st |= MOE_STATUS_CAPACITY;
    }
  }
  const uint64_t closes = __ballot(last);
  float acc[S][8];
#pragma unroll
  for (int c = 0; c < S; ++c)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[c][i] = 0.0f;
  for (int j0 = 0; j0 < k; j0 += KB) {
    u32x4 v[KB][S];
    int at[KB];   // lane of the slot at place j0 + j
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      at[j] = __builtin_ctzll(__ballot(spos == j0 + j));
      const uint64_t base = readlane64(src, at[j]);
      const Rsrc rs = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<uint8_t*>(base),
                                                        (short)0, base ? (int)rb : 0, kRsrcWord3);
#pragma unroll
      for (int c = 0; c < S; ++c)
        v[j][c] = __builtin_amdgcn_raw_buffer_load_b128(rs, o0 + c * kWaveBytes, 0,
                                                        kLoadNonTemporal);
    }
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      const float wj = readlane_f32(wl, at[j]);
#pragma unroll
      for (int c = 0; c < S; ++c) fma8(acc[c], v[j][c], wj);
      if (closes >> at[j] & 1) {
        uint8_t* d = reinterpret_cast<uint8_t*>(readlane64(dst, at[j]));
#pragma unroll
        for (int c = 0; c < S; ++c) {
          const uint32_t off = o0 + c * kWaveBytes;
          if (d && off < rb) st16_stream(d + off, pack8(acc[c]));
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[c][i] = 0.0f;
        }
      }
    }
  }
  if (q == 0) {   // one wavefront reports a token
    st = wave_or(st);
    if (st && lane == 0) atomicOr(a.status, st);
  }
}

// Workgroups of one wavefront, which frees its slot as soon as it is done, of
// two with scale rows (16384 x 14 KiB, k = 8, Zipf, us by one / two / four:
// 502 504 507; 16384 x 8 KiB 412 416 420; fp8 16384 x 7 KiB 396 394 397).
template <bool SCALES, int KB, int S>
hipError_t launch_expand_as(const ExpandArgs& a, hipStream_t stream) {
  const int slices = (int)((row_slices(a.row_bytes) + S - 1) / S);
  const int64_t width = a.row_bytes < S * kWaveBytes ? a.row_bytes : S * kWaveBytes;
  const int wpb = SCALES ? 2 : 1;
  const unsigned lds = wave_limit_lds(expand_unit_waves(a.k * width), wpb);
  return launch_token_ranges(a.tokens, slices, [&](int first, int units) {
    hipLaunchKernelGGL((expand_unit_kernel<SCALES, KB, S>), dim3((units + wpb - 1) / wpb),
                       dim3(wpb * kWave), lds, stream, a, first, slices, units);
  });
}

// Slices of 1 KiB from k = 3; 2 KiB for k = 2 and 4 KiB for k = 1 unless the
// row is no wider than half of that.
template <bool SCALES>
hipError_t launch_expand_units(const ExpandArgs& a, hipStream_t stream) {
  const bool wide = a.row_bytes > kWaveBytes;
  if (a.k == 1) {
    if (a.row_bytes > 2 * kWaveBytes) return launch_expand_as<SCALES, 1, 4>(a, stream);
    return wide ? launch_expand_as<SCALES, 1, 2>(a, stream)
                : launch_expand_as<SCALES, 1, 1>(a, stream);
  }
  if (a.k == 2)
    return wide ? launch_expand_as<SCALES, 2, 2>(a, stream)
                : launch_expand_as<SCALES, 2, 1>(a, stream);
  if (a.k <= 4) return launch_expand_as<SCALES, 4, 1>(a, stream);
  if (a.k <= 6) return launch_expand_as<SCALES, 6, 1>(a, stream);
  if (a.k <= 8) return launch_expand_as<SCALES, 8, 1>(a, stream);
  return launch_expand_as<SCALES, 16, 1>(a, stream);
}

template <int KB, int S>
hipError_t launch_local_as(const LocalArgs& a, hipStream_t stream) {
  const int slices = (int)((row_slices(a.row_bytes) + S - 1) / S);
  const int64_t width = a.row_bytes < S * kWaveBytes ? a.row_bytes : S * kWaveBytes;
  const unsigned lds = wave_limit_lds(gather_unit_waves(a.k * width), kWavesPerBlock);
  return launch_token_ranges(a.tokens, slices, [&](int first, int units) {
    hipLaunchKernelGGL((combine_local_unit_kernel<KB, S>),
                       dim3((units + kWavesPerBlock - 1) / kWavesPerBlock), dim3(kBlock), lds,
                       stream, a, first, slices, units);
  });
}

}  // namespace

DedupGeom dedup_geom(int64_t T, int k, int R) {
  DedupGeom d;
  d.g = layout_geom(T, R);
  d.spare_offset = (d.g.total + 255) / 256 * 256;
  d.total = d.spare_offset + ((size_t)(2 * R + 1) * 4 + 255) / 256 * 256;
  return d;
}

hipError_t launch_expand(const ExpandArgs& a, hipStream_t stream) {
  return a.dedup_scales ? launch_expand_units<true>(a, stream)
                        : launch_expand_units<false>(a, stream);
}

// Slices as in combine: 2 KiB for k <= 2 unless the row is no wider.
hipError_t launch_combine_local(const LocalArgs& a, hipStream_t stream) {
  const bool wide = a.row_bytes > kWaveBytes;
  switch (a.k) {
    case 1: return wide ? launch_local_as<1, 2>(a, stream) : launch_local_as<1, 1>(a, stream);
    case 2: return wide ? launch_local_as<2, 2>(a, stream) : launch_local_as<2, 1>(a, stream);
    case 3:
    case 4: return launch_local_as<4, 1>(a, stream);
    case 5:
    case 6: return launch_local_as<6, 1>(a, stream);
    default: return launch_local_as<8, 1>(a, stream);
  }
}

}  // namespace moe
