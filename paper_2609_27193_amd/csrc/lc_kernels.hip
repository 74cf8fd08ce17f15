// HIP kernels of the LayerCheck decision step for gfx950 (MI355X, CDNA4).
//
// Every kernel here is HBM-bound streaming work or a tiny O(N) step; nothing
// is a dense contraction, so there is no MFMA.  Design rules:
//  * 16-byte (dwordx4) coalesced loads/stores, several in flight per lane;
//    non-temporal, device-scope cache policy because every byte is touched
//    once per step and the per-step stream (tens of GB) dwarfs the 256 MB
//    Infinity Cache; full chunks and pieces go through buffer resources;
//  * reductions use no floating-point atomics: one fp64 pair per chunk, then a
//    fixed-order per-layer sum, so scores are bitwise reproducible;
//  * wave64 reductions (DPP moves or cross-row shuffles), LDS for the
//    cross-wave combine;
//  * kernels take the few tables that they read as arguments of their own, not
//    the struct of all of them: the loads of the arguments stand together and
//    wait once.  On 3.7 M parameters, where trips to memory bound every kernel,
//    the decision step takes 28.8 us, with the struct 30.0.
#include "lc_device.h"

#include <algorithm>
#include <atomic>
#include <type_traits>

namespace lc {
namespace {

// |W - S| and |S| of one 16-byte vector, summed pairwise in fp32.
template <int DT>
__device__ __forceinline__ void vec_terms(const u32x4 w, const u32x4 s, float& da, float& sb) {
  if constexpr (DT == 1) {
    float d[8], b[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float w0 = bf_lo(w[k]), w1 = bf_hi(w[k]);
      const float s0 = bf_lo(s[k]), s1 = bf_hi(s[k]);
      d[2 * k] = fabsf(w0 - s0);
      d[2 * k + 1] = fabsf(w1 - s1);
      b[2 * k] = fabsf(s0);
      b[2 * k + 1] = fabsf(s1);
    }
    da = ((d[0] + d[1]) + (d[2] + d[3])) + ((d[4] + d[5]) + (d[6] + d[7]));
    sb = ((b[0] + b[1]) + (b[2] + b[3])) + ((b[4] + b[5]) + (b[6] + b[7]));
  } else {
    float d[4], b[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float wf = __uint_as_float(w[k]), sf = __uint_as_float(s[k]);
      d[k] = fabsf(wf - sf);
      b[k] = fabsf(sf);
    }
    da = (d[0] + d[1]) + (d[2] + d[3]);
    sb = (b[0] + b[1]) + (b[2] + b[3]);
  }
}

template <int DT>
__device__ __forceinline__ float elem_value(const uint8_t* base, uint64_t i) {
  if constexpr (DT == 1) {
    return __uint_as_float(static_cast<uint32_t>(((const g_u16*)base)[i]) << 16);
  } else {
    return ((const g_f32*)base)[i];
  }
}

template <int DT>
__device__ __forceinline__ void elem_copy(const uint8_t* src, uint8_t* dst, uint64_t i) {
  if constexpr (DT == 1) {
    ((g_u16*)dst)[i] = ((const g_u16*)src)[i];
  } else {
    ((g_f32*)dst)[i] = ((const g_f32*)src)[i];
  }
}


// Adds the |W - S| and |S| of one 16-byte vector to (a, b): pairwise in fp32
// first, or each term by itself in fp64 (WIDE).
template <int DT, bool WIDE>
__device__ __forceinline__ void add_terms(const u32x4 w, const u32x4 s, double& a, double& b) {
  if constexpr (!WIDE) {
    float da, db;
    vec_terms<DT>(w, s, da, db);
    a += static_cast<double>(da);
    b += static_cast<double>(db);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if constexpr (DT == 1) {
        const float s0 = bf_lo(s[k]), s1 = bf_hi(s[k]);
        a += static_cast<double>(fabsf(bf_lo(w[k]) - s0));
        b += static_cast<double>(fabsf(s0));
        a += static_cast<double>(fabsf(bf_hi(w[k]) - s1));
        b += static_cast<double>(fabsf(s1));
      } else {
        const float sf = __uint_as_float(s[k]);
        a += static_cast<double>(fabsf(__uint_as_float(w[k]) - sf));
        b += static_cast<double>(fabsf(sf));
      }
    }
  }
}

// ---- score: one chunk per block and iteration ---------------------------------
// The tile of one chunk: n elements from wb and sb on, sb on a 128-byte line
// (wb too, or 16-byte aligned, unless ANYW).  A full tile goes through buffer
// resources with every load of a round in flight before the first sum.  HBM
// bounds all three forms: on a 160 M element bf16 segment (ACCUM / SNAPSHOT)
// aligned arrays take 160 / 101 us, arrays alike at an odd element 159 / 101
// us (element by element they took 433 / 309) and weights at an odd element
// against the shadow 166 / 117 us (430 / 312): the loads that straddle lines.
template <int DT, bool ACCUM, bool WIDE, bool ANYW>
__device__ __forceinline__ void score_tile(const uint8_t* wb, uint8_t* sb, uint32_t n, double& a, double& b) {
  constexpr uint32_t ESZ = DT == 1 ? 2 : 4;
  constexpr uint32_t CE = kChunkBytes / ESZ;  // elements per chunk
  constexpr uint32_t EPV = 16 / ESZ;          // elements per 16-B vector
  constexpr uint32_t NV = CE / EPV;           // vectors per full chunk
  constexpr uint32_t VPT = NV / kScoreThreads;
  constexpr uint32_t U = VPT < 4 ? VPT : 4;   // vectors per thread per round
  static_assert(VPT % U == 0, "tiling");
  const uint32_t tid = threadIdx.x;
  if (n == CE) {
    const tile_t tw = make_tile(wb, kChunkBytes), ts = make_tile(sb, kChunkBytes);
#pragma unroll
    for (uint32_t r = 0; r < VPT / U; ++r) {
      u32x4 w[U], s[U];
#pragma unroll
      for (uint32_t k = 0; k < U; ++k) {
        const uint32_t off = (tid + (r * U + k) * kScoreThreads) * 16u;
        if constexpr (ANYW) w[k] = ld_any<ESZ>(wb + off);
        else w[k] = ld_tile(tw, off);
        s[k] = ld_tile(ts, off);
      }
#pragma unroll
      for (uint32_t k = 0; k < U; ++k) {
        add_terms<DT, WIDE>(w[k], s[k], a, b);
        if constexpr (ACCUM) st_tile(ts, (tid + (r * U + k) * kScoreThreads) * 16u, w[k]);
      }
    }
    return;
  }
  u32x4* sv = reinterpret_cast<u32x4*>(sb);
  const uint32_t nv = n / EPV;
  for (uint32_t i = tid; i < nv; i += kScoreThreads) {
    const u32x4 w = ANYW ? ld_any<ESZ>(wb + i * 16u) : ld_nt(reinterpret_cast<const u32x4*>(wb) + i);
    const u32x4 s = ld_nt(sv + i);
    add_terms<DT, WIDE>(w, s, a, b);
    if constexpr (ACCUM) st_nt(sv + i, w);
  }
  for (uint32_t i = nv * EPV + tid; i < n; i += kScoreThreads) {
    const float wf = elem_value<DT>(wb, i), sf = elem_value<DT>(sb, i);
    a += static_cast<double>(fabsf(wf - sf));
    b += static_cast<double>(fabsf(sf));
    if constexpr (ACCUM) elem_copy<DT>(wb, sb, i);
  }
}

// Streams W and S of one chunk once; writes (sum|W-S|, sum|S|) in fp64.  In
// ACCUM mode the same pass stores W into S (the next step's W(t-1)).
template <int DT, bool ACCUM>
__device__ __forceinline__ void score_chunk(const ScoreSeg* segs, const uint32_t* chunk_seg, double2* partials,
                                            uint32_t c) {
  constexpr uint32_t ESZ = DT == 1 ? 2 : 4;
  constexpr uint32_t CE = kChunkBytes / ESZ;  // elements per chunk
  const ScoreSeg sg = segs[chunk_seg[c]];
  const uint32_t k = c - sg.chunk_begin;
  const uint64_t e0 = static_cast<uint64_t>(k) * CE + sg.head;  // the chunk's tile
  const uint64_t rem = sg.numel > e0 ? sg.numel - e0 : 0;
  const uint32_t n = rem < CE ? static_cast<uint32_t>(rem) : CE;
  const uint8_t* w = reinterpret_cast<const uint8_t*>(sg.w);
  uint8_t* s = reinterpret_cast<uint8_t*>(sg.s);

  double a = 0.0, b = 0.0;
  if (sg.form == kScorePairs) score_tile<DT, ACCUM, false, false>(w + e0 * ESZ, s + e0 * ESZ, n, a, b);
  else if (sg.form == kScoreWide) score_tile<DT, ACCUM, true, false>(w + e0 * ESZ, s + e0 * ESZ, n, a, b);
  else score_tile<DT, ACCUM, true, true>(w + e0 * ESZ, s + e0 * ESZ, n, a, b);
  if (k == 0 && threadIdx.x < sg.head && threadIdx.x < sg.numel) {  // the elements before the first tile
    const float wf = elem_value<DT>(w, threadIdx.x), sf = elem_value<DT>(s, threadIdx.x);
    a += static_cast<double>(fabsf(wf - sf));
    b += static_cast<double>(fabsf(sf));
    if constexpr (ACCUM) elem_copy<DT>(w, s, threadIdx.x);
  }
  block_sum2<kScoreThreads, ACCUM>(a, b);
  if (threadIdx.x == kScoreThreads - 1) partials[c] = make_double2(a, b);
}

// One chunk per block: the chunk's tables are read before any store, so they
// stay on the scalar path.  A layout with more chunks than one dispatch takes
// (2^32 work-items) is scored by consecutive launches, each over the next
// range of chunks starting at chunk_base.
template <int DT, bool ACCUM>
__global__ __launch_bounds__(kScoreThreads) void score_kernel(const ScoreSeg* segs, const uint32_t* chunk_seg,
                                                              double2* partials, uint32_t chunk_base,
                                                              uint32_t blocks) {
  const uint32_t x = ACCUM ? remap_xcd_runs<LC_RW_XCD_RUN>(blockIdx.x, blocks) : remap_xcd(blockIdx.x, blocks);
  score_chunk<DT, ACCUM>(segs, chunk_seg, partials, chunk_base + x);
}

// ---- finalize: Eq. 1 and Eq. 2 per layer, one block per layer -----------------
// Thread j sums partials j, j + NT, j + 2 NT, ... of its layer into four
// interleaved accumulators (independent loads in flight), combined in a fixed
// order, then a fixed-order block reduction: deterministic for a given layout.
// Behind a small score the launch and the trips to memory bound it, so what
// does not depend on the partials is loaded first (3.7 M parameters: decision
// step 29.7 -> 28.9 us); of a large layer, the load rate of its one CU does
// (64 K partials 12 us).
__global__ __launch_bounds__(kFinalizeThreads) void finalize_kernel(const uint32_t* layer_chunk_begin,
                                                                    const double2* partials, const uint64_t* numel_of,
                                                                    double* delta_of, double* u_of, double eps_w,
                                                                    int mode) {
  const uint32_t l = blockIdx.x;
  const uint32_t c0 = layer_chunk_begin[l], c1 = layer_chunk_begin[l + 1];
  const uint64_t numel = numel_of[l];
  const double delta = delta_of[l];
  double a[4] = {0.0, 0.0, 0.0, 0.0}, b[4] = {0.0, 0.0, 0.0, 0.0};
  uint32_t c = c0 + threadIdx.x;
  for (; c + 3 * kFinalizeThreads < c1; c += 4 * kFinalizeThreads) {
    double2 p[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) p[k] = partials[c + k * kFinalizeThreads];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      a[k] += p[k].x;
      b[k] += p[k].y;
    }
  }
  // at most three partials remain for this thread
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (c < c1) {
      const double2 p = partials[c];
      a[k] += p.x;
      b[k] += p.y;
      c += kFinalizeThreads;
    }
  }
  double x = (a[0] + a[1]) + (a[2] + a[3]);
  double y = (b[0] + b[1]) + (b[2] + b[3]);
  block_sum2<kFinalizeThreads>(x, y);
  if (threadIdx.x == kFinalizeThreads - 1) {
    const double n = static_cast<double>(numel);
    const double u = (x / n) / (y / n + eps_w);
    u_of[l] = u;
    delta_of[l] = (mode == 0) ? delta + u : u;
  }
}

// ---- select: Eq. 3-5, reset, staleness stats, pack plan ------------------------
// What one layer adds to the plan and the stats (integers: any order of the
// sums gives the same), and its inclusive scan over the lanes of a wave.
struct SelectSums {
  uint64_t pay, pieces, num, den;
  int64_t max_age;
  uint32_t ns, nf;

  __device__ __forceinline__ void add(const SelectSums& o) {
    pay += o.pay;
    pieces += o.pieces;
    num += o.num;
    den += o.den;
    max_age = o.max_age > max_age ? o.max_age : max_age;
    ns += o.ns;
    nf += o.nf;
  }
  __device__ __forceinline__ SelectSums up(int d) const {
    SelectSums o;
    o.pay = __shfl_up(pay, d, 64);
    o.pieces = __shfl_up(pieces, d, 64);
    o.num = __shfl_up(num, d, 64);
    o.den = __shfl_up(den, d, 64);
    o.max_age = __shfl_up(max_age, d, 64);
    o.ns = __shfl_up(ns, d, 64);
    o.nf = __shfl_up(nf, d, 64);
    return o;
  }
};

// One block of one wave (a layout of up to 64 layers) or four, a layer a
// lane and round: the loads of a round are independent, so a round costs one
// trip to memory, and the plan's prefixes are a scan.  The chain of loads
// bounds it.  On 18-35 layers behind a score that has swept the caches it
// takes 5 us, where one lane that walked the layers took 8-11.
template <uint32_t NT>
__global__ __launch_bounds__(NT) void select_kernel(const uint64_t* numel, const uint64_t* rec_bytes,
                                                    const uint64_t* layer_pieces, int64_t* t_last, const double* k0,
                                                    double* delta, uint32_t n_layers, int base_mode, DeviceTables t,
                                                    int64_t step, double lr_scale, uint64_t seq) {
  constexpr uint32_t NW = NT / 64;
  __shared__ SelectSums wave_total[NW];
  const uint32_t N = n_layers, lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  SelectHeader* hr = t.host_result;
  uint8_t* mask = reinterpret_cast<uint8_t*>(hr + 1);
  SelectSums before{};  // of the rounds before this one
  for (uint32_t l0 = 0; l0 < N; l0 += NT) {
    const uint32_t l = l0 + threadIdx.x;
    SelectSums s{};
    if (l < N) {
      uint32_t code = 1;  // bit0 selected, bit1 selected by the staleness guard alone
      const uint64_t n = numel[l], rec = rec_bytes[l], pieces = layer_pieces[l];
      int64_t age = step - t_last[l];
      if (!base_mode) {
        const double K = k0[l] * lr_scale;
        const bool by_drift = delta[l] >= K;
        const bool by_age = age >= t.s_max;
        code = ((by_drift || by_age) ? 1u : 0u) | ((!by_drift && by_age) ? 2u : 0u);
        if (code & 1u) {
          delta[l] = 0.0;
          t_last[l] = step;
          age = 0;
        }
      }
      s.ns = code & 1u;
      s.nf = code >> 1;
      s.pay = s.ns ? rec : 0;
      s.pieces = s.ns ? pieces : 0;
      s.num = n * static_cast<uint64_t>(age);
      s.den = n;
      s.max_age = age > 0 ? age : 0;
      mask[l] = static_cast<uint8_t>(code & 1u);
    }
    const uint32_t selected = s.ns;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const SelectSums o = s.up(d);
      if (lane >= static_cast<uint32_t>(d)) s.add(o);
    }
    if constexpr (NW > 1) {
      __syncthreads();  // the round before has read the totals
      if (lane == 63u) wave_total[wave] = s;
      __syncthreads();
      for (uint32_t w = 0; w < wave; ++w) s.add(wave_total[w]);
    }
    s.add(before);
    if (selected) {  // s counts this layer: it is the rank before the next prefix
      t.sel_layer[s.ns - 1] = l;
      t.sel_rec_prefix[s.ns] = s.pay;
      t.sel_piece_prefix[s.ns] = s.pieces;
    }
    if constexpr (NW > 1) {
      for (uint32_t w = 0; w < NW; ++w) before.add(wave_total[w]);
    } else {
      before = s;  // one round: lane 63 has the totals
    }
  }
  // The host's copy, read with no device-to-host copy and no stream
  // synchronisation: the mask and the header, then -- once system-scope
  // fences have made those visible -- the number the host waits for.
  if (threadIdx.x == NT - 1) {  // has the totals in either form
    t.sel_rec_prefix[0] = 0;
    t.sel_piece_prefix[0] = 0;
    SelectHeader h;
    h.n_selected = before.ns;
    h.n_forced = before.nf;
    h.payload_bytes = before.pay;
    h.max_age = before.max_age;
    h.weighted_age = static_cast<double>(before.num) / static_cast<double>(before.den);
    h.total_pieces = before.pieces;
    h.age_numerator = before.num;
    h.seq = 0;
    h.reserved = 0;
    *hr = h;
  }
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == NT - 1) hr->seq = seq;
}

// ---- small tables between pinned host memory and the device ---------------------
// Beside the streaming kernels in the same stream: a copy command of the
// runtime waits for its own engine or kernel and leaves gaps of 6-20 us around
// it, and a copy back to the host a round trip each.

// n 16-byte entries from pinned host memory; the flag, which needs a launch of
// one block, tells the host that the source may be written again.
__global__ __launch_bounds__(kTableThreads) void fetch_kernel(const u32x4* src, u32x4* dst, uint32_t n, uint64_t* flag,
                                                              uint64_t seq) {
  constexpr uint32_t U = 4;  // loads in flight: one trip over the link for up to 1024 entries a block
  const uint32_t stride = gridDim.x * kTableThreads;
  for (uint32_t i = blockIdx.x * kTableThreads + threadIdx.x; i < n; i += U * stride) {
    u32x4 x[U];
#pragma unroll
    for (uint32_t k = 0; k < U; ++k)
      if (i + k * stride < n) x[k] = src[i + k * stride];
#pragma unroll
    for (uint32_t k = 0; k < U; ++k)
      if (i + k * stride < n) dst[i + k * stride] = x[k];
  }
  __syncthreads();  // every load has returned: its value was stored
  if (threadIdx.x == 0 && flag) *reinterpret_cast<volatile uint64_t*>(flag) = seq;
}

// u, Delta and t_l of every layer to pinned host memory, an entry of each a
// thread up to kTableBlocks blocks: trips over the host link bound it (whole
// call, us, one block / 32 / 128: 1024 layers 18.1 / 17.4 / 17.4, 8192 34.0 /
// 25.5 / 25.6, 20000 59.0 / 38.6 / 38.6, 100000 265 / 145 / 145; three copies of
// the runtime 49.8, 37.8, 62.8, 156).
__global__ __launch_bounds__(kTableThreads) void push_state_kernel(const DeviceTables t, HostState* h) {
  const uint32_t N = t.n_layers;
  double* u = reinterpret_cast<double*>(h + 1);
  for (uint32_t l = blockIdx.x * kTableThreads + threadIdx.x; l < N; l += gridDim.x * kTableThreads) {
    u[l] = t.u[l];
    u[N + l] = t.delta[l];
    reinterpret_cast<int64_t*>(u)[2 * N + l] = t.t_last[l];
  }
}

// Delta = 0 and t_l = steps[l] (or one step for all) of every layer.
__global__ __launch_bounds__(kTableThreads) void reset_state_kernel(const DeviceTables t, const int64_t* steps,
                                                                    int64_t step) {
  for (uint32_t l = blockIdx.x * kTableThreads + threadIdx.x; l < t.n_layers; l += gridDim.x * kTableThreads) {
    t.delta[l] = 0.0;
    t.t_last[l] = steps ? steps[l] : step;
  }
}

// ---- byte movement of one piece ----------------------------------------------
// len bytes, a multiple of 2, from src to dst and, if given, to dst2, all at
// least 2-byte aligned.  Full pieces go through buffer resources, the tails
// and whatever is not 16-byte aligned through global pointers.  The callers
// cut the pieces so that dst starts on a line (see below); src and dst2 may
// start anywhere: on a 160 M element layer with every array at an odd element
// the pack takes 689 us (aligned 679; two bytes a lane took 891), with the
// shadow refreshed 763 (726; 1415) and the restore 767 (767; 1454).
// The restore reads a source that does not start on a line as one that starts
// anywhere: a line that two waves share then comes once over the host link, while
// the tiles' device scope fetches it twice.  Records in page-locked memory, arrays
// 16 bytes off a line, W, m and v of 80 MB: 50.7 -> 56.9 GB/s (through copies 56.3;
// arrays on a line 55.5); in device memory either way takes as long.
template <bool ANYS, bool ANYD>
__device__ __forceinline__ void copy_full_piece(const uint8_t* __restrict__ src, uint8_t* __restrict__ dst,
                                                uint8_t* __restrict__ dst2) {
  constexpr uint32_t V = kPieceBytes / 16 / kCopyThreads;
  const uint32_t tid = threadIdx.x;
  const tile_t td = make_tile(dst, kPieceBytes);
  u32x4 v[V];
  if constexpr (ANYS) {
#pragma unroll
    for (uint32_t k = 0; k < V; ++k) v[k] = ld_any<2>(src + (tid + k * kCopyThreads) * 16u);
  } else {
    const tile_t ts = make_tile(src, kPieceBytes);
#pragma unroll
    for (uint32_t k = 0; k < V; ++k) v[k] = ld_tile(ts, (tid + k * kCopyThreads) * 16u);
  }
#pragma unroll
  for (uint32_t k = 0; k < V; ++k) st_tile(td, (tid + k * kCopyThreads) * 16u, v[k]);
  if (dst2) {
    const tile_t te = make_tile(dst2, kPieceBytes);
#pragma unroll
    for (uint32_t k = 0; k < V; ++k) {
      const uint32_t off = (tid + k * kCopyThreads) * 16u;
      if constexpr (ANYD) st_any(dst2 + off, v[k]);
      else st_tile(te, off, v[k]);
    }
  }
}

template <uint32_t SRC_ALIGN>
__device__ __forceinline__ void copy_piece(const uint8_t* __restrict__ src, uint8_t* __restrict__ dst,
                                           uint8_t* __restrict__ dst2, uint32_t len) {
  const uint32_t tid = threadIdx.x;
  const bool any_s = reinterpret_cast<uint64_t>(src) % SRC_ALIGN != 0, any_d = reinterpret_cast<uint64_t>(dst2) % 16 != 0;
  uint32_t done = 0;
  if (reinterpret_cast<uint64_t>(dst) % 16 == 0) {
    if (len == kPieceBytes) {
      if (!any_s && !any_d) copy_full_piece<false, false>(src, dst, dst2);
      else if (!any_d) copy_full_piece<true, false>(src, dst, dst2);
      else copy_full_piece<true, true>(src, dst, dst2);
      return;
    }
    const uint32_t nv = len / 16;
    for (uint32_t i = tid; i < nv; i += kCopyThreads) {
      const u32x4 x = ld_any<2>(src + i * 16u);
      st_nt(reinterpret_cast<u32x4*>(dst) + i, x);
      if (dst2) st_any(dst2 + i * 16u, x);
    }
    done = nv * 16;
  }
  const g_u16* s2 = (const g_u16*)src;
  g_u16* d2 = (g_u16*)dst;
  g_u16* f2 = (g_u16*)dst2;
  for (uint32_t i = done / 2 + tid; i < len / 2; i += kCopyThreads) {
    const uint16_t x = s2[i];
    d2[i] = x;
    if (dst2) f2[i] = x;
  }
}

// ---- pack: selected records into the staging buffer ---------------------------
// Work item q is piece q (relative to piece_base) of the selected records of
// ranks [first, last); records are written from staging offset
// sel_rec_prefix[first] - rec_base.
struct PackTables {
  const uint64_t* sel_piece_prefix;
  const uint32_t* sel_layer;
  const uint64_t* layer_piece_begin;
  const uint32_t* piece_unit;
  const CopyUnit* units;
  const uint64_t* sel_rec_prefix;
};

template <bool REFRESH>
__device__ __forceinline__ void pack_piece(const PackTables& t, uint32_t first, uint32_t last, uint64_t q,
                                           uint64_t rec_base, uint8_t* staging) {
  uint32_t lo = first, hi = last;  // sel_piece_prefix[lo] <= q < sel_piece_prefix[hi]
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (t.sel_piece_prefix[mid] <= q) lo = mid; else hi = mid;
  }
  const uint32_t l = t.sel_layer[lo];
  const uint64_t lp = q - t.sel_piece_prefix[lo];
  const CopyUnit u = t.units[t.piece_unit[t.layer_piece_begin[l] + lp]];
  const uint64_t off = (lp - u.piece0) * kPieceBytes;
  const uint64_t rem = u.bytes - off;
  const uint32_t len = rem < kPieceBytes ? static_cast<uint32_t>(rem) : kPieceBytes;
  uint8_t* dst = staging + (t.sel_rec_prefix[lo] - rec_base) + u.rec_off + off;
  const uint8_t* src = reinterpret_cast<const uint8_t*>(u.arr) + off;
  uint8_t* dst2 = (REFRESH && u.shadow) ? reinterpret_cast<uint8_t*>(u.shadow) + off : nullptr;
  copy_piece<16>(src, dst, dst2, len);
  if (off + len == u.bytes) {  // zero the block's padding
    const uint32_t pad = static_cast<uint32_t>(round_up(u.bytes, kRecordAlign) - u.bytes);
    g_u16* z = (g_u16*)(dst + len);
    for (uint32_t i = threadIdx.x; i < pad / 2; i += kCopyThreads) z[i] = 0;
  }
}

// One piece per block; piece_base is the first piece of this launch (a pack
// with more pieces than one dispatch takes is split into consecutive launches).
template <bool REFRESH>
__global__ __launch_bounds__(kCopyThreads) void pack_kernel(const uint64_t* sel_piece_prefix,
                                                            const uint32_t* sel_layer,
                                                            const uint64_t* layer_piece_begin,
                                                            const uint32_t* piece_unit, const CopyUnit* units,
                                                            uint64_t piece_base, uint32_t first, uint32_t last,
                                                            uint32_t blocks,
                                                            const uint64_t* sel_rec_prefix, uint64_t rec_base,
                                                            uint8_t* staging) {
  const PackTables t{sel_piece_prefix, sel_layer, layer_piece_begin, piece_unit, units, sel_rec_prefix};
  pack_piece<REFRESH>(t, first, last, piece_base + remap_xcd_runs<LC_COPY_XCD_RUN>(blockIdx.x, blocks), rec_base, staging);
}

// ---- unpack: composite restore from records in device or pinned host memory ----
// rank r restores its layer from the record at address ranks[r].src; every W
// block also refreshes the shadow.  An array's pieces start behind its head,
// on a line of the array, so that the stores do not split lines; the array's
// first piece takes the head with it, and the last may be empty.
typedef __attribute__((address_space(4))) RankEntry c_RankEntry;

__device__ __forceinline__ void unpack_piece(const UnpackArgs& t, const c_RankEntry* ranks, uint64_t q) {
  uint32_t lo = 0, hi = t.n_ranks;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (ranks[mid].piece_prefix <= q) lo = mid; else hi = mid;
  }
  const uint64_t lp = q - ranks[lo].piece_prefix;
  const CopyUnit u = t.units[t.piece_unit[ranks[lo].piece_begin + lp]];
  const uint8_t* src = reinterpret_cast<const uint8_t*>(ranks[lo].src) + u.rec_off;
  uint8_t* dst = reinterpret_cast<uint8_t*>(u.arr);
  uint8_t* dst2 = u.shadow ? reinterpret_cast<uint8_t*>(u.shadow) : nullptr;
  const uint32_t p = static_cast<uint32_t>(lp) - u.piece0;
  if (p == 0 && u.head) copy_piece<kLineBytes>(src, dst, dst2, u.head);
  const uint64_t off = static_cast<uint64_t>(p) * kPieceBytes + u.head;
  const uint64_t rem = u.bytes > off ? u.bytes - off : 0;
  const uint32_t len = rem < kPieceBytes ? static_cast<uint32_t>(rem) : kPieceBytes;
  if (len) copy_piece<kLineBytes>(src + off, dst + off, dst2 ? dst2 + off : nullptr, len);
}

// One piece per block, from piece_base on (split like the pack).  Ranks in the
// arguments are read as the constants that the others are, too, and nothing is
// stored before the tables are read: scalar loads (a store before them makes
// the unit's lookup a vector load and costs 1.2% on 1.2 B parameters).
__global__ __launch_bounds__(kCopyThreads) void unpack_kernel(const UnpackArgs t) {
  const c_RankEntry* ranks = (const c_RankEntry*)(t.ranks ? t.ranks : t.inline_ranks);
  unpack_piece(t, ranks, t.piece_base + remap_xcd_runs<LC_COPY_XCD_RUN>(blockIdx.x, gridDim.x));
  if (!t.ranks && blockIdx.x == 0 && t.piece_base == 0) {
    for (uint32_t l = threadIdx.x; l < t.n_ranks; l += kCopyThreads) {
      t.delta[l] = 0.0;
      t.t_last[l] = ranks[l].step;
    }
  }
}

// Each launch takes the largest grid one dispatch allows (grid_for) and the
// next range of work items; every block does exactly one item.
template <int DT, bool ACCUM>
void launch_score_t(const DeviceTables& t, hipStream_t st) {
  // A state whose blocks all fit on the chip at once (8 per CU) fits the
  // caches, too: HBM is not what bounds it, so nothing holds blocks back (3.7 M
  // fp32 weights, ACCUM: 12.9 us with the finalize kernel, 13.7 at 3 per CU).
  constexpr uint32_t kResidentBlocks = 256 * 2048 / kScoreThreads;
  const uint32_t lds = t.n_chunks <= kResidentBlocks ? 0
                       : occupancy_lds(ACCUM ? LC_SCORE_ACCUM_BLOCKS_PER_CU : LC_SCORE_SNAPSHOT_BLOCKS_PER_CU);
  for (uint64_t done = 0; done < t.n_chunks;) {
    const uint32_t g = grid_for(t.n_chunks - done, kScoreThreads);
    hipLaunchKernelGGL((score_kernel<DT, ACCUM>), dim3(g), dim3(kScoreThreads), lds, st, t.segs,
                       t.chunk_seg, t.partials, static_cast<uint32_t>(done), g);
    done += g;
  }
}

// A copy of many ranks waits for its search over them, a chain of loads that
// more blocks hide better than the cap on them serves HBM: beyond kSearchRanks
// none is held back (us, capped / not: pack of 240 ranks, 32 M elements 147.0 /
// 140.7, 8 M 45.0 / 41.0, of 2400 179.6 / 154.5; restore of 300 layers, 40 M elements
// 232.8 / 207.0; packs of up to 60 ranks gain 3% by the cap on large states).
constexpr uint32_t kSearchRanks = 128;

uint32_t copy_lds(uint32_t ranks) { return ranks > kSearchRanks ? 0 : occupancy_lds(LC_COPY_BLOCKS_PER_CU); }

template <bool REFRESH>
void launch_pack_t(const DeviceTables& t, uint32_t first, uint32_t last, uint64_t piece_base, uint64_t n_pieces,
                   uint64_t rec_base, uint8_t* stg, hipStream_t st) {
  const uint32_t lds = copy_lds(last - first);
  for (uint64_t done = 0; done < n_pieces;) {
    const uint32_t g = grid_for(n_pieces - done, kCopyThreads);
    hipLaunchKernelGGL((pack_kernel<REFRESH>), dim3(g), dim3(kCopyThreads), lds, st, t.sel_piece_prefix, t.sel_layer,
                       t.layer_piece_begin, t.piece_unit, t.units, piece_base + done, first, last, g,
                       t.sel_rec_prefix, rec_base, stg);
    done += g;
  }
}

}  // namespace

// A CU holds L bytes of LDS; a block that asks for more than L / (k + 1)
// leaves room for at most k blocks.  The reservation asks for 2 KiB more than
// that (rounded to 512 B) so the kernel's own few bytes of static LDS cannot
// push it past L / k.  Queried once per device.
uint32_t occupancy_lds(uint32_t blocks_per_cu) {
  if (blocks_per_cu == 0) return 0;
  constexpr int kMaxDevices = 64;
  static std::atomic<int64_t> lds_cu[kMaxDevices], lds_block[kMaxDevices];  // 0: not queried yet
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
  if (lds_cu[dev].load(std::memory_order_relaxed) == 0) {
    int cu = 0, blk = 0;
    if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess ||
        hipDeviceGetAttribute(&blk, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) {
      (void)hipGetLastError();
      return 0;
    }
    lds_block[dev].store(blk, std::memory_order_relaxed);
    lds_cu[dev].store(cu > 0 ? cu : -1, std::memory_order_relaxed);
  }
  const int64_t cu = lds_cu[dev].load(std::memory_order_relaxed);
  const int64_t blk = lds_block[dev].load(std::memory_order_relaxed);
  if (cu <= 0) return 0;
  const int64_t k = blocks_per_cu;
  const int64_t want = (cu / (k + 1) + 2048 + 511) / 512 * 512;
  if (want > cu / k - 1024 || want > blk) return 0;
  return static_cast<uint32_t>(want);
}

hipError_t launch_score(const DeviceTables& t, hipStream_t st) {
  if (t.dtype == 1) {
    if (t.mode == 0) launch_score_t<1, true>(t, st);
    else launch_score_t<1, false>(t, st);
  } else {
    if (t.mode == 0) launch_score_t<2, true>(t, st);
    else launch_score_t<2, false>(t, st);
  }
  return launch_finalize(t, st);
}

hipError_t launch_finalize(const DeviceTables& t, hipStream_t st) {
  hipLaunchKernelGGL(finalize_kernel, dim3(t.n_layers), dim3(kFinalizeThreads), 0, st, t.layer_chunk_begin, t.partials,
                     t.numel, t.delta, t.u, t.eps_w, t.mode);
  return hipGetLastError();
}

hipError_t launch_select(const DeviceTables& t, int64_t step, double lr_scale, int base_mode, uint64_t seq,
                         hipStream_t st) {
  if (t.n_layers <= 64)
    hipLaunchKernelGGL(select_kernel<64>, dim3(1), dim3(64), 0, st, t.numel, t.rec_bytes, t.layer_pieces, t.t_last,
                       t.k0, t.delta, t.n_layers, base_mode, t, step, lr_scale, seq);
  else
    hipLaunchKernelGGL(select_kernel<kSelectThreads>, dim3(1), dim3(kSelectThreads), 0, st, t.numel, t.rec_bytes,
                       t.layer_pieces, t.t_last, t.k0, t.delta, t.n_layers, base_mode, t, step, lr_scale, seq);
  return hipGetLastError();
}

// A launch that reports its own error and leaves the caller's alone: for the
// kernels that stand in a copy's place, in calls that a stale error of the
// program has never failed.
template <typename... P>
static hipError_t launch_own(void (*kernel)(P...), uint32_t grid, uint32_t threads, uint32_t lds, hipStream_t st,
                             std::common_type_t<P>... args) {
  void* at[] = {&args...};
  const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kernel), dim3(grid), dim3(threads), at, lds, st);
  if (e != hipSuccess) (void)hipGetLastError();  // reported here
  return e;
}

static uint32_t table_blocks(uint32_t n) { return std::min(kTableBlocks, (n + kTableThreads - 1) / kTableThreads); }

// Beyond kOneBlockEntries the entries are shared out to several blocks and the
// flag is set by a launch behind them, which costs 2 us and more (AdamW steps of
// n segments of 40 fp32 elements, us, one step / four in a row, one block; several
// blocks; a copy command of the runtime): 1300: 39.2 / 115; 40.6 / 123; 47.1 / 134;
// 2000: 48.0 / 144; 49.7 / 155; 56.2 / 153; 3500: 71.9 / 210; 71.7 / 222; 78.8 / 218.
// An SGD step as a C call, several blocks; copy: 5000: 34.8; 49; 20000: 103; 127;
// 100000: 524; 571.
constexpr uint32_t kOneBlockEntries = 4096;

hipError_t launch_fetch(const void* host_src, void* dst, uint32_t n16, uint64_t* flag, uint64_t seq, hipStream_t st) {
  const bool one = flag && n16 <= kOneBlockEntries;
  const hipError_t e = launch_own(fetch_kernel, one ? 1 : table_blocks(n16), kTableThreads, 0, st,
                                  static_cast<const u32x4*>(host_src), static_cast<u32x4*>(dst), n16,
                                  one ? flag : nullptr, seq);
  if (e != hipSuccess || !flag || one) return e;
  return launch_own(fetch_kernel, 1, kTableThreads, 0, st, nullptr, nullptr, 0, flag, seq);
}

hipError_t launch_push_state(const DeviceTables& t, HostState* host, hipStream_t st) {
  return launch_own(push_state_kernel, table_blocks(t.n_layers), kTableThreads, 0, st, t, host);
}

hipError_t launch_reset_state(const DeviceTables& t, const int64_t* host_steps, int64_t step, hipStream_t st) {
  return launch_own(reset_state_kernel, table_blocks(t.n_layers), kTableThreads, 0, st, t, host_steps, step);
}

hipError_t launch_pack(const DeviceTables& t, uint32_t first_rank, uint32_t last_rank,
                       uint64_t piece_base, uint64_t n_pieces, uint64_t rec_base, void* staging,
                       int refresh_shadow, hipStream_t st) {
  uint8_t* stg = static_cast<uint8_t*>(staging);
  if (refresh_shadow) launch_pack_t<true>(t, first_rank, last_rank, piece_base, n_pieces, rec_base, stg, st);
  else launch_pack_t<false>(t, first_rank, last_rank, piece_base, n_pieces, rec_base, stg, st);
  return hipGetLastError();
}

hipError_t launch_unpack(const DeviceTables& t, const RankEntry* ranks, uint32_t n_ranks, uint64_t n_pieces,
                         hipStream_t st) {
  UnpackArgs a;
  a.piece_unit = t.piece_unit;
  a.units = t.units;
  a.ranks = ranks ? nullptr : t.ranks;
  a.delta = t.delta;
  a.t_last = t.t_last;
  a.n_ranks = n_ranks;
  a.pad = 0;
  if (ranks) std::copy(ranks, ranks + n_ranks + 1, a.inline_ranks);
  const uint32_t lds = copy_lds(n_ranks);
  for (uint64_t done = 0; done < n_pieces;) {
    const uint32_t g = grid_for(n_pieces - done, kCopyThreads);
    a.piece_base = done;
    const hipError_t e = launch_own(unpack_kernel, g, kCopyThreads, lds, st, a);
    if (e != hipSuccess) return e;
    done += g;
  }
  return hipSuccess;
}

}  // namespace lc
