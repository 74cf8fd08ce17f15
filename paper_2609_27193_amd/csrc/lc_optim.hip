// HIP kernels of the optimizer steps that yield the drift statistic (Section
// 3.4: the drift is taken from the optimizer's own update): AdamW, as the
// paper trains, and plain SGD, which Section 4.7 notes the method carries
// over to.  One pass over the optimizer state per step; per chunk of the
// score layout the kernel updates the parameters and writes the Eq. 1
// partial sums of |p_new - p| and |p|, which the finalize kernel turns into
// u and Delta.  Streaming rules as in lc_kernels.hip (full chunks through
// buffer resources, ragged ones through global pointers).
#include "lc_device.h"

namespace lc {
namespace {

constexpr int kAdamW = 0;
constexpr int kSGD = 1;

// Threads per block: a block takes its whole tile in one burst of loads, so
// 512 threads of two groups for the 4096 elements of a bf16 chunk (256 threads
// of four: AdamW 1663 us, 512: 1529, one block per CU, 336 M parameters).  An
// fp32 chunk has 2048 elements: 256 threads of two groups (AdamW 1465 us, 512
// threads of one: 1475), with a master 512 (1822; 256: 1840).
template <int WDT, bool MASTER>
constexpr uint32_t kOptThreads = WDT == 1 || MASTER ? 512 : 256;

__device__ __forceinline__ uint16_t bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7FC0u;  // NaN stays a quiet NaN
  u += 0x7FFFu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

// One AdamW element update in fp32, one rounding per operation, fixed order.
// The library is built with -ffp-contract=off (no fused multiply-adds), and
// fp32 division and sqrtf compile to their correctly rounded sequences
// (div_scale/div_fmas/div_fixup; v_sqrt with neighbour correction), so every
// operation below is the IEEE round-to-nearest-even result.
__device__ __forceinline__ float adamw_elem(float p, float& m, float& v, float g, const AdamScalars& sc,
                                            bool decay) {
  m = sc.b1 * m + sc.omb1 * g;
  v = sc.b2 * v + sc.omb2 * (g * g);
  const float mh = m * sc.c1;
  const float vh = v * sc.c2;
  const float den = sqrtf(vh) + sc.eps;
  const float upd = mh / den;
  const float p1 = decay ? p * sc.decay : p;
  return p1 - sc.lr * upd;
}

template <int WDT>
__device__ __forceinline__ float w_load(const uint8_t* w, uint64_t i) {
  if constexpr (WDT == 1) return __uint_as_float(static_cast<uint32_t>(((const g_u16*)w)[i]) << 16);
  else return ((const g_f32*)w)[i];
}
template <int WDT>
__device__ __forceinline__ void w_store(uint8_t* w, uint64_t i, float x) {
  if constexpr (WDT == 1) ((g_u16*)w)[i] = bf16_rne(x);
  else ((g_f32*)w)[i] = x;
}
template <int GDT>
__device__ __forceinline__ float g_load(const uint8_t* g, uint64_t i) {
  if constexpr (GDT == 1) return __uint_as_float(static_cast<uint32_t>(((const g_u16*)g)[i]) << 16);
  else return ((const g_f32*)g)[i];
}

// One SGD element update in fp32 with decoupled weight decay, one rounding
// per operation: p_new = p * (1 - lr wd) - lr g (the decay only for decayed
// segments).
__device__ __forceinline__ float sgd_elem(float p, float g, const SgdScalars& sc, bool decay) {
  const float p1 = decay ? p * sc.decay : p;
  return p1 - sc.lr * g;
}

// The arrays of one chunk from the first element of its tile on: the
// parameters (the fp32 master, else the weights), the weights, the gradient
// and, for AdamW, the moments.
struct ChunkPtrs {
  uint8_t *p, *w, *m, *v;
  const uint8_t* g;
};
struct ChunkTiles {
  tile_t p, w, g, m, v;
};

__device__ __forceinline__ u32x4 widen_bf16x4(u32x2 x) {
  return u32x4{x[0] << 16, x[0] & 0xffff0000u, x[1] << 16, x[1] & 0xffff0000u};
}
__device__ __forceinline__ u32x2 narrow_bf16x4(u32x4 p) {
  return u32x2{bf16_rne(__uint_as_float(p[0])) | (static_cast<uint32_t>(bf16_rne(__uint_as_float(p[1]))) << 16),
               bf16_rne(__uint_as_float(p[2])) | (static_cast<uint32_t>(bf16_rne(__uint_as_float(p[3]))) << 16)};
}

// Four consecutive elements (group j of the tile), updated in place: of a
// full tile whose arrays are aligned to groups through buffer resources,
// else through global pointers at the arrays' own alignment.  AdamW also
// streams m and v; SGD touches only the parameters.
template <int OPT, int WDT, int GDT, bool MASTER>
struct Group4 {
  u32x4 p, m, v;  // parameters as fp32 bits, moments
  float g[4];

  __device__ __forceinline__ void set_grad(u32x2 x) {
    g[0] = __uint_as_float(x[0] << 16); g[1] = __uint_as_float(x[0] & 0xffff0000u);
    g[2] = __uint_as_float(x[1] << 16); g[3] = __uint_as_float(x[1] & 0xffff0000u);
  }
  __device__ __forceinline__ void set_grad(u32x4 x) {
    for (int k = 0; k < 4; ++k) g[k] = __uint_as_float(x[k]);
  }
  __device__ __forceinline__ void load_p(const ChunkPtrs& c, uint32_t j) {
    if constexpr (!MASTER && WDT == 1) p = widen_bf16x4(ld_any2(c.p + j * 8u));
    else p = ld_any<4>(c.p + j * 16u);
  }
  __device__ __forceinline__ void load_m(const ChunkPtrs& c, uint32_t j) { m = ld_any<4>(c.m + j * 16u); }
  __device__ __forceinline__ void load_v(const ChunkPtrs& c, uint32_t j) { v = ld_any<4>(c.v + j * 16u); }
  __device__ __forceinline__ void load_g(const ChunkPtrs& c, uint32_t j) {
    if constexpr (GDT == 1) set_grad(ld_any2(c.g + j * 8u));
    else set_grad(ld_any<4>(c.g + j * 16u));
  }
  __device__ __forceinline__ void load_p(const ChunkTiles& t, uint32_t j) {
    if constexpr (!MASTER && WDT == 1) p = widen_bf16x4(ld_tile2(t.p, j * 8u));
    else p = ld_tile(t.p, j * 16u);
  }
  __device__ __forceinline__ void load_m(const ChunkTiles& t, uint32_t j) { m = ld_tile(t.m, j * 16u); }
  __device__ __forceinline__ void load_v(const ChunkTiles& t, uint32_t j) { v = ld_tile(t.v, j * 16u); }
  __device__ __forceinline__ void load_g(const ChunkTiles& t, uint32_t j) {
    if constexpr (GDT == 1) set_grad(ld_tile2(t.g, j * 8u));
    else set_grad(ld_tile(t.g, j * 16u));
  }
  // One optimizer step of the four elements in place; adds the drift terms
  // (|p_new - p|, |p|) to (a, b): pairwise in fp32 first, or each term by
  // itself in fp64 (WIDE).
  template <bool WIDE, typename SC>
  __device__ __forceinline__ void update(const SC& sc, bool decay, double& a, double& b) {
    float d[4], q[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float po = __uint_as_float(p[k]);
      float x;
      if constexpr (OPT == kAdamW) {
        float mm = __uint_as_float(m[k]), vv = __uint_as_float(v[k]);
        x = adamw_elem(po, mm, vv, g[k], sc, decay);
        m[k] = __float_as_uint(mm);
        v[k] = __float_as_uint(vv);
      } else {
        x = sgd_elem(po, g[k], sc, decay);
      }
      p[k] = __float_as_uint(x);
      d[k] = fabsf(x - po);
      q[k] = fabsf(po);
    }
    if constexpr (WIDE) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        a += static_cast<double>(d[k]);
        b += static_cast<double>(q[k]);
      }
    } else {
      a += static_cast<double>((d[0] + d[1]) + (d[2] + d[3]));
      b += static_cast<double>((q[0] + q[1]) + (q[2] + q[3]));
    }
  }
  __device__ __forceinline__ void store_m(const ChunkPtrs& c, uint32_t j) const { st_any4(c.m + j * 16u, m); }
  __device__ __forceinline__ void store_v(const ChunkPtrs& c, uint32_t j) const { st_any4(c.v + j * 16u, v); }
  __device__ __forceinline__ void store_p(const ChunkPtrs& c, uint32_t j) const { st_any4(c.p + j * 16u, p); }
  __device__ __forceinline__ void store_w(const ChunkPtrs& c, uint32_t j) const {
    if constexpr (WDT == 1) st_any2(c.w + j * 8u, narrow_bf16x4(p));
    else st_any4(c.w + j * 16u, p);
  }
  __device__ __forceinline__ void store_m(const ChunkTiles& t, uint32_t j) const { st_tile(t.m, j * 16u, m); }
  __device__ __forceinline__ void store_v(const ChunkTiles& t, uint32_t j) const { st_tile(t.v, j * 16u, v); }
  __device__ __forceinline__ void store_p(const ChunkTiles& t, uint32_t j) const { st_tile(t.p, j * 16u, p); }
  __device__ __forceinline__ void store_w(const ChunkTiles& t, uint32_t j) const {
    if constexpr (WDT == 1) st_tile2(t.w, j * 8u, narrow_bf16x4(p));
    else st_tile(t.w, j * 16u, p);
  }
};

// N groups of a thread, loaded, updated and stored one array after the other:
// each array's part of the tile is one run of HBM accesses (336 M parameters,
// one block per CU: AdamW 1529 us, group after group 1542).
template <int OPT, int WDT, int GDT, bool MASTER, bool WIDE, uint32_t N, typename SRC, typename GSRC, typename SC>
__device__ __forceinline__ void optim_groups(const SRC& t, const GSRC& tg, uint32_t j, const SC& sc, bool decay,
                                             double& a, double& b) {
  Group4<OPT, WDT, GDT, MASTER> grp[N];
#define LC_EACH_GROUP(stmt)           \
  _Pragma("unroll") for (uint32_t k = 0; k < N; ++k) stmt
  LC_EACH_GROUP(grp[k].load_p(t, j + k * kOptThreads<WDT, MASTER>);)
  if constexpr (OPT == kAdamW) {
    LC_EACH_GROUP(grp[k].load_m(t, j + k * kOptThreads<WDT, MASTER>);)
    LC_EACH_GROUP(grp[k].load_v(t, j + k * kOptThreads<WDT, MASTER>);)
  }
  LC_EACH_GROUP(grp[k].load_g(tg, j + k * kOptThreads<WDT, MASTER>);)
  LC_EACH_GROUP(grp[k].template update<WIDE>(sc, decay, a, b);)
  if constexpr (OPT == kAdamW) {
    LC_EACH_GROUP(grp[k].store_m(t, j + k * kOptThreads<WDT, MASTER>);)
    LC_EACH_GROUP(grp[k].store_v(t, j + k * kOptThreads<WDT, MASTER>);)
  }
  if constexpr (MASTER) LC_EACH_GROUP(grp[k].store_p(t, j + k * kOptThreads<WDT, MASTER>);)
  LC_EACH_GROUP(grp[k].store_w(t, j + k * kOptThreads<WDT, MASTER>);)
#undef LC_EACH_GROUP
}

// A full tile: every load in flight before the first update.  ANYG: the
// gradient at any alignment; ANY: every array.  On a 160 M element segment
// with bf16 weights, master and bf16 gradients (AdamW / SGD): aligned arrays
// 806 / 355 us, arrays alike at an odd element 819 / 363 us (element by
// element 1282 / 440), only the gradient apart 820 / 365 us (1277 / 405),
// weights and gradient apart from the fp32 arrays 865 / 390 us (1288 / 415).
template <int OPT, int WDT, int GDT, bool MASTER, bool WIDE, bool ANYG, bool ANY, typename SC>
__device__ __forceinline__ void optim_tile(const ChunkPtrs& c, const SC& sc, bool decay, double& a, double& b) {
  constexpr uint32_t WSZ = WDT == 1 ? 2 : 4, GSZ = GDT == 1 ? 2 : 4;
  constexpr uint32_t CE = kChunkBytes / WSZ;      // elements per chunk (the score chunks)
  constexpr uint32_t GPT = CE / 4 / kOptThreads<WDT, MASTER>;  // 4-element groups per thread in a full chunk
  static_assert(GPT >= 1 && CE % (4 * kOptThreads<WDT, MASTER>) == 0, "tiling");
  if constexpr (ANY) {
    optim_groups<OPT, WDT, GDT, MASTER, WIDE, GPT>(c, c, threadIdx.x, sc, decay, a, b);
  } else {
    ChunkTiles t;
    t.w = make_tile(c.w, CE * WSZ);
    t.p = MASTER ? make_tile(c.p, CE * 4) : t.w;
    t.g = make_tile(c.g, CE * GSZ);
    t.m = t.v = t.p;
    if constexpr (OPT == kAdamW) {
      t.m = make_tile(c.m, CE * 4);
      t.v = make_tile(c.v, CE * 4);
    }
    if constexpr (ANYG) optim_groups<OPT, WDT, GDT, MASTER, WIDE, GPT>(t, c, threadIdx.x, sc, decay, a, b);
    else optim_groups<OPT, WDT, GDT, MASTER, WIDE, GPT>(t, t, threadIdx.x, sc, decay, a, b);
  }
}

// Whether a gradient apart from state arrays that are aligned at element 0
// leaves these their tiles (ANYG).  160 M elements, gradient at an odd element,
// every array through unaligned accesses / only the gradient, AdamW and SGD
// (us): bf16 with master, bf16 gradients 793 / 724 and 308 / 305, fp32 gradients
// 802 / 768 and 358 / 349; bf16 alone 561 / 551 and 153 / 153; fp32 with bf16
// gradients 698 / 683 and 252 / 252, with fp32 gradients 734 / 737 and 312 / 319.
template <int WDT, int GDT, bool MASTER>
constexpr bool kGradApart = MASTER || WDT == 1 || GDT == 1;

// Element e of a segment.
template <int OPT, int WDT, int GDT, bool MASTER, typename SC>
__device__ __forceinline__ void optim_elem(const OptSeg& sg, const GradSeg& gs, const SC& sc, uint64_t e, double& a,
                                           double& b) {
  const float po = MASTER ? ((const g_f32*)sg.master)[e]
                          : w_load<WDT>(reinterpret_cast<const uint8_t*>(sg.w), e);
  const float gv = g_load<GDT>(reinterpret_cast<const uint8_t*>(gs.grad), e);
  const bool decay = gs.decay != 0;
  float x;
  if constexpr (OPT == kAdamW) {
    g_f32* mp = (g_f32*)sg.m + e;
    g_f32* vp = (g_f32*)sg.v + e;
    float mm = *mp, vv = *vp;
    x = adamw_elem(po, mm, vv, gv, sc, decay);
    *mp = mm;
    *vp = vv;
  } else {
    x = sgd_elem(po, gv, sc, decay);
  }
  if constexpr (MASTER) ((g_f32*)sg.master)[e] = x;
  w_store<WDT>(reinterpret_cast<uint8_t*>(sg.w), e, x);
  a += static_cast<double>(fabsf(x - po));
  b += static_cast<double>(fabsf(po));
}

typedef __attribute__((address_space(4))) GradSeg c_GradSeg;

struct OptTables {
  const uint32_t* chunk_seg;
  const OptSeg* opt_segs;
  const GradSeg* grad_segs;
  double2* partials;
};

template <int OPT, int WDT, int GDT, bool MASTER, typename SC>
__device__ __forceinline__ void optim_chunk(const OptTables& t, const InlineGrads& ig, const SC& sc, uint32_t c) {
  constexpr uint32_t WSZ = WDT == 1 ? 2 : 4, GSZ = GDT == 1 ? 2 : 4;
  constexpr uint32_t CE = kChunkBytes / WSZ;  // elements per chunk (the score chunks)
  const uint32_t tid = threadIdx.x;
  const uint32_t si = t.chunk_seg[c];
  const OptSeg sg = t.opt_segs[si];
  // a constant either way, so that the lookup stays a scalar load
  const c_GradSeg* gt = (const c_GradSeg*)(t.grad_segs ? t.grad_segs : ig.g);
  const GradSeg gs{gt[si].grad, gt[si].decay, gt[si].vec_ok};
  const uint32_t k = c - sg.chunk_begin;
  const uint64_t e0 = static_cast<uint64_t>(k) * CE + sg.head;  // the chunk's tile
  const uint64_t rem = sg.numel > e0 ? sg.numel - e0 : 0;
  const uint32_t n = rem < CE ? static_cast<uint32_t>(rem) : CE;
  const bool decay = gs.decay != 0;
  const bool pairs = sg.form == kOptPairs && gs.vec_ok;
  ChunkPtrs cp;
  cp.w = reinterpret_cast<uint8_t*>(sg.w) + e0 * WSZ;
  cp.p = MASTER ? reinterpret_cast<uint8_t*>(sg.master) + e0 * 4 : cp.w;
  cp.m = reinterpret_cast<uint8_t*>(sg.m) + e0 * 4;
  cp.v = reinterpret_cast<uint8_t*>(sg.v) + e0 * 4;
  cp.g = reinterpret_cast<const uint8_t*>(gs.grad) + e0 * GSZ;
  double a = 0.0, b = 0.0;
  if (n == CE && pairs) {
    optim_tile<OPT, WDT, GDT, MASTER, false, false, false>(cp, sc, decay, a, b);
  } else if (n == CE && (sg.form == kOptWide || (kGradApart<WDT, GDT, MASTER> && sg.form == kOptPairs))) {
    optim_tile<OPT, WDT, GDT, MASTER, true, true, false>(cp, sc, decay, a, b);
  } else if (n == CE) {
    optim_tile<OPT, WDT, GDT, MASTER, true, true, true>(cp, sc, decay, a, b);
  } else {
    const uint32_t ng = n / 4;
    for (uint32_t i = tid; i < ng; i += kOptThreads<WDT, MASTER>) {
      if (pairs) optim_groups<OPT, WDT, GDT, MASTER, false, 1>(cp, cp, i, sc, decay, a, b);
      else optim_groups<OPT, WDT, GDT, MASTER, true, 1>(cp, cp, i, sc, decay, a, b);
    }
    for (uint32_t i = ng * 4 + tid; i < n; i += kOptThreads<WDT, MASTER>)
      optim_elem<OPT, WDT, GDT, MASTER>(sg, gs, sc, e0 + i, a, b);
  }
  // the elements before the first tile
  if (k == 0 && tid < sg.head && tid < sg.numel) optim_elem<OPT, WDT, GDT, MASTER>(sg, gs, sc, tid, a, b);
  block_sum2<kOptThreads<WDT, MASTER>>(a, b);
  if (tid == kOptThreads<WDT, MASTER> - 1) t.partials[c] = make_double2(a, b);
}

template <int OPT, int WDT, int GDT, bool MASTER, bool LOOP, typename SC>
__global__ __launch_bounds__((kOptThreads<WDT, MASTER>)) void optim_kernel(
    const uint32_t* chunk_seg, const OptSeg* opt_segs, const GradSeg* grad_segs, double2* partials, uint32_t n_chunks,
    uint32_t blocks, const SC sc, const InlineGrads ig) {
  const OptTables t{chunk_seg, opt_segs, grad_segs, partials};
  if constexpr (!LOOP) {
    optim_chunk<OPT, WDT, GDT, MASTER>(t, ig, sc, remap_xcd_runs<LC_RW_XCD_RUN>(blockIdx.x, blocks));
  } else {
    for (uint64_t base = 0; base < n_chunks; base += blocks) {
      const uint64_t left = n_chunks - base;
      const uint32_t span = left < blocks ? static_cast<uint32_t>(left) : blocks;
      if (blockIdx.x >= span) return;
      optim_chunk<OPT, WDT, GDT, MASTER>(t, ig, sc, static_cast<uint32_t>(base + remap_xcd(blockIdx.x, span)));
      __syncthreads();
    }
  }
}

// Blocks per CU of an optimizer step, by the bytes that one block loads and
// stores.  HBM moves most with about 100 KB of them open per CU, in tiles as
// large as fit: on 336 M parameters (us at 1 / 2 / 3 / 4 / 5 blocks per CU)
//   AdamW, master, bf16 / fp32 gradients (112 / 120 KB): 1546 / 1656 / 1722,
//     1682 / 1804 / 1852;
//   AdamW, bf16 weights alone (88 / 96 KB): 1280 / 1230 / 1306, 1369 / 1363 /
//     1434: a lone block leaves gaps that its tile does not make up for;
//   AdamW, fp32 weights (52-64 KB): 1675 / 1478 / 1531;
//   SGD, master (48 / 56 KB): 753 / 648 / 677 / 689, 839 / 773 / 813;
//   SGD, bf16 weights alone, bf16 / fp32 gradients (24 / 32 KB): 646 / 437 /
//     335 / 320 / 320, 667 / 475 / 426 / 440;
//   SGD, fp32 weights, bf16 gradients (20 KB): 1358 / 817 / 619 / 540 / 532.
// Chunks that are in the mean less than 7/8 full, of many small segments, wait for
// their tables and the reduction instead, and nothing holds them back (AdamW, bf16
// with master, capped / not: 12000 segments of 40 elements 242 / 182, of 3300 366 /
// 335, of 13000 937 / 918; 90% full: 6000 of 26000 776 / 846).
constexpr uint32_t kOptBytesPerCU = 100 * 1024;

template <int OPT, int WDT, int GDT, bool MASTER, typename SC>
void launch_optim_t(const DeviceTables& t, const InlineGrads& ig, const SC& sc, hipStream_t st) {
  const uint32_t g = grid_for(t.n_chunks, kOptThreads<WDT, MASTER>);
  constexpr uint32_t CE = kChunkBytes / (WDT == 1 ? 2 : 4);
  constexpr uint32_t wsz = WDT == 1 ? 2 : 4;
  constexpr uint32_t tile = CE * ((MASTER ? 8 + wsz : 2 * wsz) + (OPT == kAdamW ? 16 : 0) + (GDT == 1 ? 2 : 4));
  constexpr uint32_t fit = (kOptBytesPerCU + tile / 2) / tile;
  constexpr uint32_t blocks = LC_OPT_BLOCKS_PER_CU ? LC_OPT_BLOCKS_PER_CU
                              : tile >= kOptBytesPerCU ? 1 : fit < 2 ? 2 : fit;
  const bool full = t.total_numel * 8 >= static_cast<uint64_t>(t.n_chunks) * CE * 7;
  const uint32_t lds = full ? occupancy_lds(blocks) : 0;
  if (g == t.n_chunks)
    hipLaunchKernelGGL((optim_kernel<OPT, WDT, GDT, MASTER, false, SC>), dim3(g), dim3(kOptThreads<WDT, MASTER>), lds,
                       st, t.chunk_seg, t.opt_segs, t.grad_segs, t.partials, t.n_chunks, g, sc, ig);
  else
    hipLaunchKernelGGL((optim_kernel<OPT, WDT, GDT, MASTER, true, SC>), dim3(g), dim3(kOptThreads<WDT, MASTER>), lds,
                       st, t.chunk_seg, t.opt_segs, t.grad_segs, t.partials, t.n_chunks, g, sc, ig);
}

template <int OPT, typename SC>
void launch_optim(const DeviceTables& t, const InlineGrads& ig, int grad_dtype, int has_master, const SC& sc,
                  hipStream_t st) {
  const bool gb = grad_dtype == 1;
  if (t.dtype == 1) {
    if (has_master) { if (gb) launch_optim_t<OPT, 1, 1, true>(t, ig, sc, st); else launch_optim_t<OPT, 1, 2, true>(t, ig, sc, st); }
    else { if (gb) launch_optim_t<OPT, 1, 1, false>(t, ig, sc, st); else launch_optim_t<OPT, 1, 2, false>(t, ig, sc, st); }
  } else {
    if (has_master) { if (gb) launch_optim_t<OPT, 2, 1, true>(t, ig, sc, st); else launch_optim_t<OPT, 2, 2, true>(t, ig, sc, st); }
    else { if (gb) launch_optim_t<OPT, 2, 1, false>(t, ig, sc, st); else launch_optim_t<OPT, 2, 2, false>(t, ig, sc, st); }
  }
}

}  // namespace

hipError_t launch_adamw(const DeviceTables& t, const InlineGrads& grads, int grad_dtype, int has_master,
                        const AdamScalars& sc, hipStream_t st) {
  launch_optim<kAdamW>(t, grads, grad_dtype, has_master, sc, st);
  return hipGetLastError();
}

hipError_t launch_sgd(const DeviceTables& t, const InlineGrads& grads, int grad_dtype, int has_master,
                      const SgdScalars& sc, hipStream_t st) {
  launch_optim<kSGD>(t, grads, grad_dtype, has_master, sc, st);
  return hipGetLastError();
}

}  // namespace lc
