// Internal tables and kernel launchers of the LayerCheck HIP library.
// Shared by the host runtime (lc_runtime.cpp) and the kernels (lc_kernels.hip,
// lc_optim.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lc {

// ---- tiling ------------------------------------------------------------------
// Score: a chunk is a run of consecutive elements of one segment holding
// kChunkBytes of weights (and the same of shadow).  Chunks never cross a
// segment, so every layer owns a contiguous range of chunks and one fp64
// (sum|W-S|, sum|S|) pair per chunk is reduced in a fixed order per layer.
#ifndef LC_CHUNK_BYTES
#define LC_CHUNK_BYTES (8u * 1024u)
#endif
#ifndef LC_XCD_REMAP
#define LC_XCD_REMAP 1  // 0: blocks take their items as they are dispatched (tuning builds)
#endif
#ifndef LC_RW_XCD_RUN
#define LC_RW_XCD_RUN 32  // consecutive chunks per XCD in the ACCUM score and the optimizer kernels
#endif
#ifndef LC_COPY_XCD_RUN
#define LC_COPY_XCD_RUN 64  // consecutive pieces per XCD in the pack and unpack kernels
#endif
#ifndef LC_MAX_GRID_BLOCKS
#define LC_MAX_GRID_BLOCKS 0  // 0: only the dispatch limit caps a grid (testing builds set it low)
#endif
#ifndef LC_PIECE_BYTES
#define LC_PIECE_BYTES (8u * 1024u)
#endif
constexpr uint32_t kScoreThreads = 256;
constexpr uint32_t kChunkBytes = LC_CHUNK_BYTES;
// Pack/restore: a piece is kPieceBytes of one copy unit (one array of one
// segment); records are laid out so that every unit starts 256-B aligned.
constexpr uint32_t kCopyThreads = 256;
constexpr uint32_t kPieceBytes = LC_PIECE_BYTES;
static_assert(kChunkBytes % (16u * kScoreThreads) == 0, "score tiling: whole vectors per thread");
static_assert(kPieceBytes % (16u * kCopyThreads) == 0, "pack tiling");
constexpr uint32_t kRecordAlign = 256u;
constexpr uint32_t kFinalizeThreads = 1024;
constexpr uint32_t kSelectThreads = 256;  // beyond 64 layers
constexpr uint32_t kTableThreads = 256;
constexpr uint32_t kTableBlocks = 32;  // at most

// Resident blocks per CU of the streaming kernels (0: as many as registers
// and waves allow), held there by a dynamic LDS reservation the kernel never
// touches.  HBM serves mixed reads and writes best with about 48 KB of loads
// open per CU, and the more of them come in one block's burst the better;
// kernels that only read want more open.  Measured on MI355X, same arrays, one
// process (us at the blocks per CU given, 1.24 B bf16 weights; the optimizer
// steps are in lc_optim.hip):
//   ACCUM score (two reads, one write; 16 KB of loads a block): 2: 1292, 3:
//     1132, 4: 1147, 5: 1163;
//   SNAPSHOT score (two reads): 3: 829, 4: 749, 5: 693, 6: 718;
//   pack (copies, 8 KB a block), a fifth of the layers: 4: 787, 5: 779, 6:
//     789, 8: 807; with the shadow refreshed 846, 847, 859, 880.
// Not kept: several chunks or pieces per block (score 1157-1360, pack 786-829),
// blocks of one wave (score 1181-1258), and the chunk's addresses in one table
// entry with the kernel arguments preloaded (1130-1133: the lookups are hidden).
// Only the score lifts its cap where every block is resident (lc_kernels.hip);
// of 3.7 M fp32 weights the pack takes 6.3 us with the cap or without, AdamW 19.8
// with it and 19.1 without.
#ifndef LC_SCORE_ACCUM_BLOCKS_PER_CU
#define LC_SCORE_ACCUM_BLOCKS_PER_CU 3
#endif
#ifndef LC_SCORE_SNAPSHOT_BLOCKS_PER_CU
#define LC_SCORE_SNAPSHOT_BLOCKS_PER_CU 5
#endif
#ifndef LC_COPY_BLOCKS_PER_CU
#define LC_COPY_BLOCKS_PER_CU 5
#endif
#ifndef LC_OPT_BLOCKS_PER_CU
#define LC_OPT_BLOCKS_PER_CU 0  // 0: by the bytes a block loads (lc_optim.hip)
#endif
// Dynamic LDS bytes per block that leave room for at most `blocks_per_cu`
// blocks on a CU of the current device (0 when blocks_per_cu is 0 or the
// device's limits leave no such size).
uint32_t occupancy_lds(uint32_t blocks_per_cu);

// A segment may start at any element, as the pieces of a ZeRO-3 rank do.  Its
// first `head` elements run up to a 128-byte line of one of its arrays; the
// chunks' tiles follow from there, so every tile starts on a line whatever the
// segment starts on, and the first chunk holds the head beside its tile.  The
// segment has ceil(numel / chunk elements) chunks whatever its head; with a
// head, the last of them may hold no element.  Each kernel's head is of the
// array whose stores weigh most: a store that starts inside a line leaves two
// partial lines where a block ends (measured on one 160 M element segment 16 B
// past a line: ACCUM score 189 -> 160 us, AdamW 1040 -> 818 us, SGD 469 -> 360
// us), an unaligned load costs a few percent.
constexpr uint32_t kLineBytes = 128u;
inline uint16_t seg_head(uint64_t addr, uint32_t esz) {
  return static_cast<uint16_t>((kLineBytes - addr % kLineBytes) % kLineBytes / esz);
}

// How the score kernel reads a segment's vectors and adds up their terms.
enum ScoreForm : uint16_t {
  kScorePairs = 0,    // w and s 16-B aligned: 16-B vectors, summed pairwise in fp32
  kScoreWide = 1,     // w and s alike modulo 16: aligned vectors behind the head, each term added in fp64
  kScoreWideAny = 2,  // w at any element against s: unaligned loads of w, each term added in fp64
};

// One segment as the score kernel sees it.
struct ScoreSeg {
  uint64_t w;            // device address of the weights
  uint64_t s;            // device address of the shadow
  uint64_t numel;
  uint32_t chunk_begin;  // global index of the segment's first chunk
  uint16_t form;         // ScoreForm
  uint16_t head;         // elements before the first tile
};
inline ScoreSeg score_seg(uint64_t w, uint64_t s, uint64_t numel, uint32_t esz, uint32_t chunk_begin) {
  ScoreSeg g;
  g.w = w;
  g.s = s;
  g.numel = numel;
  g.chunk_begin = chunk_begin;
  g.form = w % 16 == 0 && s % 16 == 0 ? kScorePairs : w % 16 == s % 16 ? kScoreWide : kScoreWideAny;
  g.head = seg_head(s ? s : w, esz);
  return g;
}

// One block of a layer record: one array (W, master, m or v) of one segment.
struct CopyUnit {
  uint64_t arr;      // device address of the array range
  uint64_t shadow;   // shadow range for W units, 0 otherwise
  uint64_t rec_off;  // byte offset of the block inside the record (256-B aligned)
  uint64_t bytes;    // payload bytes (the block is padded to kRecordAlign)
  uint32_t piece0;   // first layer-local piece index of this unit
  uint32_t head;     // bytes of arr before its first 128-byte line (at most `bytes`)
  uint32_t elem;     // element size in bytes (2 or 4)
  uint32_t pad;
};

// How the optimizer kernels read a segment's groups of four elements and add
// up their drift terms.
enum OptForm : uint16_t {
  kOptPairs = 0,  // every array group-aligned at element 0: summed pairwise in fp32 (if the gradient is, too)
  kOptWide = 1,   // every array group-aligned behind the head: each term added in fp64
  kOptAny = 2,    // arrays at any element against each other: unaligned accesses, each term added in fp64
};

// One segment as the optimizer kernels see it (static part).
struct OptSeg {
  uint64_t w;            // weights (bf16 or fp32)
  uint64_t master;       // fp32 master, 0 when absent
  uint64_t m;            // fp32 Adam first moment (AdamW only)
  uint64_t v;            // fp32 Adam second moment (AdamW only)
  uint64_t numel;
  uint32_t chunk_begin;  // same chunks as the score kernel
  uint16_t form;         // OptForm
  uint16_t head;         // elements before the first tile
};

// Per-call part: gradient address and weight-decay flag of each segment.
struct GradSeg {
  uint64_t grad;
  uint32_t decay;
  uint32_t vec_ok;  // gradient aligned to 4 elements at element 0
};

// The gradient table of a layout of up to kInlineGrads segments goes into the
// kernel's arguments (their limit is 4 KiB): no table in memory, no launch to
// fill it and no gap behind that (with select and pack, fetched table against
// arguments, three pairs: AdamW step on 3.7 M parameters 44.7-44.9 -> 41.4-42.2 us,
// SGD step on 336 M 747 -> 742).
constexpr uint32_t kInlineGrads = 224;
struct InlineGrads {
  GradSeg g[kInlineGrads];
};

// fp32 scalars of one AdamW step, formed in fp64 on the host and rounded once.
struct AdamScalars {
  float b1, omb1, b2, omb2, c1, c2, eps, lr, decay;
};

// fp32 scalars of one SGD step: lr and the decoupled decay factor 1 - lr wd.
struct SgdScalars {
  float lr, decay;
};

// Written by the select kernel to pinned host memory, followed by the 0/1 mask
// of n_layers bytes.  `seq` is written last, after system-scope fences: the
// host waits for the number it passed to the kernel instead of synchronising
// the stream.
struct SelectHeader {
  uint32_t n_selected;
  uint32_t n_forced;
  uint64_t payload_bytes;
  int64_t max_age;
  double weighted_age;
  uint64_t total_pieces;
  uint64_t age_numerator;
  uint64_t seq;
  uint64_t reserved;
};
static_assert(sizeof(SelectHeader) == 64, "header layout");

// One rank of a restore: the address of its record, the pieces of the ranks
// before it (the entry behind the last holds their total), where its own
// pieces begin in piece_unit, and the step that its record was persisted at.
struct RankEntry {
  uint64_t src;
  uint64_t piece_prefix;
  uint64_t piece_begin;
  int64_t step;
};

// The ranks of a restore of every layer of a layout of few layers go into the
// kernel's arguments, and the kernel sets Delta and t_l itself: one launch
// instead of three and no table to fetch.
constexpr uint32_t kInlineRanks = 108;
struct UnpackArgs {
  const uint32_t* piece_unit;
  const CopyUnit* units;
  const RankEntry* ranks;  // null: `inline_ranks`, which are every layer in order
  double* delta;
  int64_t* t_last;
  uint64_t piece_base;     // first piece of this launch
  uint32_t n_ranks;
  uint32_t pad;
  RankEntry inline_ranks[kInlineRanks + 1];
};
static_assert(sizeof(UnpackArgs) < 4096 - 256, "kernel arguments, with the launch's own");

// Pinned host memory that small tables pass through, in both directions.
// Followed by u, Delta and t_l of n_layers each (written by the device), then
// n_layers + 1 RankEntry and n_layers steps of a restore (written by the host).
// grad_seq is written by the device when the gradient table has been read.
struct HostState {
  uint64_t grad_seq;
  uint64_t reserved[7];
};
static_assert(sizeof(HostState) == 64, "tables stay 16-byte aligned");

// Device-resident state of one context.
struct DeviceTables {
  uint32_t n_layers;
  uint32_t n_chunks;
  uint64_t total_numel;
  int dtype;  // 1 bf16, 2 f32
  int mode;   // 0 accum, 1 snapshot
  double eps_w;
  int64_t s_max;

  const ScoreSeg* segs;
  const uint32_t* chunk_seg;          // [n_chunks]
  const uint32_t* layer_chunk_begin;  // [N+1]
  double2* partials;                  // [n_chunks] (sum|W-S|, sum|S|)
  double* u;                          // [N]
  double* delta;                      // [N]
  int64_t* t_last;                    // [N]
  const double* k0;                   // [N]
  const uint64_t* numel;              // [N]
  const uint64_t* rec_bytes;          // [N]
  const uint64_t* layer_pieces;       // [N] pieces of one record
  const CopyUnit* units;              // all units, layer-major, record order
  const uint32_t* piece_unit;         // layout-wide piece -> unit index
  const uint64_t* layer_piece_begin;  // [N+1] offset of each layer in piece_unit
  uint32_t* sel_layer;                // [N] layer of each selected rank
  uint64_t* sel_rec_prefix;           // [N+1] record byte offsets by rank
  uint64_t* sel_piece_prefix;         // [N+1] piece offsets by rank
  SelectHeader* host_result;          // pinned host memory (device address): header + mask[N]
  const OptSeg* opt_segs;             // [n_segments]
  const GradSeg* grad_segs;           // [n_segments], refreshed per optimizer call; null: InlineGrads
  RankEntry* ranks;                   // [N+1] restore scratch
};

// Launchers: return hipGetLastError() of the launches; the fetch, the state's
// kernels and the unpack their own launches' error only.
// launch_score: score kernel, then the finalize kernel (u and Delta).
hipError_t launch_score(const DeviceTables& t, hipStream_t st);
// Eq. 1-2 from the per-chunk partials alone (after an optimizer step).
hipError_t launch_finalize(const DeviceTables& t, hipStream_t st);
hipError_t launch_select(const DeviceTables& t, int64_t step, double lr_scale, int base_mode, uint64_t seq,
                         hipStream_t st);
// Small tables through pinned host memory (HostState): device addresses.
hipError_t launch_fetch(const void* host_src, void* dst, uint32_t n16, uint64_t* flag, uint64_t seq, hipStream_t st);
hipError_t launch_push_state(const DeviceTables& t, HostState* host, hipStream_t st);
hipError_t launch_reset_state(const DeviceTables& t, const int64_t* host_steps, int64_t step, hipStream_t st);
hipError_t launch_pack(const DeviceTables& t, uint32_t first_rank, uint32_t last_rank,
                       uint64_t piece_base, uint64_t n_pieces, uint64_t rec_base,
                       void* staging, int refresh_shadow, hipStream_t st);
// ranks (host, n_ranks + 1 entries): every layer, at most kInlineRanks, and
// Delta and t_l are set, too; null: the ranks are in t.ranks.
hipError_t launch_unpack(const DeviceTables& t, const RankEntry* ranks, uint32_t n_ranks, uint64_t n_pieces,
                         hipStream_t st);
// Optimizer steps writing the per-chunk drift partials (lc_optim.hip).
// t.grad_segs null: the gradient table is `grads`.
hipError_t launch_adamw(const DeviceTables& t, const InlineGrads& grads, int grad_dtype, int has_master,
                        const AdamScalars& sc, hipStream_t st);
hipError_t launch_sgd(const DeviceTables& t, const InlineGrads& grads, int grad_dtype, int has_master,
                      const SgdScalars& sc, hipStream_t st);

}  // namespace lc
