// Internal interface between the C ABI (psa_api.hip) and the kernels (psa_kernels.hip).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include <hip/hip_runtime.h>

#include "psa.h"

namespace psa {

// Number of work queues of the sparse scheduler: one per XCD of an MI355X (8 XCDs of 32 CUs).
constexpr int kNumQueues = 8;

// Heads whose stripe parameters travel in one kernel-argument block.
constexpr int kHeadsPerChunk = 64;

struct ParamChunk {
  int32_t n;                        // heads in this chunk
  psa_stripe_t m[kHeadsPerChunk];
};

// Sequence geometry in blocks.  With one-dimensional blocks (pbt = 0) a block is `block`
// consecutive tokens of the frame-major sequence.  With 3D PSABlocks (pbt > 0) the sequence is
// the PSABlock-centric layout: the padded grid ordered (T', H', W', bt, bh, bw), then the text
// tokens; a block (tile) is `block` consecutive positions of it, and a PSABlock is a whole
// number of tiles.
struct Geometry {
  int32_t hw;       // tokens per frame of the video grid, H*W
  int32_t n_video;  // F*H*W
  int32_t n;        // tokens of the sequence: n_video + n_text, or n_blk + n_text (3D)
  int32_t n_text;
  int32_t block;
  int32_t nb;       // ceil(n / block)
  int32_t frames, height, width;
  int32_t pbt, pbh, pbw;   // PSABlock shape; pbt = 0 for one-dimensional blocks
  int32_t tp, hp, wp;      // PSABlock grid T', H', W' (3D)
  int32_t n_blk;           // positions of the padded video grid, T'H'W' * pbt*pbh*pbw (3D)
};

// Coordinate of a tile that holds only padding: never kept as a key, no work as a query.
constexpr int32_t kDeadTile = -2;

// Identifies a finished plan in the workspace header; the sizes it was made for follow it.
// Block 64 has a number of its own: "PSA1" plans of it list single query blocks, and a run that took
// them for pairs would read the pairs of an unwritten section.
constexpr uint32_t kPlanMagic = 0x50534131u;    // "PSA1"
constexpr uint32_t kPlanMagic64 = 0x50534132u;  // "PSA2"
// Set in the magic of a plan in which every head keeps every key block (or may, see plan_full), where
// the engine of a run depends on that.
constexpr uint32_t kPlanFull = 0x80000000u;

struct PlanHeader {
  uint32_t magic;   // kPlanMagic*, maybe with kPlanFull, once the plan's kernels have run, 0 while they run
  int32_t n_bh;     // batch * n_heads
  int32_t n_heads;
  int32_t nb;
  int32_t block;
  int32_t n;
  int32_t frames, height, width, n_text;
  int32_t pbt, pbh, pbw;
};

// Layout of the queue area (int32 words): kNumQueues + 1 boundaries in the first 128-byte line,
// then one pop counter per queue, each in a line of its own (device-scope atomics on one line
// are serialised).
constexpr int kCounterStride = 32;
constexpr int kQueueCounters = 32;
constexpr int kQueueWords = kQueueCounters + kNumQueues * kCounterStride;
// Word of the first line (after the boundaries) counting the finished workgroups of the plan's
// last kernel (psa_starts_kernel).
constexpr int kStartsDone = 16;
// Another one: whether runs of head dim 64 at block 128 take each pair as two items (halves_pay), set by
// the plan.
constexpr int kHalvesWord = 17;
static_assert(kStartsDone > kNumQueues && kHalvesWord < kQueueCounters, "free words of the first line");

// Workspace of psa_dense_fwd: the queue area alone, rounded up to 256 bytes.
constexpr size_t kDenseWorkspaceBytes = (sizeof(int32_t) * kQueueWords + 255) / 256 * 256;

// Workspace of psa_attention_plan / psa_attention_run (byte offsets, each 256-aligned).
struct WorkspaceLayout {
  size_t header;    // PlanHeader
  size_t params;    // psa_stripe_t [n_heads]
  size_t coords;    // int2 [nb]: (frame, slot) of each block, frame = -1 for a global block
  size_t counts;    // int32 [batch*n_heads*nb], the first batch*n_heads*ceil(nb/2): key blocks kept by
                    // either row of each pair item
  size_t order;     // the same: pair items in schedule order
  size_t queues;    // int32 [kQueueWords]: queue boundaries and pop counters
  size_t sigs;      // uint64 [n_heads][nb]: signature of each query block's kept set
  size_t pairs;     // int2 [n_heads][ceil(nb/2)]: query blocks paired into one work item
  size_t spans;     // uint32 [batch*n_heads*ceil(nb/2)]: first and last kept non-global key block
                    // of each pair item (bits 0-15, 16-31; 0xffffffff: none)
  size_t runspans;  // uint32 [batch*n_heads*ceil(nb/2)]: union of the spans of the items of the
                    // item's run (its head's range in its queue; a long item alone)
  size_t starts;    // int32 [batch*n_heads*ceil(nb/2)]: key block each pair item's stream starts at
  size_t masks;     // uint64 [nb][2]: valid positions of each tile (3D only)
  size_t total;
};

// Query blocks of one head processed together by the pair engine: ceil(nb / 2) pairs per head, the
// second member -1 for a single.
__host__ __device__ inline int32_t pairs_per_head(int32_t nb) { return (nb + 1) / 2; }

// Whether an axis of `extent` positions keeps every distance: the residues of |delta - offset|, which
// takes every value of [lo, hi], all lie below the width.
inline bool axis_full(int32_t w, int32_t o, int32_t s, int32_t extent) {
  if (w >= s) return true;
  const int64_t a = o < 0 ? -(int64_t)o : o, lo = std::max<int64_t>(0, a - (extent - 1)), hi = a + extent - 1;
  return lo % s + (hi - lo) < w;
}

// Whether every head keeps every key block.  Never for PSABlocks (their dense counterpart runs on
// another sequence).  A head keeps everything if it keeps every distance between two blocks that are
// not global, on either axis: each such distance belongs to a pair of blocks, which needs both axes.
// With a block no longer than a frame the coordinates of the n_local blocks before the first global
// one are whole ranges from zero: every frame up to that of the last of them starts a block, and the
// first frame's blocks are slots 0, 1, ...  (The text of the first global block may have taken the
// video's last frame or slot from the map.)  Where a block is longer than a frame not every frame
// starts one, so stripes that miss only distances no two blocks have would pass for sparse: such
// grids count as full.
inline bool plan_full(const Geometry& g, const psa_stripe_t* params, int32_t n_heads) {
  if (g.pbt > 0) return false;
  const int32_t n_local = g.n_text > 0 ? g.n_video / g.block : g.nb;
  if (g.block > g.hw || n_local == 0) return true;
  const int32_t frames = (int32_t)((int64_t)(n_local - 1) * g.block / g.hw) + 1;
  const int32_t slots = std::min((g.hw - 1) / g.block + 1, n_local);
  for (int32_t h = 0; h < n_heads; h++)
    if (!axis_full(params[h].t_w, params[h].t_o, params[h].t_s, frames) ||
        !axis_full(params[h].s_w, params[h].s_o, params[h].s_s, slots))
      return false;
  return true;
}

// Which problems run on the split engine, by their query blocks; the lines are for the 256 CUs of an
// MI355X (fixed numbers: a plan and its runs have to agree).
//  * Up to one workgroup per CU (at block 64, two of the half as large ones): always.
//  * Up to two: unless every head keeps every key block.  Rows of unequal length gain 1.0 to 1.75
//    times over pairs (28 drawn calls: 1.08 in the mean), because the longest pair sets the time;
//    rows of equal length lose up to 13 %, two rounds of half the work and more for one.  The dense
//    path therefore stays on pairs, and so does the sparse path at full density, where it returns
//    the dense path's bits.  At block 128 also not with two to eight blocks per head, whose rows
//    differ by little (head dim 128: 200 heads x 256 tokens 22.1 us split and 18.2 in pairs, 128 x 512
//    28.8 and 24.7, 64 x 1024 35.4 and 31.2; but 40 x 1280 31.9 and 32.7, 25 x 2048 39.1 and 47.9).
//    Beyond two the longest-first list of pairs is 2 % faster in the mean (24 drawn calls).
inline bool split_any(int32_t n_bh, int32_t nb, int32_t block) { return n_bh * nb <= 256 * (128 / block); }
inline bool split_sparse(int32_t n_bh, int32_t nb, int32_t block) {
  return split_any(n_bh, nb, block) || (n_bh * nb <= 512 * (128 / block) && (block == 64 || nb == 1 || nb > 8));
}
// Whether the density decides; such a plan's header says which it is (kPlanFull).
inline bool split_by_density(int32_t n_bh, int32_t nb, int32_t block) {
  return split_sparse(n_bh, nb, block) && !split_any(n_bh, nb, block);
}
// Whether no run of this plan needs pairs.
inline bool split_plan(int32_t n_bh, int32_t nb, int32_t block, bool full) {
  return split_any(n_bh, nb, block) || (!full && split_sparse(n_bh, nb, block));
}

// Head dim 64 at block 128: whether a run takes every pair of query blocks as two items of one block
// each, on four-wave workgroups, four to a CU (psa_pair_kernel<64, 64, 2>), or as one item on an
// eight-wave one, one to a CU (<64, 128, 1>).  Four workgroups per CU hide more latency, but an item
// that outlasts the others of its CU then runs on at one wave per SIMD, and every block streams K and
// V for itself.  Two items pay where a CU's share of the work is at least 1.4 times the longest pair
// and pairs keep six blocks or more in the mean: of the lines tried (0.8 to 2.5 times, 3 to 12 blocks)
// the one with the best mean over 201 calls of 2 to 591 blocks per head at densities of 0.05 to 1.
// There it is 1.08 times as fast as one item always with the order by heads, the slowest call 0.94;
// two items always are 1.04, the slowest 0.75.  One item and two: 12 heads x 17776 tokens at density
// 0.25 297 and 356 us, 16 x 7800 84 and 103; 60 x 17776 1414 and 1322, 24 x 3600 at density 1 126 and
// 107.
// `work` and `longest` count kept key blocks over the plan's n_items pairs.
constexpr int64_t kHalvesShare = 7 * 256, kHalvesUnit = 5;     // 1.4 times the longest, on each of 256 CUs
constexpr int32_t kHalvesMean = 6;
__host__ __device__ inline bool halves_pay(int64_t work, int64_t longest, int64_t n_items) {
  return work * kHalvesUnit >= kHalvesShare * longest && work >= kHalvesMean * n_items;
}
// Whether any plan of these sizes can pass that line (every item keeping every block): where this says
// no, no plan's word says yes.
inline bool halves_possible(int32_t block, int64_t n_items, int32_t nb) {
  return block == 128 && halves_pay(n_items * nb, nb, n_items);
}

WorkspaceLayout workspace_layout(int32_t batch, int32_t n_heads, int32_t nb, bool masks);

// Launchers; each returns the hipError_t of its launch(es).
hipError_t launch_blockmap(const ParamChunk& pc, int32_t head0, const Geometry& g,
                           uint8_t* blockmap, int32_t* kept_per_row, int64_t* kept_per_head,
                           hipStream_t stream);

// PSABlock-level block map: groups 0 .. T'H'W'-1 are the PSABlocks, group T'H'W' (with text)
// the text; g.nb must be the group count.
hipError_t launch_group_blockmap(const ParamChunk& pc, int32_t head0, const Geometry& g,
                                 uint8_t* blockmap, int32_t* kept_per_row, int64_t* kept_per_head,
                                 hipStream_t stream);

// Chunks per (batch, head) of the L2 distance's first pass.
constexpr int kL2Chunks = 64;

// Per (batch, head) sums of (o - ref)^2 and ref^2 over [tokens][d] bf16 rows: fp32 partial sums
// per chunk, combined in fp64 in a fixed order (partial: kL2Chunks * 2 doubles per row).
hipError_t launch_l2(const void* o, const void* ref, int32_t n_bh, int64_t elems_per_bh,
                     double* partial, double* sq_err, double* sq_ref, hipStream_t stream);

// PSABlock-centric layout of [bh][tokens][d] tensors (to: original -> blocked, else back).
hipError_t launch_layout(const void* src, void* dst, int32_t n_bh, int32_t head_dim,
                         const Geometry& g, bool to_blocks, hipStream_t stream);

// The plan: stripe parameters (chunks of kHeadsPerChunk heads) and block coordinates, the pairs of
// query blocks, their work and their order; the header last.
hipError_t launch_plan(const ParamChunk* chunks, const Geometry& g, int32_t batch, int32_t n_heads,
                       bool full, void* workspace, const WorkspaceLayout& wl, int32_t* kept_per_row,
                       hipStream_t stream);

// full: right after the plan's own kernels whether it is full (they leave the queue counters at zero);
// -1 for a run of an earlier plan, whose counters are set first.
hipError_t launch_sparse(const void* q, const void* k, const void* v, void* o, float* lse,
                         int32_t batch, int32_t n_heads, int32_t head_dim, const Geometry& g,
                         float scale_log2, void* workspace, const WorkspaceLayout& wl,
                         int32_t cus, hipStream_t stream, int32_t full);

// queues: the int32 [kQueueWords] queue area of a dense workspace (persistent grid), or nullptr
// (one workgroup per work item).
hipError_t launch_dense(const void* q, const void* k, const void* v, void* o, float* lse,
                        int32_t batch, int32_t n_heads, int32_t head_dim, int32_t n_tokens,
                        int32_t block, float scale_log2, int32_t* queues, int32_t cus, hipStream_t stream);

// Device address of the static scratch of psa_attention_fwd_noalloc on the current device
// (PSA_NOALLOC_SCRATCH_BYTES, 256-byte aligned), looked up once per device.
hipError_t scratch_pointer(void** out);

}  // namespace psa
