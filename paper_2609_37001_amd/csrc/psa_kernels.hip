// PSA block-sparse attention forward: HIP kernels for gfx950 (CDNA4, MI355X).
//
// Kernels
//   psa_map_kernel                             block map and kept counts (Algorithm 1 per block)
//   psa_setup_kernel                           stripe parameters and block coordinates -> workspace
//   psa_count_kernel                           kept key blocks of every (batch, head, query block),
//                                              and kept-set signatures for the pairing
//   psa_pairing_kernel / psa_paircount_kernel  pairs of query blocks and their work
//   psa_head_plan_kernel                       all of these for a head of a short sequence
//   psa_rank_kernel                            work order of a short list: longest first, over 8 XCD
//                                              queues
//   psa_schedule_kernel                        ... of a long one: by heads, load-balanced
//   psa_starts_kernel                          block 128: where each pair item's K/V stream starts
//   psa_pair_kernel                            persistent block-sparse attention (Algorithm 2) on
//                                              pairs of query blocks, or dense
//   psa_split_kernel                           the same for few query blocks, one workgroup each
//
// Tile engine (per wave; a workgroup holds 2 BLK rows in 2 BLK/32 wave64s, and PairShape says how
// many share a CU; head dim D):
//   * every wave owns 32 query rows of a query block and all keys of each key/value block; lane l
//     holds row l & 31, lanes l and l ^ 32 split its keys.  A block is processed in steps of 64
//     keys, each with its own online-softmax update.
//   * S^T = K Q^T with v_mfma_f32_32x32x16_bf16: K rows come from LDS (A operand), Q^T stays in
//     registers (B operand).  K rows are read in a permuted order so that each lane's fp32
//     accumulators hold 8 consecutive keys of every 16-key chunk, which is exactly the B operand
//     layout of the next product: P^T needs no data movement.
//   * O^T += V^T P^T: V stays row-major in LDS and the A operand is assembled with the gfx950 LDS
//     transpose read (ds_read_b64_tr_b16).
//   * K and V fill LDS by direct global->LDS 16-byte loads (global_load_lds_dwordx4): a double
//     buffer shared by the two query blocks of a pair, one barrier per block.  16-byte chunks are
//     XOR-swizzled per row so both the K reads and the transposed V reads are bank-conflict free at
//     head dim 128 (see swz).
//   * Softmax in the exp2 domain: Q is multiplied by scale*log2(e) once, and the S^T
//     accumulators start at -m, so the MFMAs deliver the exponent directly; m is raised lazily
//     (only when a weight would reach 2^8, at head dim 64 2), which is exact.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "psa_launch.h"

namespace psa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

#define PSA_LDS __attribute__((address_space(3)))

// ---------------------------------------------------------------------------------------------
// Stripe decoder: Algorithm 1 evaluated on block coordinates.
// ---------------------------------------------------------------------------------------------

// One axis of Algorithm 1: (|delta - offset| mod stride) <= width - 1.
__device__ __forceinline__ bool axis_keep(int32_t delta, int32_t width, int32_t offset,
                                          int32_t stride) {
  const int32_t x = delta - offset;
  const uint32_t ax = (uint32_t)(x < 0 ? -x : x);
  return (ax % (uint32_t)stride) < (uint32_t)width;
}

// The same test for many distances of one stripe, without a division: x / stride as a multiplication
// by a 32-bit reciprocal (Granlund and Montgomery, "Division by invariant integers using
// multiplication"): with 2^(l-1) < stride <= 2^l and mul = ceil(2^(31+l) / stride), the quotient
// of any x < 2^31 is (x mul) >> (31 + l).
struct AxisTest {
  uint32_t mul, shift, stride, width;
  int32_t offset;

  __device__ __forceinline__ AxisTest(int32_t w, int32_t o, int32_t s) {
    // A stripe at least as wide as its stride keeps the whole axis.
    const bool all = w >= s;
    stride = all ? 0x7fffffffu : (uint32_t)s;               // >= 2
    width = all ? 0x7fffffffu : (uint32_t)w;
    offset = all ? 0 : o;
    const uint32_t l = 32 - __builtin_clz(stride - 1);
    mul = (uint32_t)(((1ull << (31 + l)) + stride - 1) / stride);
    shift = l - 1;
  }
  __device__ __forceinline__ bool keep(int32_t delta) const {
    const int32_t x = delta - offset;
    const uint32_t ax = (uint32_t)(x < 0 ? -x : x);
    return ax - (__umulhi(ax, mul) >> shift) * stride < width;
  }
};

// Coordinates of block b from its first token: frame t and slot s; t = -1 marks a global block
// (a block holding at least one appended text token).
__device__ __forceinline__ int2 block_coord(const Geometry& g, int32_t b) {
  const int32_t i0 = b * g.block;
  const int32_t len = min(g.block, g.n - i0);
  if (g.n_text > 0 && i0 + len > g.n_video) return make_int2(-1, 0);
  const int32_t t = i0 / g.hw;
  return make_int2(t, (i0 - t * g.hw) / g.block);
}

// Coordinates of tile b of the PSABlock-centric layout: those of the PSABlock holding it
// (t', s' = h' W' + w'), or global for a text tile.  A PSABlock is a whole number of tiles.
__device__ __forceinline__ int2 tile_coord3d(const Geometry& g, int32_t b) {
  const int32_t i0 = b * g.block;
  if (i0 >= g.n_blk) return make_int2(-1, 0);
  const int32_t pb = i0 / (g.pbt * g.pbh * g.pbw), plane = g.hp * g.wp;
  const int32_t t = pb / plane;
  return make_int2(t, pb - t * plane);
}

// Coordinates of group i of a PSABlock-level map: PSABlock i, or the text group (global).
__device__ __forceinline__ int2 group_coord(const Geometry& g, int32_t i) {
  const int32_t plane = g.hp * g.wp;
  if (i >= g.tp * plane) return make_int2(-1, 0);
  const int32_t t = i / plane;
  return make_int2(t, i - t * plane);
}

// Whether position p of the PSABlock-centric layout holds a token (not 3D padding, not past
// the end).
__device__ __forceinline__ bool position_valid(const Geometry& g, int32_t p) {
  if (p >= g.n) return false;
  if (p >= g.n_blk) return true;
  const int32_t area = g.pbh * g.pbw, vol = g.pbt * area, plane = g.hp * g.wp;
  const int32_t pb = p / vol, x = p - pb * vol;
  const int32_t tq = pb / plane, r = pb - tq * plane, hq = r / g.wp, wq = r - hq * g.wp;
  const int32_t it = x / area, r2 = x - it * area, ih = r2 / g.pbw, iw = r2 - ih * g.pbw;
  return tq * g.pbt + it < g.frames && hq * g.pbh + ih < g.height && wq * g.pbw + iw < g.width;
}

__device__ __forceinline__ bool tile_keep(const psa_stripe_t& m, int2 q, int2 k) {
  if (q.x == kDeadTile || k.x == kDeadTile) return false;
  if (q.x < 0 || k.x < 0) return true;
  return axis_keep(k.x - q.x, m.t_w, m.t_o, m.t_s) && axis_keep(k.y - q.y, m.s_w, m.s_o, m.s_s);
}

__device__ __forceinline__ int wave_sum(int v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Wave-wide sum (OP 0), minimum (1) or maximum (2) in every lane, without LDS: DPP moves
// within the 16-lane rows, then the gfx950 permlane swaps across rows.
template <int OP>
__device__ __forceinline__ int32_t wave_reduce(int32_t v) {
  auto op = [](int32_t a, int32_t b) { return OP == 0 ? a + b : (OP == 1 ? min(a, b) : max(a, b)); };
  v = op(v, __builtin_amdgcn_update_dpp(v, v, 0xb1, 0xf, 0xf, false));   // quad_perm 1,0,3,2
  v = op(v, __builtin_amdgcn_update_dpp(v, v, 0x4e, 0xf, 0xf, false));   // quad_perm 2,3,0,1
  v = op(v, __builtin_amdgcn_update_dpp(v, v, 0x124, 0xf, 0xf, false));  // row_ror:4
  v = op(v, __builtin_amdgcn_update_dpp(v, v, 0x128, 0xf, 0xf, false));  // row_ror:8
  const auto r16 = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
  v = op((int32_t)r16[0], (int32_t)r16[1]);                               // lanes l, l ^ 16
  const auto r32 = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
  return op((int32_t)r32[0], (int32_t)r32[1]);                            // lanes l, l ^ 32
}

// Lane i receives lane i ^ m of x (m = 1, 2, 4, 8 by DPP within a 16-lane row; 16 by a shuffle).
template <int M>
__device__ __forceinline__ int32_t lane_xor(int32_t x, int lane) {
  if constexpr (M == 1) return __builtin_amdgcn_update_dpp(x, x, 0xb1, 0xf, 0xf, false);  // quad_perm 1,0,3,2
  if constexpr (M == 2) return __builtin_amdgcn_update_dpp(x, x, 0x4e, 0xf, 0xf, false);  // quad_perm 2,3,0,1
  if constexpr (M == 4) {
    const int32_t fwd = __builtin_amdgcn_update_dpp(x, x, 0x104, 0xf, 0xf, false);      // row_shl:4
    const int32_t bwd = __builtin_amdgcn_update_dpp(x, x, 0x114, 0xf, 0xf, false);      // row_shr:4
    return (lane & 4) ? bwd : fwd;
  }
  if constexpr (M == 8) return __builtin_amdgcn_update_dpp(x, x, 0x128, 0xf, 0xf, false); // row_ror:8
  return __shfl_xor(x, M);
}

// Inclusive prefix sum over the lanes of a wave: shifted DPP adds within each row, then the
// totals of the rows below added from scalar reads of their last lanes.
__device__ __forceinline__ int32_t wave_incl_sum(int32_t v, int lane) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);         // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);         // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);         // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);         // row_shr:8
  const int32_t r0 = __builtin_amdgcn_readlane(v, 15), r1 = __builtin_amdgcn_readlane(v, 31),
                r2 = __builtin_amdgcn_readlane(v, 47);
  const int row = lane >> 4;
  return v + (row > 0 ? r0 : 0) + (row > 1 ? r1 : 0) + (row > 2 ? r2 : 0);
}

// ---------------------------------------------------------------------------------------------
// Block map (psa_build_blockmap).
// ---------------------------------------------------------------------------------------------

// Coordinates of entry i of a block map: a one-dimensional block, or a PSABlock-level group.
template <bool GROUPS>
__device__ __forceinline__ int2 map_coord(const Geometry& g, int32_t i) {
  return GROUPS ? group_coord(g, i) : block_coord(g, i);
}

__global__ __launch_bounds__(256) void psa_zero_kernel(int64_t* __restrict__ x, int32_t n) {
  const int32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) x[i] = 0;
}

// Map rows, row counts and head totals in one pass (each output may be null).  A workgroup takes
// kMapRows rows of one head, a wave kMapRows / 4 of them; a lane decides four consecutive entries of
// each of its wave's rows at a time and stores them as one word (rows start at any byte).  TABLE:
// both axes' tests for every distance of the grid are looked up in LDS, filled once per workgroup;
// without (an axis of more than kMapExtent positions) each is evaluated by multiplication.
// The map's bytes alone would take 3 us at 40 heads x 591^2 entries (14 MB); what bounds the kernel
// are the vector and LDS instructions per entry, 22 us with the counts: a column's coordinates still
// cost two integer divisions for every four rows (the tests of the stripes cost none), and a workgroup
// begins with those of its rows and two 64-bit ones.  One byte, four divisions and two moduli per
// thread took 63 us, and the counts of one workgroup per head 403 us more.
constexpr int kMapRows = 16;
constexpr int kMapExtent = 4096;
template <bool GROUPS, bool TABLE>
__global__ __launch_bounds__(256) void psa_map_kernel(ParamChunk pc, int32_t head0, Geometry g,
                                                      int32_t t_ext, int32_t s_ext,
                                                      uint8_t* __restrict__ map,
                                                      int32_t* __restrict__ kept_per_row,
                                                      unsigned long long* __restrict__ kept_per_head) {
  constexpr int R = kMapRows / 4;
  __shared__ uint8_t t_keep[TABLE ? 2 * kMapExtent : 1], s_keep[TABLE ? 2 * kMapExtent : 1];
  __shared__ int32_t partial[4];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int32_t nb = g.nb, hc = blockIdx.y;
  const psa_stripe_t m = pc.m[hc];
  const AxisTest ta(m.t_w, m.t_o, m.t_s), sa(m.s_w, m.s_o, m.s_s);
  if constexpr (TABLE) {
    for (int32_t i = tid; i < 2 * t_ext - 1; i += 256) t_keep[i] = ta.keep(i - (t_ext - 1));
    for (int32_t i = tid; i < 2 * s_ext - 1; i += 256) s_keep[i] = sa.keep(i - (s_ext - 1));
    __syncthreads();
  }
  int2 cq[R];
  int32_t cnt[R];
  const int32_t q0 = blockIdx.x * kMapRows + wave * R;
#pragma unroll
  for (int r = 0; r < R; r++) {
    cq[r] = map_coord<GROUPS>(g, min(q0 + r, nb - 1));
    cnt[r] = 0;
  }
  for (int32_t k0 = 4 * lane; k0 < nb; k0 += 256) {
    int2 ck[4];
#pragma unroll
    for (int j = 0; j < 4; j++) ck[j] = map_coord<GROUPS>(g, min(k0 + j, nb - 1));
#pragma unroll
    for (int r = 0; r < R; r++) {
      if (q0 + r >= nb) break;
      uint32_t word = 0;
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int32_t dt = ck[j].x - cq[r].x, ds = ck[j].y - cq[r].y;
        uint32_t keep;
        if (cq[r].x < 0 || ck[j].x < 0)
          keep = 1;
        else if constexpr (TABLE)
          keep = t_keep[dt + t_ext - 1] & s_keep[ds + s_ext - 1];
        else
          keep = ta.keep(dt) && sa.keep(ds);
        word |= (k0 + j < nb ? keep : 0u) << (8 * j);
      }
      cnt[r] += __builtin_popcount(word);
      if (map) {
        uint8_t* dst = map + ((int64_t)(head0 + hc) * nb + q0 + r) * nb + k0;
        if (k0 + 3 < nb) {
          __builtin_memcpy(dst, &word, 4);
        } else {
          for (int j = 0; k0 + j < nb; j++) dst[j] = (uint8_t)(word >> (8 * j));
        }
      }
    }
  }
  int32_t total = 0;
#pragma unroll
  for (int r = 0; r < R; r++) {
    cnt[r] = wave_reduce<0>(cnt[r]);
    if (q0 + r < nb) {
      total += cnt[r];
      if (kept_per_row && lane == 0) kept_per_row[(int64_t)(head0 + hc) * nb + q0 + r] = cnt[r];
    }
  }
  if (kept_per_head) {
    if (lane == 0) partial[wave] = total;
    __syncthreads();
    if (tid == 0)
      atomicAdd(&kept_per_head[head0 + hc],
                (unsigned long long)((int64_t)partial[0] + partial[1] + partial[2] + partial[3]));
  }
}

template <bool GROUPS>
static hipError_t launch_map(const ParamChunk& pc, int32_t head0, const Geometry& g,
                             uint8_t* blockmap, int32_t* kept_per_row, int64_t* kept_per_head,
                             hipStream_t stream) {
  if (!blockmap && !kept_per_row && !kept_per_head) return hipSuccess;
  if (kept_per_head) {
    hipLaunchKernelGGL(psa_zero_kernel, dim3((pc.n + 255) / 256), dim3(256), 0, stream, kept_per_head + head0,
                       pc.n);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int32_t t_ext = GROUPS ? g.tp : g.frames;
  const int32_t s_ext = GROUPS ? g.hp * g.wp : (g.hw - 1) / g.block + 1;
  const dim3 grid((unsigned)((g.nb + kMapRows - 1) / kMapRows), (unsigned)pc.n);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, pc, head0, g, t_ext, s_ext, blockmap, kept_per_row,
                       (unsigned long long*)kept_per_head);
  };
  if (t_ext <= kMapExtent && s_ext <= kMapExtent)
    go(psa_map_kernel<GROUPS, true>);
  else
    go(psa_map_kernel<GROUPS, false>);
  return hipGetLastError();
}

hipError_t launch_blockmap(const ParamChunk& pc, int32_t head0, const Geometry& g,
                           uint8_t* blockmap, int32_t* kept_per_row, int64_t* kept_per_head,
                           hipStream_t stream) {
  return launch_map<false>(pc, head0, g, blockmap, kept_per_row, kept_per_head, stream);
}

hipError_t launch_group_blockmap(const ParamChunk& pc, int32_t head0, const Geometry& g,
                                 uint8_t* blockmap, int32_t* kept_per_row, int64_t* kept_per_head,
                                 hipStream_t stream) {
  return launch_map<true>(pc, head0, g, blockmap, kept_per_row, kept_per_head, stream);
}

// ---------------------------------------------------------------------------------------------
// PSABlock-centric layout (psa_to_blocks / psa_from_blocks): one workgroup per (batch*head,
// PSABlock), or per 64 text rows; 16-byte chunks, CPR per row.  The blocked side is written or
// read in order, the original side in runs of bw rows.
// ---------------------------------------------------------------------------------------------

// ---------------------------------------------------------------------------------------------
// L2 distance per (batch, head) (the loss of PSA-Search).
// ---------------------------------------------------------------------------------------------

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Fixed-order sum over a 256-thread workgroup (butterfly in each wave, then the four waves).
__device__ __forceinline__ double block_sum(double x, double* red) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  const double t = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return t;
}

__global__ __launch_bounds__(256) void psa_l2_partial_kernel(const uint4* __restrict__ o,
                                                             const uint4* __restrict__ ref,
                                                             int64_t vec_per_bh,
                                                             double* __restrict__ partial) {
  __shared__ double red[4];
  const int64_t per = (vec_per_bh + kL2Chunks - 1) / kL2Chunks;
  const int64_t lo = (int64_t)blockIdx.x * per, hi = min(lo + per, vec_per_bh);
  const uint4* a = o + (int64_t)blockIdx.y * vec_per_bh;
  const uint4* b = ref + (int64_t)blockIdx.y * vec_per_bh;
  float se = 0.0f, sr = 0.0f;
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
    const uint4 x = a[i], y = b[i];
    const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const float r0 = bf16_lo(ys[j]), r1 = bf16_hi(ys[j]);
      const float d0 = bf16_lo(xs[j]) - r0, d1 = bf16_hi(xs[j]) - r1;
      se = __builtin_fmaf(d0, d0, __builtin_fmaf(d1, d1, se));
      sr = __builtin_fmaf(r0, r0, __builtin_fmaf(r1, r1, sr));
    }
  }
  const double te = block_sum(se, red), tr = block_sum(sr, red);
  if (threadIdx.x == 0) {
    double* dst = partial + ((int64_t)blockIdx.y * kL2Chunks + blockIdx.x) * 2;
    dst[0] = te;
    dst[1] = tr;
  }
}

__global__ __launch_bounds__(64) void psa_l2_final_kernel(const double* __restrict__ partial,
                                                          double* __restrict__ sq_err,
                                                          double* __restrict__ sq_ref) {
  const double* p = partial + (int64_t)blockIdx.x * kL2Chunks * 2;
  double e = p[2 * threadIdx.x], r = p[2 * threadIdx.x + 1];
  for (int off = 32; off > 0; off >>= 1) {
    e += __shfl_xor(e, off);
    r += __shfl_xor(r, off);
  }
  if (threadIdx.x == 0) {
    sq_err[blockIdx.x] = e;
    if (sq_ref) sq_ref[blockIdx.x] = r;
  }
}

hipError_t launch_l2(const void* o, const void* ref, int32_t n_bh, int64_t elems_per_bh,
                     double* partial, double* sq_err, double* sq_ref, hipStream_t stream) {
  static_assert(kL2Chunks == 64, "the final pass sums one partial per lane of a wave");
  hipLaunchKernelGGL(psa_l2_partial_kernel, dim3(kL2Chunks, (unsigned)n_bh), dim3(256), 0, stream,
                     (const uint4*)o, (const uint4*)ref, elems_per_bh / 8, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(psa_l2_final_kernel, dim3((unsigned)n_bh), dim3(64), 0, stream, partial, sq_err,
                     sq_ref);
  return hipGetLastError();
}

template <bool TO, int CPR>
__global__ __launch_bounds__(256) void psa_layout_kernel(const uint4* __restrict__ src,
                                                         uint4* __restrict__ dst, Geometry g) {
  const int32_t n_p = g.tp * g.hp * g.wp;
  const size_t n_orig = (size_t)g.n_video + g.n_text, n_blkd = (size_t)g.n;
  const uint4* s = src + (size_t)blockIdx.y * (TO ? n_orig : n_blkd) * CPR;
  uint4* d = dst + (size_t)blockIdx.y * (TO ? n_blkd : n_orig) * CPR;
  if ((int32_t)blockIdx.x < n_p) {
    const int32_t pb = blockIdx.x, plane = g.hp * g.wp, area = g.pbh * g.pbw;
    const int32_t vol = g.pbt * area;
    const int32_t tq = pb / plane, r = pb - tq * plane, hq = r / g.wp, wq = r - hq * g.wp;
    const int32_t t0 = tq * g.pbt, h0 = hq * g.pbh, w0 = wq * g.pbw;
    // Four 16-byte chunks per thread and round: every load is issued before the first store.
    for (int32_t e0 = threadIdx.x; e0 < vol * CPR; e0 += 4 * 256) {
      size_t from[4], to[4];
      bool live[4];
      uint4 val[4];
#pragma unroll
      for (int u = 0; u < 4; u++) {
        const int32_t e = e0 + u * 256;
        const int32_t x = e / CPR, c = e % CPR;
        const int32_t it = x / area, r2 = x - it * area, ih = r2 / g.pbw, iw = r2 - ih * g.pbw;
        const int32_t t = t0 + it, h = h0 + ih, w = w0 + iw;
        const bool valid = e < vol * CPR && t < g.frames && h < g.height && w < g.width;
        const size_t orow = ((size_t)t * g.height + h) * g.width + w;
        const size_t brow = (size_t)pb * vol + x;
        from[u] = (TO ? orow : brow) * CPR + c;
        to[u] = (TO ? brow : orow) * CPR + c;
        live[u] = TO ? e < vol * CPR : valid;
        val[u] = valid ? s[from[u]] : make_uint4(0u, 0u, 0u, 0u);
      }
#pragma unroll
      for (int u = 0; u < 4; u++)
        if (live[u]) d[to[u]] = val[u];
    }
  } else {
    const int32_t r0 = ((int32_t)blockIdx.x - n_p) * 64;
    for (int32_t e = threadIdx.x; e < 64 * CPR; e += 256) {
      const int32_t rr = r0 + e / CPR, c = e % CPR;
      if (rr < g.n_text) {
        const size_t orow = (size_t)g.n_video + rr, brow = (size_t)g.n_blk + rr;
        if (TO)
          d[brow * CPR + c] = s[orow * CPR + c];
        else
          d[orow * CPR + c] = s[brow * CPR + c];
      }
    }
  }
}

template <bool TO, int CPR>
static hipError_t launch_layout_t(const void* src, void* dst, int32_t n_bh, const Geometry& g,
                                  hipStream_t stream) {
  const int32_t n_p = g.tp * g.hp * g.wp;
  dim3 grid((unsigned)(n_p + (g.n_text + 63) / 64), (unsigned)n_bh);
  hipLaunchKernelGGL((psa_layout_kernel<TO, CPR>), grid, dim3(256), 0, stream, (const uint4*)src,
                     (uint4*)dst, g);
  return hipGetLastError();
}

hipError_t launch_layout(const void* src, void* dst, int32_t n_bh, int32_t head_dim,
                         const Geometry& g, bool to_blocks, hipStream_t stream) {
  if (head_dim == 128)
    return to_blocks ? launch_layout_t<true, 16>(src, dst, n_bh, g, stream)
                     : launch_layout_t<false, 16>(src, dst, n_bh, g, stream);
  if (head_dim == 64)
    return to_blocks ? launch_layout_t<true, 8>(src, dst, n_bh, g, stream)
                     : launch_layout_t<false, 8>(src, dst, n_bh, g, stream);
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------------------------
// Scheduler pre-pass (psa_attention_fwd).
// ---------------------------------------------------------------------------------------------

WorkspaceLayout workspace_layout(int32_t batch, int32_t n_heads, int32_t nb, bool masks) {
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t items = (size_t)batch * n_heads * nb;
  WorkspaceLayout wl;
  wl.header = 0;
  wl.params = up(wl.header + sizeof(PlanHeader));
  wl.coords = up(wl.params + sizeof(psa_stripe_t) * (size_t)n_heads);
  wl.counts = up(wl.coords + sizeof(int2) * (size_t)nb);
  wl.order = up(wl.counts + sizeof(int32_t) * items);
  wl.queues = up(wl.order + sizeof(int32_t) * items);
  wl.sigs = up(wl.queues + sizeof(int32_t) * kQueueWords);
  wl.pairs = up(wl.sigs + sizeof(uint64_t) * (size_t)n_heads * nb);
  const size_t pair_items = (size_t)batch * n_heads * pairs_per_head(nb);
  wl.spans = up(wl.pairs + sizeof(int2) * (size_t)n_heads * pairs_per_head(nb));
  wl.runspans = up(wl.spans + sizeof(uint32_t) * pair_items);
  wl.starts = up(wl.runspans + sizeof(uint32_t) * pair_items);
  wl.masks = up(wl.starts + sizeof(int32_t) * pair_items);
  wl.total = masks ? up(wl.masks + 2 * sizeof(uint64_t) * (size_t)nb) : wl.masks;
  return wl;
}

// Copies one chunk of stripe parameters into the workspace; the first chunk also invalidates
// the plan header (write_coords != 0) and writes the block coordinate table of one-dimensional
// blocks (write_coords == 1; 3D tiles get theirs from psa_tiles3d_kernel).  write_header: the plan
// has no other kernel after this one.
__global__ __launch_bounds__(256) void psa_setup_kernel(ParamChunk pc, int32_t head0, Geometry g,
                                                        PlanHeader* __restrict__ header,
                                                        psa_stripe_t* __restrict__ params,
                                                        int2* __restrict__ coords,
                                                        int32_t write_coords, PlanHeader done,
                                                        int32_t write_header) {
  const int32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i == 0) {
    if (write_header)
      *header = done;
    else if (write_coords)
      header->magic = 0;
  }
  if (i < pc.n) params[head0 + i] = pc.m[i];
  if (write_coords == 1 && i < g.nb) coords[i] = block_coord(g, i);
}

// One wave per tile of the PSABlock-centric layout: the valid positions of the tile (bit r of
// word r / 64) and its coordinates, kDeadTile when it holds only padding.
__global__ __launch_bounds__(256) void psa_tiles3d_kernel(Geometry g, int2* __restrict__ coords,
                                                          uint64_t* __restrict__ masks) {
  const int32_t b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (b >= g.nb) return;
  const int32_t i0 = b * g.block;
  const uint64_t lo = __builtin_amdgcn_ballot_w64(lane < g.block && position_valid(g, i0 + lane));
  const uint64_t hi = g.block > 64 ? __builtin_amdgcn_ballot_w64(position_valid(g, i0 + 64 + lane))
                                   : ~0ull;
  if (lane == 0) {
    masks[2 * b] = lo;
    masks[2 * b + 1] = hi;
    const bool dead = lo == 0 && (g.block <= 64 || hi == 0);
    coords[b] = dead ? make_int2(kDeadTile, 0) : tile_coord3d(g, b);
  }
}

// A 64-bit mix of a block index (the splitmix64 finalizer); the XOR of the mixes of a kept set
// is a hash of the set that does not depend on the order of its members.
__device__ __forceinline__ uint64_t mix64(uint64_t x) {
  x += 0x9e3779b97f4a7c15ull;
  x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
  x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
  return x ^ (x >> 31);
}

// One wave per (head, query block): the number of kept key blocks (kept_per_row, if asked) and the
// signature of the kept set (sigs, if asked).  With a header, this is the plan's last kernel.
__global__ __launch_bounds__(256) void psa_count_kernel(const psa_stripe_t* __restrict__ params,
                                                        const int2* __restrict__ coords,
                                                        int32_t* __restrict__ kept_per_row,
                                                        uint64_t* __restrict__ sigs, int32_t n_rows,
                                                        int32_t nb, PlanHeader* __restrict__ header,
                                                        PlanHeader done) {
  if (header && blockIdx.x == 0 && threadIdx.x == 0) *header = done;
  const int32_t row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= n_rows) return;
  const int32_t h = row / nb, qb = row - h * nb;
  const psa_stripe_t m = params[h];
  const int2 cq = coords[qb];
  int cnt = 0;
  uint64_t sig = 0;
  for (int32_t kb = lane; kb < nb; kb += 64) {
    const bool keep = tile_keep(m, cq, coords[kb]);
    cnt += keep ? 1 : 0;
    sig ^= keep ? mix64((uint64_t)kb) : 0ull;
  }
  cnt = wave_sum(cnt);
  for (int off = 32; off > 0; off >>= 1) sig ^= __shfl_xor(sig, off);
  if (lane == 0) {
    if (kept_per_row) kept_per_row[row] = cnt;
    if (sigs) sigs[row] = sig;
  }
}

// Exclusive prefix sum (OP = +) or inclusive running maximum (OP = max) over v[0 .. n) in LDS by
// a 1024-thread workgroup; n <= 8 * 1024.  Returns the total (sum) or the last value (max).
template <bool MAX>
__device__ int32_t block_scan(int32_t* v, int32_t n, int32_t* part) {
  constexpr int E = 8;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int32_t loc[E];
  int32_t acc = MAX ? -1 : 0;
#pragma unroll
  for (int e = 0; e < E; e++) {
    const int32_t i = tid * E + e;
    const int32_t x = i < n ? v[i] : (MAX ? -1 : 0);
    loc[e] = acc;                                         // exclusive within the thread
    acc = MAX ? max(acc, x) : acc + x;
  }
  int32_t incl = acc;                                     // inclusive over the wave
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t t = __shfl_up(incl, off);
    if (lane >= off) incl = MAX ? max(incl, t) : incl + t;
  }
  if (lane == 63) part[wave] = incl;
  __syncthreads();
  int32_t before = MAX ? -1 : 0;                          // over the waves before this one
  for (int w = 0; w < wave; w++) before = MAX ? max(before, part[w]) : before + part[w];
  int32_t total = MAX ? -1 : 0;
  for (int w = 0; w < 16; w++) total = MAX ? max(total, part[w]) : total + part[w];
  const int32_t lane_excl = __shfl_up(incl, 1);
  const int32_t prior = lane == 0 ? before : (MAX ? max(before, lane_excl) : before + lane_excl);
#pragma unroll
  for (int e = 0; e < E; e++) {
    const int32_t i = tid * E + e;
    if (i < n) {
      if (MAX)
        v[i] = max(prior, max(loc[e], v[i]));             // inclusive running maximum
      else
        v[i] = prior + loc[e];
    }
  }
  __syncthreads();
  return total;
}

// One workgroup per head: pairs of query blocks for the pair engine.  The rows are sorted by the
// signature of their kept set (then by index); within a run of equal signatures consecutive
// rows pair up.  The rows left over pair up consecutively in one of two orders, chosen from the
// head's stripes: index order (neighbouring slots of one frame), or slot-major (one slot in
// neighbouring frames) where a one-frame shift widens the kept set less than a one-slot shift.
// A shift by one position grows an axis' kept set by (w + 1) / w for a stripe narrower than its
// stride and leaves a full axis unchanged, so slot-major is taken when the spatial stripes are
// partial and the temporal ones either cover their axis or are wider (T_w > S_w).
// pairs[h][p] = (first row, second row or -1), in the order of the first rows.  Rows with
// equal kept sets share every key block, so most pairs of the stripe patterns waste no work;
// the pairing only affects speed, the run decodes each row's own kept set.
constexpr int kPairSort = 8192;                 // a power of two >= PSA_MAX_BLOCKS
__global__ __launch_bounds__(1024) void psa_pairing_kernel(const uint64_t* __restrict__ sigs,
                                                           const psa_stripe_t* __restrict__ params,
                                                           const int2* __restrict__ coords,
                                                           int2* __restrict__ pairs, int32_t nb) {
  __shared__ uint64_t key[kPairSort];         // sorted (signature, row); later leftover rows
  __shared__ int32_t run[kPairSort];          // start of each sorted position's run
  __shared__ int16_t partner[kPairSort];      // by row: partner (first row), -1 single, -2 second
  __shared__ int32_t part[16];
  const int tid = threadIdx.x, lane = tid & 63;
  const uint64_t* sg = sigs + (size_t)blockIdx.x * nb;
  int32_t n2 = 1;
  while (n2 < nb) n2 <<= 1;
  for (int32_t i = tid; i < n2; i += 1024) {
    key[i] = i < nb ? ((sg[i] >> 13) << 13) | (uint64_t)i : ~0ull;
    partner[i] = -3;
  }
  __syncthreads();
  // Bitonic sort of key[0 .. n2), ascending.  Partners 64 or more apart meet in LDS (one
  // barrier per step); the steps of a stage with partners less than 64 apart run inside each
  // wave, on registers exchanged across lanes, with one barrier for all of them.
  auto sort_keys = [&]() {
    for (int32_t k = 2; k <= n2; k <<= 1) {
      int32_t j = k >> 1;
      for (; j >= 64; j >>= 1) {
        for (int32_t i = tid; i < n2; i += 1024) {
          const int32_t ixj = i ^ j;
          if (ixj > i) {
            const uint64_t a = key[i], b = key[ixj];
            if ((a > b) == ((i & k) == 0)) {
              key[i] = b;
              key[ixj] = a;
            }
          }
        }
        __syncthreads();
      }
      for (int32_t i = tid; i < n2; i += 1024) {        // n2 < 64, or whole waves
        uint64_t x = key[i];
        const bool up = (i & k) == 0;
        auto step = [&](auto m) {
          constexpr int M = decltype(m)::value;
          if (M > j) return;
          const uint64_t y = ((uint64_t)(uint32_t)lane_xor<M>((int32_t)(x >> 32), lane) << 32) |
                             (uint32_t)lane_xor<M>((int32_t)(uint32_t)x, lane);
          x = (((i & M) == 0) == up) ? min(x, y) : max(x, y);
        };
        step(std::integral_constant<int, 32>());
        step(std::integral_constant<int, 16>());
        step(std::integral_constant<int, 8>());
        step(std::integral_constant<int, 4>());
        step(std::integral_constant<int, 2>());
        step(std::integral_constant<int, 1>());
        key[i] = x;
      }
      __syncthreads();
    }
  };
  sort_keys();
  auto row_of = [&](int32_t i) { return (int32_t)(key[i] & 8191u); };
  auto same = [&](int32_t i, int32_t j) { return (key[i] >> 13) == (key[j] >> 13); };
  for (int32_t i = tid; i < nb; i += 1024) run[i] = (i == 0 || !same(i, i - 1)) ? i : -1;
  __syncthreads();
  block_scan<true>(run, nb, part);
  for (int32_t i = tid; i < nb; i += 1024) {
    if (((i - run[i]) & 1) != 0) continue;
    const int32_t r = row_of(i);
    if (i + 1 < nb && run[i + 1] == run[i]) {
      const int32_t r2 = row_of(i + 1);
      partner[min(r, r2)] = (int16_t)max(r, r2);
      partner[max(r, r2)] = -2;
    } else {
      partner[r] = -4;                                  // left over
    }
  }
  __syncthreads();
  // Leftover rows: rank in the chosen order (a prefix sum over the rows gives index order), pair
  // ranks 2k and 2k + 1.
  const psa_stripe_t m = params[blockIdx.x];
  const bool slot_major = m.s_w < m.s_s && (m.t_w >= m.t_s || m.t_w > m.s_w);
  for (int32_t i = tid; i < nb; i += 1024) run[i] = partner[i] == -4 ? 1 : 0;
  __syncthreads();
  const int32_t n_left = block_scan<false>(run, nb, part);
  uint32_t* left = (uint32_t*)key;                        // rank -> row
  if (!slot_major) {
    for (int32_t i = tid; i < nb; i += 1024)
      if (partner[i] == -4) left[run[i]] = (uint32_t)i;
  } else {
    // Sort the leftover rows by (slot, frame, row); other rows sort last.  Coordinates beyond
    // the fields (global and padding blocks have negative frames) are clamped: any order is a
    // valid pairing.
    for (int32_t i = tid; i < n2; i += 1024) {
      uint64_t kk = ~0ull;
      if (i < nb && partner[i] == -4) {
        const int2 c = coords[i];
        kk = ((uint64_t)min((uint32_t)c.y, (1u << 26) - 1) << 38) |
             ((uint64_t)min((uint32_t)c.x, (1u << 25) - 1) << 13) | (uint64_t)i;
      }
      key[i] = kk;
    }
    __syncthreads();
    sort_keys();
    // left[] overlays key[]: every thread reads its sorted rows before any is written.
    uint32_t rows[kPairSort / 1024];
#pragma unroll
    for (int j = 0; j < kPairSort / 1024; j++) {
      const int32_t r = tid + 1024 * j;
      rows[j] = r < n_left ? (uint32_t)(key[r] & 8191u) : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPairSort / 1024; j++) {
      const int32_t r = tid + 1024 * j;
      if (r < n_left) left[r] = rows[j];
    }
    __syncthreads();
    for (int32_t r = tid; r < n_left; r += 1024) run[left[r]] = r;
  }
  __syncthreads();
  for (int32_t i = tid; i < nb; i += 1024)
    if (partner[i] == -4) {
      const int32_t r = run[i];
      partner[i] = (r & 1) ? -2 : (r + 1 < n_left ? (int16_t)left[r + 1] : -1);
    }
  __syncthreads();
  // Pairs in the order of their first rows.
  for (int32_t i = tid; i < nb; i += 1024) run[i] = partner[i] >= -1 ? 1 : 0;
  __syncthreads();
  block_scan<false>(run, nb, part);
  int2* dst = pairs + (size_t)blockIdx.x * pairs_per_head(nb);
  for (int32_t i = tid; i < nb; i += 1024)
    if (partner[i] >= -1 && run[i] < pairs_per_head(nb)) dst[run[i]] = make_int2(i, partner[i]);
}

// Setup, counts, signatures, pairs and pair counts of one head in one workgroup, for sequences of at
// most kHeadPlanRows blocks (one-dimensional ones, or PSABlock tiles whose coordinates the workspace
// already holds).  The same pairs as the kernels above, found by comparing every row with every
// other -- at this size less work than the barriers of a sort.  What bounds the plan of a short
// sequence is the number of its kernels, 2 to 4 us and more each: 12 heads x 61 blocks took 23 us
// in four kernels (setup, counts, pairing, pair counts), 11 us in this one.  The work of its one
// workgroup grows with the square of the rows, though: at 256 blocks it takes 50 us, the four
// kernels 28, so the line is at 128.
constexpr int kHeadPlanRows = 128;
__global__ __launch_bounds__(1024) void psa_head_plan_kernel(
    ParamChunk pc, int32_t head0, Geometry g, int32_t batch, int32_t n_heads,
    PlanHeader* __restrict__ header, psa_stripe_t* __restrict__ params, int2* __restrict__ coords,
    int2* __restrict__ pairs, int32_t* __restrict__ counts, int32_t* __restrict__ kept_per_row) {
  constexpr int K = kHeadPlanRows / 64;         // blocks per lane
  constexpr int kTable = 512;                   // axis extents with a table of the distances' tests
  __shared__ int2 c_of[kHeadPlanRows];
  __shared__ uint4 sig4[kHeadPlanRows / 4];     // signatures, compared four at a time
  __shared__ uint64_t key[kHeadPlanRows];       // of the leftover rows, ~0 for the others
  __shared__ int32_t by_rank[kHeadPlanRows];    // leftover rows in their order
  __shared__ int2 list[kHeadPlanRows];          // the pairs in the order of their first rows
  __shared__ uint8_t t_keep[2 * kTable], s_keep[2 * kTable];
  __shared__ int32_t firsts[K];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  uint32_t* const sig = (uint32_t*)sig4;
  const int32_t nb = g.nb, np = pairs_per_head(nb), h = head0 + (int32_t)blockIdx.x;
  const psa_stripe_t m = pc.m[blockIdx.x];
  const AxisTest ta(m.t_w, m.t_o, m.t_s), sa(m.s_w, m.s_o, m.s_s);
  const int32_t t_ext = g.pbt > 0 ? g.tp : g.frames;
  const int32_t s_ext = g.pbt > 0 ? g.hp * g.wp : (g.hw - 1) / g.block + 1;
  const bool table = t_ext <= kTable && s_ext <= kTable;
  auto keeps = [&](int2 q, int2 k) {
    if (q.x == kDeadTile || k.x == kDeadTile) return false;
    if (q.x < 0 || k.x < 0) return true;
    if (table) return (t_keep[k.x - q.x + t_ext - 1] & s_keep[k.y - q.y + s_ext - 1]) != 0;
    return ta.keep(k.x - q.x) && sa.keep(k.y - q.y);
  };
  if (tid == 0) {
    params[h] = m;
    if (h == 0) header->magic = 0;
  }
  if (tid < kHeadPlanRows) {
    int2 c = make_int2(kDeadTile, 0);
    if (tid < nb) {
      c = g.pbt > 0 ? coords[tid] : block_coord(g, tid);
      if (h == 0 && g.pbt == 0) coords[tid] = c;
    }
    c_of[tid] = c;
    sig[tid] = 0;
  }
  if (table) {
    if (tid < 2 * t_ext - 1) t_keep[tid] = ta.keep(tid - (t_ext - 1));
    if (tid < 2 * s_ext - 1) s_keep[tid] = sa.keep(tid - (s_ext - 1));
  }
  __syncthreads();
  int2 ck[K];
  uint32_t mix[K];
#pragma unroll
  for (int i = 0; i < K; i++) {
    ck[i] = c_of[lane + 64 * i];
    mix[i] = (uint32_t)mix64((uint64_t)(lane + 64 * i));
  }
  // Counts and signatures (32 bits of the mix do: a collision costs speed only), a wave per row.
  for (int32_t q = wave; q < nb; q += 16) {
    const int2 cq = c_of[q];
    int32_t cnt = 0;
    uint32_t x = 0;
#pragma unroll
    for (int i = 0; i < K; i++) {
      if (64 * i >= nb) break;
      const bool keep = keeps(cq, ck[i]);
      cnt += __builtin_popcountll(__builtin_amdgcn_ballot_w64(keep));
      x ^= keep ? mix[i] : 0u;
    }
    for (int off = 32; off > 0; off >>= 1) x ^= __shfl_xor(x, off);
    if (lane == 0) {
      sig[q] = x;
      if (kept_per_row) kept_per_row[(int64_t)h * nb + q] = cnt;
    }
  }
  __syncthreads();
  // Rows of equal sets pair up in the order of their indices; the last of an odd run is left over.
  int32_t next = nb;                            // the row this one is the first of a pair with
  bool first = false, left = false;
  if (tid < nb) {
    const uint32_t mine = sig[tid];
    int32_t before = 0;
    for (int32_t j = 0; j < nb; j += 4) {       // (rows past the end come after every real one)
      const uint4 o = sig4[j / 4];
      const uint32_t os[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
      for (int u = 0; u < 4; u++) {
        const bool same = os[u] == mine;
        before += same && j + u < tid ? 1 : 0;
        next = min(next, same && j + u > tid ? j + u : nb);
      }
    }
    first = !(before & 1);
    left = first && next == nb;
    // Order of the leftover rows: see psa_pairing_kernel.
    const bool slot_major = m.s_w < m.s_s && (m.t_w >= m.t_s || m.t_w > m.s_w);
    const int2 c = c_of[tid];
    uint64_t kk = (uint64_t)tid;
    if (slot_major)
      kk |= ((uint64_t)min((uint32_t)c.y, (1u << 26) - 1) << 38) |
            ((uint64_t)min((uint32_t)c.x, (1u << 25) - 1) << 13);
    key[tid] = left ? kk : ~0ull;
    by_rank[tid] = -1;
  }
  __syncthreads();
  int32_t rank = 0;
  if (left) {
    const uint64_t mine = key[tid];
    for (int32_t j = 0; j < nb; j++) rank += key[j] < mine ? 1 : 0;
    by_rank[rank] = tid;
    first = !(rank & 1);
  }
  const uint64_t starts = __builtin_amdgcn_ballot_w64(first);
  if (lane == 0 && wave < K) firsts[wave] = __builtin_popcountll(starts);
  __syncthreads();
  if (first) {
    if (left) next = rank + 1 < nb ? by_rank[rank + 1] : -1;
    int32_t at = __builtin_popcountll(starts & ((1ull << lane) - 1));
    for (int w = 0; w < wave; w++) at += firsts[w];
    if (at < np) {
      list[at] = make_int2(tid, next);
      pairs[(int64_t)h * np + at] = make_int2(tid, next);
    }
  }
  __syncthreads();
  // Work of the pairs, a wave per pair.
  for (int32_t p = wave; p < np; p += 16) {
    const int2 pr = list[p];
    const int2 ca = c_of[pr.x], cb = pr.y >= 0 ? c_of[pr.y] : make_int2(kDeadTile, 0);
    int32_t cnt = 0;
#pragma unroll
    for (int i = 0; i < K; i++) {
      if (64 * i >= nb) break;
      cnt += __builtin_popcountll(__builtin_amdgcn_ballot_w64(keeps(ca, ck[i]) || keeps(cb, ck[i])));
    }
    for (int32_t b = lane; b < batch; b += 64) counts[((int64_t)b * n_heads + h) * np + p] = cnt;
  }
}

// One wave per pair item (batch, head, pair): number of key blocks kept by either row, and the
// first and last of them that are not global (video blocks; the span the start of the item's
// stream is placed in).
__global__ __launch_bounds__(256) void psa_paircount_kernel(const psa_stripe_t* __restrict__ params,
                                                            const int2* __restrict__ coords,
                                                            const int2* __restrict__ pairs,
                                                            int32_t* __restrict__ counts,
                                                            uint32_t* __restrict__ spans,
                                                            int32_t n_items, int32_t n_heads,
                                                            int32_t nb) {
  const int32_t np = pairs_per_head(nb);
  const int32_t item = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (item >= n_items) return;
  const int32_t bh = item / np, p = item - bh * np, h = bh % n_heads;
  const psa_stripe_t m = params[h];
  const int2 pr = pairs[(int64_t)h * np + p];
  const int2 ca = coords[pr.x];
  const int2 cb = pr.y >= 0 ? coords[pr.y] : make_int2(kDeadTile, 0);
  int cnt = 0, lo = nb, hi = -1;
  for (int32_t kb = lane; kb < nb; kb += 64) {
    const int2 ck = coords[kb];
    const bool keep = tile_keep(m, ca, ck) || tile_keep(m, cb, ck);
    cnt += keep ? 1 : 0;
    if (keep && ck.x >= 0) {
      lo = min(lo, kb);
      hi = max(hi, kb);
    }
  }
  cnt = wave_sum(cnt);
  for (int off = 32; off > 0; off >>= 1) {
    lo = min(lo, __shfl_xor(lo, off));
    hi = max(hi, __shfl_xor(hi, off));
  }
  if (lane == 0) {
    counts[item] = cnt;
    spans[item] = hi < 0 ? 0xffffffffu : ((uint32_t)lo | ((uint32_t)hi << 16));
  }
}

// Work estimate of an item, in tiles: kept key blocks plus a fixed cost for loading Q,
// decoding the list and the epilogue.
constexpr int kItemOverhead = 2;

// An item whose work exceeds kLongFactor times the mean item work is scheduled ahead of all
// others (for example the rows of the global text tokens, which keep every key block): taken
// late, one such item would still run long after the rest of the device has drained.
constexpr int kLongFactor = 3;
// Long items are sorted into this many classes of equal width in [0, max work].
constexpr int kWorkClasses = 64;
constexpr int kScheduleWaves = 16;

// The schedule of a short list: every queue takes a
// contiguous range of equal work of every (batch, head), as in the schedule below, but lists its
// items longest first (in kRankClasses classes, by index within one; with 32, 8 and 4 classes the
// Wan 2.1 1.3B layer takes 1, 2 and 4 % longer).  With few items per workgroup
// the last ones to be taken set the time: a makespan model of the drawn shapes puts the order by
// heads at 1.2 to 2 x the ideal with one to three items per workgroup and 1.05 to 1.15 x at six,
// longest first at 1.1 to 1.45 x and 1.01 to 1.05 x.  Measured: 3 heads of 41774 tokens (1.9 items
// per workgroup) 1333 -> 982 us, 10 heads of 28875 (4.4) 2204 -> 1910 us; at 12 items per workgroup
// and more the order by heads is 1 to 4 % faster, because the workgroups of an XCD then read the
// same key blocks at about the same time.
// With `whole`, heads of a few items go to one queue whole, ranked by their mean work: the items of a
// head then run one after the other on one XCD, whose L2 serves K and V once.  Spread over the queues
// they are read by several XCDs at different times, which cost lists of more than three items per CU
// up to 8 % (256 heads x 1024 tokens of head dim 128 77.8 us, whole 71.8, in the order by heads 71.4;
// block 64, 512 x 512 72 and 65, head dim 64 1024 x 512 95 and 86).  Shorter lists and fewer heads than
// CUs are a matter of balance, where whole heads lose 1 to 4 %.
// One workgroup; a wave owns a contiguous slice of the items, 64 cw of them, 64 at a time.
constexpr int kRankItems = 16384;
constexpr int kRankClasses = 64;
constexpr int kWholeHead = 5;             // items of a head that goes whole ...
constexpr int kWholeItems = 768;          // ... in a list of more than this many items
constexpr int kWholeHeads = 256;          // ... of at least this many heads
__global__ __launch_bounds__(1024) void psa_rank_kernel(const int32_t* __restrict__ counts,
                                                        int32_t* __restrict__ order,
                                                        int32_t* __restrict__ queues,
                                                        int32_t* __restrict__ starts,
                                                        PlanHeader* __restrict__ header,
                                                        PlanHeader done, int32_t per_head,
                                                        int32_t whole) {
  constexpr int C = kRankItems / 1024, kBins = kNumQueues * kRankClasses;
  static_assert(kBins <= 1024, "a thread per bin");
  __shared__ int32_t hist[16][kBins];
  __shared__ int32_t head_at[PSA_MAX_BATCH_HEADS + 1];    // work before each (batch, head)
  __shared__ int32_t part[16], part_max[16], bin_part[16];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int32_t n = done.n_bh * per_head, cw = (n + 1023) / 1024;
  for (int32_t i = tid; i < 16 * kBins; i += 1024) (&hist[0][0])[i] = 0;
  int32_t cnt[C], at[C], bh[C], sum = 0, mx = 0;
#pragma unroll
  for (int c = 0; c < C; c++) {
    if (c >= cw) continue;
    const int32_t i = 64 * (cw * wave + c) + lane;
    cnt[c] = i < n ? counts[i] : -kItemOverhead;
    bh[c] = i / per_head;
  }
#pragma unroll
  for (int c = 0; c < C; c++) {
    if (c >= cw) continue;
    const int32_t w = cnt[c] + kItemOverhead;
    const int32_t incl = wave_incl_sum(w, lane);
    at[c] = sum + incl - w;                               // work before the item within the wave
    sum += __builtin_amdgcn_readlane(incl, 63);
    mx = max(mx, cnt[c]);
  }
  mx = wave_reduce<2>(mx);
  if (lane == 0) {
    part[wave] = sum;
    part_max[wave] = mx;
  }
  __syncthreads();
  int32_t before = 0, total = 0;
  for (int w = 0; w < 16; w++) {
    before += w < wave ? part[w] : 0;
    total += part[w];
    mx = max(mx, part_max[w]);
  }
#pragma unroll
  for (int c = 0; c < C; c++) {
    if (c >= cw) continue;
    const int32_t i = 64 * (cw * wave + c) + lane;
    at[c] += before;
    if (i < n && i == bh[c] * per_head) head_at[bh[c]] = at[c];
  }
  if (tid == 0) head_at[done.n_bh] = total;
  __syncthreads();
  int32_t bin[C];
#pragma unroll
  for (int c = 0; c < C; c++) {
    if (c >= cw) continue;
    const int32_t i = 64 * (cw * wave + c) + lane;
    bin[c] = 0;
    if (i < n) {
      // The (batch, head)s start on different queues: one of fewer than kNumQueues items does not
      // fill them all.
      const uint32_t h0 = head_at[bh[c]], head = head_at[bh[c] + 1] - h0;
      const uint32_t range = whole ? 0 : (uint32_t)(((uint64_t)(at[c] - h0) * kNumQueues) / head);
      const uint32_t len = whole ? head / per_head - kItemOverhead : (uint32_t)cnt[c];
      const int32_t cls = (int32_t)(len * kRankClasses / (uint32_t)(mx + 1));
      bin[c] = (int32_t)((range + bh[c]) % kNumQueues) * kRankClasses + kRankClasses - 1 - cls;
      atomicAdd(&hist[wave][bin[c]], 1);
    }
  }
  __syncthreads();
  // Positions: an exclusive sum over (bin, wave).
  int32_t col = 0, incl = 0;
  if (tid < kBins) {
    for (int w = 0; w < 16; w++) col += hist[w][tid];
    incl = wave_incl_sum(col, lane);
    if (lane == 63) bin_part[wave] = incl;
  }
  __syncthreads();
  if (tid < kBins) {
    int32_t pos = incl - col;
    for (int w = 0; w < wave; w++) pos += bin_part[w];
    if (tid % kRankClasses == 0) queues[tid / kRankClasses] = pos;
    if (tid == 0) queues[kNumQueues] = n;
    for (int w = 0; w < 16; w++) {
      const int32_t x = hist[w][tid];
      hist[w][tid] = pos;
      pos += x;
    }
  }
  if (tid < kNumQueues) queues[kQueueCounters + tid * kCounterStride] = 0;
  __syncthreads();
  // Stable scatter: the lanes of 64 items that share a bin are found with one ballot per bit.
#pragma unroll
  for (int c = 0; c < C; c++) {
    if (c >= cw) continue;
    const int32_t i = 64 * (cw * wave + c) + lane;
    const bool valid = i < n;
    uint64_t same = __builtin_amdgcn_ballot_w64(valid);
    if (!same) break;
#pragma unroll
    for (int bit = 1; bit < kBins; bit <<= 1) {
      const uint64_t ones = __builtin_amdgcn_ballot_w64(valid && (bin[c] & bit));
      same &= (bin[c] & bit) ? ones : ~ones;
    }
    const int32_t base = valid ? hist[wave][bin[c]] : 0;
    __builtin_amdgcn_wave_barrier();
    if (valid) {
      order[base + __builtin_popcountll(same & ((1ull << lane) - 1))] = i;
      if (starts) starts[i] = 0;                          // streams ascend from their first block
      if (__builtin_ctzll(same) == lane) hist[wave][bin[c]] = base + __builtin_popcountll(same);
    }
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  if (tid == 0) {
    queues[kHalvesWord] = halves_pay(total - kItemOverhead * n, mx, n);
    __threadfence();
    *header = done;
  }
}

// Single workgroup.  Every queue x (the XCD of the workgroups that start on it) begins with its
// share of the long items, longest first and dealt round-robin over the queues.  The other items
// follow head by head: the (batch, head) pairs are ordered by their work, longest first, and
// every head's query blocks are cut into kNumQueues contiguous ranges of equal work, queue x
// listing range x of every head.  All XCDs therefore sweep the heads together -- the K/V of the
// one or two heads in flight stay in the memory-side cache -- and the workgroups of one XCD
// stream neighbouring key blocks through its L2.
__global__ __launch_bounds__(1024) void psa_schedule_kernel(const int32_t* __restrict__ counts,
                                                            int32_t* __restrict__ order,
                                                            int32_t* __restrict__ queues,
                                                            PlanHeader* __restrict__ header,
                                                            PlanHeader done, int32_t nb,
                                                            int32_t write_header,
                                                            const uint32_t* __restrict__ spans,
                                                            uint32_t* __restrict__ runspans) {
  const int32_t n_bh = done.n_bh, n = n_bh * nb;
  __shared__ int64_t total[PSA_MAX_BATCH_HEADS];
  __shared__ int32_t by_rank[PSA_MAX_BATCH_HEADS];
  __shared__ uint16_t bounds[PSA_MAX_BATCH_HEADS][kNumQueues + 1];
  __shared__ int32_t qoff[PSA_MAX_BATCH_HEADS][kNumQueues];
  __shared__ int32_t hist[kScheduleWaves][kWorkClasses];
  __shared__ int32_t qstart[kNumQueues + 1];
  __shared__ uint64_t all_work;
  __shared__ int32_t max_count, n_long;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;

  if (tid == 0) {
    all_work = 0;
    max_count = 0;
  }
  for (int32_t i = tid; i < kScheduleWaves * kWorkClasses; i += 1024) (&hist[0][0])[i] = 0;
  __syncthreads();
  constexpr int kLoads = 4;                 // loads in flight per lane in the sweeps below
  // Sums of one pair's work stay below 2^31: at most PSA_MAX_BLOCKS items of at most
  // PSA_MAX_BLOCKS + kItemOverhead tiles.
  for (int32_t bh = wave; bh < n_bh; bh += kScheduleWaves) {
    int32_t s = 0;
    int32_t mx = 0;
    for (int32_t q0 = lane; q0 < nb; q0 += 64 * kLoads) {
      int32_t c[kLoads];
#pragma unroll
      for (int j = 0; j < kLoads; j++) c[j] = q0 + 64 * j < nb ? counts[bh * nb + q0 + 64 * j] : -1;
#pragma unroll
      for (int j = 0; j < kLoads; j++) {
        s += c[j] < 0 ? 0 : c[j] + kItemOverhead;
        mx = max(mx, c[j]);
      }
    }
    s = wave_reduce<0>(s);
    mx = wave_reduce<2>(mx);
    if (lane == 0) {
      total[bh] = s;
      atomicAdd(&all_work, (uint64_t)s);
      atomicMax(&max_count, mx);
    }
  }
  __syncthreads();
  const int64_t long_above = (int64_t)kLongFactor * (int64_t)all_work;
  auto work_of = [&](int32_t item) { return (int64_t)counts[item] + kItemOverhead; };
  // Whether any item is long follows from the largest one; without long items every pass that
  // looks for them is skipped.
  const bool any_long = ((int64_t)max_count + kItemOverhead) * n > long_above;
  auto is_long = [&](int32_t item) { return any_long && work_of(item) * n > long_above; };
  if (any_long) {
    // Work of each pair without its long items.
    for (int32_t bh = wave; bh < n_bh; bh += kScheduleWaves) {
      int32_t s = 0;
      for (int32_t q0 = lane; q0 < nb; q0 += 64 * kLoads) {
        int64_t w[kLoads];
#pragma unroll
        for (int j = 0; j < kLoads; j++) w[j] = q0 + 64 * j < nb ? work_of(bh * nb + q0 + 64 * j) : 0;
#pragma unroll
        for (int j = 0; j < kLoads; j++) s += w[j] * n > long_above ? 0 : (int32_t)w[j];
      }
      s = wave_reduce<0>(s);
      if (lane == 0) total[bh] = s;
    }
    __syncthreads();
  }
  for (int32_t bh = tid; bh < n_bh; bh += 1024) {
    int32_t r = 0;
    const int64_t mine = total[bh];
    for (int32_t j = 0; j < n_bh; j++) r += (total[j] > mine || (total[j] == mine && j < bh)) ? 1 : 0;
    by_rank[r] = bh;
  }
  __syncthreads();

  // Equal-work ranges of each head over its other items: bounds[r][x] = first query block of
  // range x.
  for (int32_t r = wave; r < n_bh; r += kScheduleWaves) {
    const int32_t bh = by_rank[r];
    const int64_t head_total = total[bh];
    int32_t base = 0;
    int32_t next = 1;                       // next boundary to place
    if (lane == 0) bounds[r][0] = 0;
    for (int32_t g0 = 0; g0 < nb && next < kNumQueues; g0 += 64 * kLoads) {
      int32_t wv[kLoads];
#pragma unroll
      for (int j = 0; j < kLoads; j++) {
        const int32_t qb = g0 + 64 * j + lane;
        wv[j] = qb < nb && !is_long(bh * nb + qb) ? (int32_t)work_of(bh * nb + qb) : 0;
      }
#pragma unroll
      for (int j = 0; j < kLoads; j++) {
        const int32_t q0 = g0 + 64 * j, qb = q0 + lane;
        const int32_t w = wv[j];
        const int32_t incl = wave_incl_sum(w, lane);        // inclusive prefix over the wave
        const int64_t excl = base + incl - w;
        // range x starts at the first block whose preceding work reaches x/Q of the head
        while (next < kNumQueues) {
          const int64_t target = head_total * next / kNumQueues;
          const uint64_t hit = __builtin_amdgcn_ballot_w64(qb < nb && excl >= target);
          if (!hit) break;
          const int32_t first = q0 + __builtin_ctzll(hit);
          if (lane == 0) bounds[r][next] = (uint16_t)first;
          next++;
        }
        base += __builtin_amdgcn_readlane(incl, 63);
      }
    }
    for (; next < kNumQueues; next++)
      if (lane == 0) bounds[r][next] = (uint16_t)nb;
    if (lane == 0) bounds[r][kNumQueues] = (uint16_t)nb;
  }

  // Long items: stable class sort.  Entry s of the unsorted list is query block s mod nb of the
  // pair of rank s div nb; wave w owns the slice [w n / W, (w + 1) n / W).  Class 0 holds the
  // longest items.
  const int32_t lo = (int32_t)((int64_t)n * wave / kScheduleWaves);
  const int32_t hi = (int32_t)((int64_t)n * (wave + 1) / kScheduleWaves);
  const int32_t top = max_count + 1;
  auto item_of = [&](int32_t s) { const int32_t r = s / nb; return by_rank[r] * nb + (s - r * nb); };
  auto class_of = [&](int32_t item) {
    return kWorkClasses - 1 - (int32_t)((int64_t)counts[item] * kWorkClasses / top);
  };
  if (any_long)
    for (int32_t s = lo + lane; s < hi; s += 64) {
      const int32_t item = item_of(s);
      if (is_long(item)) atomicAdd(&hist[wave][class_of(item)], 1);
    }
  __syncthreads();

  // Number of the other items in every (head, queue) range, one wave per range.
  for (int32_t pair = wave; pair < n_bh * kNumQueues; pair += kScheduleWaves) {
    const int32_t r = pair / kNumQueues, x = pair - r * kNumQueues;
    const int32_t item0 = by_rank[r] * nb, end = bounds[r][x + 1];
    int32_t c = end - bounds[r][x];
    if (any_long)
      for (int32_t qb = bounds[r][x] + lane; __builtin_amdgcn_readfirstlane(qb - lane) < end; qb += 64)
        c -= __builtin_popcountll(__builtin_amdgcn_ballot_w64(qb < end && is_long(item0 + qb)));
    if (lane == 0) qoff[r][x] = c;
  }
  // Exclusive scan of the class histogram in (class, wave) order: hist[w][c] becomes the first
  // list position of the class-c long items of slice w.
  if (wave == 0) {
    int32_t col = 0;
    for (int w = 0; w < kScheduleWaves; w++) col += hist[w][lane];
    int32_t incl = col;
    for (int off = 1; off < 64; off <<= 1) {
      const int32_t t = __shfl_up(incl, off);
      if (lane >= off) incl += t;
    }
    int32_t pos = incl - col;
    for (int w = 0; w < kScheduleWaves; w++) {
      const int32_t h = hist[w][lane];
      hist[w][lane] = pos;
      pos += h;
    }
    if (lane == 63) n_long = incl;
  }
  __syncthreads();
  // Offsets of each head's range inside its queue, and the queue starts: queue x holds long
  // list positions x, x + Q, ... (n_long div Q of them, one more for x < n_long mod Q), then
  // its ranges.
  if (tid < kNumQueues) {
    int32_t acc = n_long / kNumQueues + (tid < n_long % kNumQueues ? 1 : 0);
    for (int32_t r = 0; r < n_bh; r++) {
      const int32_t c = qoff[r][tid];
      qoff[r][tid] = acc;
      acc += c;
    }
    qstart[tid + 1] = acc;                  // length, turned into a start below
  }
  __syncthreads();
  if (tid == 0) {
    qstart[0] = 0;
    for (int x = 0; x < kNumQueues; x++) qstart[x + 1] += qstart[x];
  }
  __syncthreads();

  // Stable scatter of the long items: the lanes of one 64-entry chunk that share a class are
  // found with one ballot per class bit; each takes the next position of its class in the order
  // of its lane.
  for (int32_t s0 = lo; any_long && s0 < hi; s0 += 64) {
    const int32_t s = s0 + lane;
    const int32_t item = s < hi ? item_of(s) : 0;
    const bool valid = s < hi && is_long(item);
    if (!__builtin_amdgcn_ballot_w64(valid)) continue;
    const int32_t cls = valid ? class_of(item) : 0;
    uint64_t same = __builtin_amdgcn_ballot_w64(valid);
    for (int bit = 1; bit < kWorkClasses; bit <<= 1) {
      const uint64_t ones = __builtin_amdgcn_ballot_w64(valid && (cls & bit));
      same &= (cls & bit) ? ones : ~ones;
    }
    const int32_t base = valid ? hist[wave][cls] : 0;
    __builtin_amdgcn_wave_barrier();
    if (valid) {
      const int32_t pos = base + __builtin_popcountll(same & ((1ull << lane) - 1));
      order[qstart[pos % kNumQueues] + pos / kNumQueues] = item;
      if (runspans) runspans[item] = spans[item];        // a long item is a run of its own
      if (__builtin_ctzll(same) == lane) hist[wave][cls] = base + __builtin_popcountll(same);
    }
    __builtin_amdgcn_wave_barrier();
  }
  // Each wave takes ranges W, W + 16, ...; the count and span of the first 64 items of the next
  // range are loaded while the current one is written.
  const int32_t n_ranges = n_bh * kNumQueues;
  auto head_of = [&](int32_t range, int32_t& cnt, uint32_t& span) {
    cnt = 0;
    span = 0xffffffffu;
    if (range >= n_ranges) return;
    const int32_t r = range / kNumQueues, x = range - r * kNumQueues;
    const int32_t qb = bounds[r][x] + lane;
    if (qb >= bounds[r][x + 1]) return;
    if (any_long) cnt = counts[by_rank[r] * nb + qb];
    if (runspans) span = spans[by_rank[r] * nb + qb];
  };
  int32_t next_cnt;
  uint32_t next_span;
  head_of(wave, next_cnt, next_span);
  for (int32_t range = wave; range < n_ranges; range += kScheduleWaves) {
    const int32_t head_cnt = next_cnt;
    const uint32_t head_span = next_span;
    head_of(range + kScheduleWaves, next_cnt, next_span);
    const int32_t r = range / kNumQueues, x = range - r * kNumQueues;
    const int32_t item0 = by_rank[r] * nb, begin = bounds[r][x], end = bounds[r][x + 1];
    int32_t* dst = order + qstart[x] + qoff[r][x];
    int32_t lo = 0xffff, hi = 0;
    bool head_keep = false;
    for (int32_t qb = begin + lane; __builtin_amdgcn_readfirstlane(qb - lane) < end; qb += 64) {
      const bool head = qb - lane == begin;
      const int32_t cnt = head ? head_cnt : (any_long && qb < end ? counts[item0 + qb] : 0);
      const uint32_t span = head ? head_span : (runspans && qb < end ? spans[item0 + qb] : 0xffffffffu);
      const bool keep = qb < end && !(any_long && ((int64_t)cnt + kItemOverhead) * n > long_above);
      if (head) head_keep = keep;
      const uint64_t mask = __builtin_amdgcn_ballot_w64(keep);
      if (keep) dst[__builtin_popcountll(mask & ((1ull << lane) - 1))] = item0 + qb;
      dst += __builtin_popcountll(mask);
      if (keep && span != 0xffffffffu) {
        lo = min(lo, (int32_t)(span & 0xffffu));
        hi = max(hi, (int32_t)(span >> 16));
      }
    }
    if (runspans) {
      // the run's span: the union of its items' spans of non-global blocks
      lo = wave_reduce<1>(lo);
      hi = wave_reduce<2>(hi);
      const uint32_t run = lo > hi ? 0xffffffffu : ((uint32_t)lo | ((uint32_t)hi << 16));
      for (int32_t qb = begin + lane; qb < end; qb += 64)
        if (qb - lane == begin ? head_keep : !is_long(item0 + qb)) runspans[item0 + qb] = run;
    }
  }
  if (tid <= kNumQueues) queues[tid] = qstart[tid];
  if (tid < kNumQueues) queues[kQueueCounters + tid * kCounterStride] = 0;
  if (tid == 0) {
    queues[kStartsDone] = 0;
    queues[kHalvesWord] = halves_pay((int64_t)all_work - (int64_t)kItemOverhead * n, max_count, n);
  }
  __syncthreads();
  if (tid == 0 && write_header) {
    __threadfence();
    *header = done;
  }
}

// Where each pair item's K/V stream starts.  The workgroups of one XCD share its L2, and a K/V
// block stays there for only about two block steps of the XCD's 32 workgroups; so a block is
// reused only when the items in flight on the XCD read it at nearly the same time.  Each item
// therefore starts its cyclic walk over its key blocks where the item started just before it on
// the same queue is predicted to be by then: the queue is replayed with 32 workgroups taking
// items as they become free (work = kept blocks + item overhead, the schedule's estimate), and
// the predecessor's position is placed by linear interpolation over the span of non-global key
// blocks of their run.  (With two items a pair at head dim 64 four times as many workgroups take
// halves of the pairs in the same order, which the prediction does not model.)  Items that keep every
// key block start at block 0 (ascending, as in the dense kernel).  The result depends on the plan
// only, so runs stay deterministic.
// One 1024-thread workgroup per queue, over tiles of kStartsTile queue entries; the last
// workgroup to finish writes the plan header.
//  0. All waves load the tile's items, kept counts and spans into LDS.
//  1. Start times (wave 0): the 32 times at which the XCD's workgroups become free are kept
//     sorted over lanes 0..31; the queue's items are replayed 16 at a time -- they start at the
//     16 earliest free times (this differs from taking them one by one only when an item of the
//     group would end before a later one of the group starts), their workgroups' next free times
//     replace those lanes, and a bitonic sort over the 32 lanes restores the order.
//  2. Start blocks (all waves): within a run (the items of one head's range in the queue), each
//     item starts where its predecessor is predicted to be by then: the predecessor's start block
//     advanced by (its elapsed time / its work) of the run's span, cyclically; a run's first item
//     starts at its own first non-global block.  These are segmented prefix sums: a plain prefix
//     sum over the tile less its value where the item's run began (a running maximum of the run
//     starts), the last item's sum carried into the next tile.
constexpr int kStartGroup = 16;
constexpr uint32_t kNoSpan = 0xffffffffu;

template <int K, int H>
__device__ __forceinline__ int32_t bitonic_step(int32_t v, int lane) {
  const int32_t other = lane_xor<H>(v, lane);
  const bool up = ((lane & K) == 0) == ((lane & H) == 0);
  return up ? min(v, other) : max(v, other);
}

constexpr int kStartsTile = 2048;
static_assert(kStartsTile % kStartGroup == 0, "the replay's groups of a queue must not straddle tiles");
__global__ __launch_bounds__(1024) void psa_starts_kernel(
    const int32_t* __restrict__ counts, const uint32_t* __restrict__ spans,
    const uint32_t* __restrict__ runspans, const int32_t* __restrict__ order,
    int32_t* __restrict__ queues, int32_t* __restrict__ starts, PlanHeader* __restrict__ header,
    PlanHeader done, int32_t np, int32_t nb) {
  constexpr int kSlots = 32;                       // workgroups of one XCD
  constexpr int kPer = kStartsTile / 1024;         // entries per thread in the loads
  __shared__ int32_t s_item[kStartsTile], s_cnt[kStartsTile], s_t[kStartsTile];
  __shared__ uint32_t s_own[kStartsTile], s_run[kStartsTile];
  __shared__ int32_t s_v[kStartsTile], s_sum[kStartsTile], s_seg[kStartsTile];
  __shared__ int32_t part[16];
  __shared__ int32_t c_bh, c_t, c_work, c_acc;     // the entry before the tile
  __shared__ uint32_t c_run;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, queue = blockIdx.x;
  const int32_t q0 = queues[queue], q1 = queues[queue + 1];
  if (tid == 0) {
    c_bh = -1;
    c_t = 0;
    c_work = 1;
    c_acc = 0;
    c_run = kNoSpan;
  }
  int32_t free_at = lane < kSlots ? 0 : INT32_MAX; // wave 0, carried over the tiles
  for (int32_t t0 = q0; t0 < q1; t0 += kStartsTile) {
    const int32_t tn = min(kStartsTile, q1 - t0);
    // 0. loads: every thread issues its item indices, then their counts and spans
    int32_t it[kPer];
#pragma unroll
    for (int r = 0; r < kPer; r++) {
      const int32_t i = tid + 1024 * r;
      it[r] = i < tn ? order[t0 + i] : 0;
    }
#pragma unroll
    for (int r = 0; r < kPer; r++) {
      const int32_t i = tid + 1024 * r;
      if (i < tn) {
        s_item[i] = it[r];
        s_cnt[i] = counts[it[r]];
        s_own[i] = spans[it[r]];
        s_run[i] = runspans[it[r]];
      }
    }
    __syncthreads();
    // 1. start times
    if (wave == 0) {
      int32_t w_next = lane < kStartGroup && lane < tn ? s_cnt[lane] : 0;
      for (int32_t g = 0; g < tn; g += kStartGroup) {
        const int32_t gn = min(kStartGroup, tn - g);
        const int32_t w = w_next;
        w_next = lane < kStartGroup && g + kStartGroup + lane < tn ? s_cnt[g + kStartGroup + lane] : 0;
        if (lane < gn) s_t[g + lane] = free_at;    // lane i: the i-th earliest free time
        free_at += lane < gn ? w + kItemOverhead : 0;
        free_at = bitonic_step<2, 1>(free_at, lane);
        free_at = bitonic_step<4, 2>(free_at, lane);
        free_at = bitonic_step<4, 1>(free_at, lane);
        free_at = bitonic_step<8, 4>(free_at, lane);
        free_at = bitonic_step<8, 2>(free_at, lane);
        free_at = bitonic_step<8, 1>(free_at, lane);
        free_at = bitonic_step<16, 8>(free_at, lane);
        free_at = bitonic_step<16, 4>(free_at, lane);
        free_at = bitonic_step<16, 2>(free_at, lane);
        free_at = bitonic_step<16, 1>(free_at, lane);
        free_at = bitonic_step<32, 16>(free_at, lane);
        free_at = bitonic_step<32, 8>(free_at, lane);
        free_at = bitonic_step<32, 4>(free_at, lane);
        free_at = bitonic_step<32, 2>(free_at, lane);
        free_at = bitonic_step<32, 1>(free_at, lane);
        free_at = lane < kSlots ? free_at : INT32_MAX;
      }
    }
    __syncthreads();
    // 2. each entry's step from its predecessor (v), and where its run began (seg)
    for (int32_t i = tid; i < tn; i += 1024) {
      const int32_t bh = s_item[i] / np, t = s_t[i];
      const uint32_t run = s_run[i], own = s_own[i];
      int32_t p_bh, p_t, p_work;
      uint32_t p_run;
      if (i > 0) {
        p_bh = s_item[i - 1] / np;
        p_t = s_t[i - 1];
        p_work = s_cnt[i - 1] + kItemOverhead;
        p_run = s_run[i - 1];
      } else {
        p_bh = c_bh;
        p_t = c_t;
        p_work = c_work;
        p_run = c_run;
      }
      const bool first = p_bh != bh || p_run != run || t0 + i == q0;
      const int32_t lo = (int32_t)(run & 0xffffu), len = (int32_t)(run >> 16) - lo + 1;
      int32_t v = 0;
      if (run != kNoSpan) {
        if (first)
          v = own != kNoSpan ? (int32_t)(own & 0xffffu) - lo : 0;
        else
          v = min(max(t - p_t, 0), p_work - 1) * len / p_work;   // < 2^13 * 2^13
      }
      s_v[i] = v;
      s_sum[i] = v;
      s_seg[i] = first ? i : -1;
    }
    __syncthreads();
    const int32_t carry = c_acc;
    block_scan<false>(s_sum, tn, part);              // exclusive sums
    block_scan<true>(s_seg, tn, part);               // start of each entry's run, -1: before the tile
    for (int32_t i = tid; i < tn; i += 1024) {
      const int32_t seg = s_seg[i];
      const int32_t acc = s_sum[i] + s_v[i] - (seg >= 0 ? s_sum[seg] : -carry);
      const uint32_t run = s_run[i];
      const int32_t lo = (int32_t)(run & 0xffffu), len = (int32_t)(run >> 16) - lo + 1;
      int32_t kb = run == kNoSpan ? 0 : lo + acc % len;
      if (s_cnt[i] >= nb) kb = 0;
      starts[s_item[i]] = kb;
      if (i == tn - 1) {                             // carry into the next tile
        c_bh = s_item[i] / np;
        c_t = s_t[i];
        c_work = s_cnt[i] + kItemOverhead;
        c_run = run;
        c_acc = acc;
      }
    }
    __syncthreads();
  }
  if (tid == 0) {
    __threadfence();
    if (atomicAdd(&queues[kStartsDone], 1) == kNumQueues - 1) {
      __threadfence();
      *header = done;
    }
  }
}

static PlanHeader plan_header(const Geometry& g, int32_t batch, int32_t n_heads) {
  PlanHeader h;
  h.magic = g.block == 64 ? kPlanMagic64 : kPlanMagic;
  h.n_bh = batch * n_heads;
  h.n_heads = n_heads;
  h.nb = g.nb;
  h.block = g.block;
  h.n = g.n;
  h.frames = g.frames;
  h.height = g.height;
  h.width = g.width;
  h.n_text = g.n_text;
  h.pbt = g.pbt;
  h.pbh = g.pbh;
  h.pbw = g.pbw;
  return h;
}

// Whether the plan chooses where the items' K/V streams start (psa_starts_kernel).
static bool has_starts(const Geometry& g) { return g.block == 128; }

// Whether the items are listed longest first (psa_rank_kernel).  Block 128: up to eight pairs per CU;
// from there to 32 per CU the order by heads and this one differ by -1.5 to +1.5 %, beyond it is up to
// 4 % faster (K/V blocks shared in the L2).  Block 64: as long as the kernel can hold the list.  There
// the run alone is 2 % faster in the mean in this order (48 calls of 57 to 1182 blocks a head, 1112 to
// 29184 query blocks, 0.985 to 1.11; with 16 blocks a head and more than 8000 in all 2 to 6 % slower),
// and the plan takes 25 to 35 us less (the schedule kernel 35 to 45 us, this one 10).
static bool ranked(const Geometry& g, int32_t n_items) { return n_items <= (g.block == 64 ? kRankItems : 2048); }

// Whether one kernel per head makes the whole plan but the order.
static bool head_planned(const Geometry& g) { return g.nb <= kHeadPlanRows; }

hipError_t launch_plan(const ParamChunk* chunks, const Geometry& g, int32_t batch, int32_t n_heads,
                       bool full, void* workspace, const WorkspaceLayout& wl, int32_t* kept_per_row,
                       hipStream_t stream) {
  char* ws = (char*)workspace;
  PlanHeader* header = (PlanHeader*)(ws + wl.header);
  psa_stripe_t* params = (psa_stripe_t*)(ws + wl.params);
  int2* coords = (int2*)(ws + wl.coords);
  int2* pairs = (int2*)(ws + wl.pairs);
  int32_t* counts = (int32_t*)(ws + wl.counts);
  const int32_t per_head = pairs_per_head(g.nb), n_items = batch * n_heads * per_head;
  const int32_t n_chunks = (n_heads + kHeadsPerChunk - 1) / kHeadsPerChunk;
  const bool blocks3d = g.pbt > 0, fused = head_planned(g) && ranked(g, n_items);
  const bool split = split_plan(batch * n_heads, g.nb, g.block, full);
  PlanHeader done = plan_header(g, batch, n_heads);
  if (split_by_density(batch * n_heads, g.nb, g.block) && full) done.magic |= kPlanFull;
  hipError_t e;
  if (blocks3d) {
    hipLaunchKernelGGL(psa_tiles3d_kernel, dim3((g.nb + 3) / 4), dim3(256), 0, stream, g, coords,
                       (uint64_t*)(ws + wl.masks));
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  for (int32_t c = 0; c < n_chunks; c++) {
    const ParamChunk& pc = chunks[c];
    const int32_t head0 = c * kHeadsPerChunk;
    if (fused && !split) {
      hipLaunchKernelGGL(psa_head_plan_kernel, dim3(pc.n), dim3(1024), 0, stream, pc, head0, g, batch, n_heads,
                         header, params, coords, pairs, counts, kept_per_row);
    } else {
      const int32_t n = c == 0 && !blocks3d ? max(g.nb, pc.n) : pc.n;
      hipLaunchKernelGGL(psa_setup_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, pc, head0, g, header,
                         params, coords, (int32_t)(c == 0 ? (blocks3d ? 2 : 1) : 0),
                         done, (int32_t)(split && !kept_per_row && c == n_chunks - 1));
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (split) {
    // The split engine needs the parameters and coordinates only.
    if (!kept_per_row) return hipSuccess;
    const int32_t n_rows = n_heads * g.nb;
    hipLaunchKernelGGL(psa_count_kernel, dim3((n_rows + 3) / 4), dim3(256), 0, stream,
                       (const psa_stripe_t*)params, (const int2*)coords, kept_per_row, nullptr, n_rows, g.nb,
                       header, done);
    return hipGetLastError();
  }
  if (!fused) {
    // Row counts and kept-set signatures of one batch element, the pairs of each head, then the
    // work of every pair item.
    const int32_t n_rows = n_heads * g.nb;
    hipLaunchKernelGGL(psa_count_kernel, dim3((n_rows + 3) / 4), dim3(256), 0, stream,
                       (const psa_stripe_t*)params, (const int2*)coords, kept_per_row,
                       (uint64_t*)(ws + wl.sigs), n_rows, g.nb, nullptr, done);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(psa_pairing_kernel, dim3(n_heads), dim3(1024), 0, stream,
                       (const uint64_t*)(ws + wl.sigs), (const psa_stripe_t*)params, (const int2*)coords, pairs,
                       g.nb);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(psa_paircount_kernel, dim3((n_items + 3) / 4), dim3(256), 0, stream,
                       (const psa_stripe_t*)params, (const int2*)coords, (const int2*)pairs, counts,
                       (uint32_t*)(ws + wl.spans), n_items, n_heads, g.nb);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  int32_t* order = (int32_t*)(ws + wl.order);
  int32_t* queues = (int32_t*)(ws + wl.queues);
  int32_t* starts = has_starts(g) ? (int32_t*)(ws + wl.starts) : nullptr;
  if (ranked(g, n_items)) {
    hipLaunchKernelGGL(psa_rank_kernel, dim3(1), dim3(1024), 0, stream, (const int32_t*)counts, order, queues,
                       starts, header, done, per_head,
                       (int32_t)(per_head <= kWholeHead && n_items > kWholeItems && done.n_bh >= kWholeHeads));
    return hipGetLastError();
  }
  const uint32_t* spans = starts ? (const uint32_t*)(ws + wl.spans) : nullptr;
  uint32_t* runspans = starts ? (uint32_t*)(ws + wl.runspans) : nullptr;
  hipLaunchKernelGGL(psa_schedule_kernel, dim3(1), dim3(1024), 0, stream, (const int32_t*)counts, order, queues,
                     header, done, per_head, (int32_t)!starts, spans, runspans);
  if ((e = hipGetLastError()) != hipSuccess || !starts) return e;
  hipLaunchKernelGGL(psa_starts_kernel, dim3(kNumQueues), dim3(1024), 0, stream, (const int32_t*)counts, spans,
                     (const uint32_t*)runspans, (const int32_t*)order, queues, starts, header, done, per_head,
                     g.nb);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Tile engine.
// ---------------------------------------------------------------------------------------------

template <int D, int BLK>
struct Tile {
  static constexpr int kWaves = BLK / 32;      // one wave per 32 query rows
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int KT = BLK / 32;          // 32-key row groups of S^T
  static constexpr int DC = D / 16;            // 16-wide head-dim chunks (Q K^T contraction)
  static constexpr int DT = D / 32;            // 32-row head-dim groups of O^T
  static constexpr int KC = BLK / 16;          // 16-key chunks (P V contraction)
  static constexpr int RB = D * 2;             // LDS bytes per row
  static constexpr int CPR = D / 8;            // 16-byte chunks per row
  static constexpr int BYTES = BLK * RB;       // one K or V block in LDS
  static constexpr int LPW = BYTES / (1024 * kWaves);  // 1 KB DMA slots per wave per tensor
  static_assert(LPW >= 1 && BYTES % (1024 * kWaves) == 0, "tile shape");
};

// XOR swizzle of the 16-byte chunks of LDS row `row` (D = 128: 16 chunks per row).  K reads
// touch the 16 rows {x..x+15} (8 lanes per cycle: rows {x..x+3, x+8..x+11}) at one logical
// chunk; transposed V reads touch 4 consecutive rows r0..r0+3 at 4 consecutive chunks (16 lanes
// per cycle: 2 chunks).  Within a quad of rows, bits (1,2) and bits (2,3) of the swizzle are
// both all distinct; row bits 2 and 3 flip bits 1 and 0.  Every one of these access groups then
// hits distinct banks whether the LDS serves 128 or 256 bytes per clock.  The 8 chunks of D = 64 take
// the low three bits, for which this does not hold: half of its LDS cycles are bank conflicts.
template <int CPR>
__device__ __forceinline__ int swz(int row) {
  const int i = row & 3;
  const int s = (((i >> 1) << 3) | ((i & 1) << 2) | ((i >> 1) << 1)) ^ (((row >> 2) & 1) << 1) ^
                ((row >> 3) & 1);
  return s & (CPR - 1);
}

// Lane l supplies K row sigma(l & 31) of a 32-row group so that accumulator element i of lane l
// holds key 16*(i/8) + 8*(l/32) + (i%8).
__device__ __forceinline__ int key_perm(int r) {
  const int a = r >> 3, hh = (r >> 2) & 1, b = r & 3;
  return 16 * (a >> 1) + 8 * hh + 4 * (a & 1) + b;
}

__device__ __forceinline__ float pair_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ float pair_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}


__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(const PSA_LDS void*)p;
}

__device__ __forceinline__ void dma16(uint32_t lds_addr, uint32_t voff, const void* base) {
  // One wait state separates the M0 write from the LDS DMA that reads it.
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds_addr), "v"(voff), "s"(base)
               : "memory");
}

// Wait until at most N of this wave's DMA loads are outstanding.
template <int N>
__device__ __forceinline__ void wait_dma() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Per-wave state: 32 query rows (lane l owns row l & 31; lanes l and l^32 split its keys).
// Scores live in the exp2 domain: Q is multiplied by scale*log2(e) once, when it is loaded, and
// the S^T accumulators start at -m instead of 0, so the MFMAs deliver S - m and the softmax needs
// no per-score multiply or subtract.
template <int D, int BLK>
struct WaveState {
  using T = Tile<D, BLK>;
  bf16x8 q[T::DC];     // (scale*log2(e) Q)^T B operands
  f32x16 o[T::DT];     // O^T accumulators
  // -m (0 while m = -inf), the initial S^T accumulators.  Head dim 128 keeps all 16 elements in
  // registers; head dim 64 needs those registers for its four waves per SIMD and broadcasts one
  // (16 moves per step; with 16 kept the block loop spills).
  static constexpr bool kScalarM = D == 64;
  using NegM = typename std::conditional<kScalarM, float, f32x16>::type;
  NegM negm;
  __device__ __forceinline__ f32x16 neg_max() const {
    if constexpr (kScalarM) {
      f32x16 z;
#pragma unroll
      for (int i = 0; i < 16; i++) z[i] = negm;
      return z;
    } else {
      return negm;
    }
  }
  __device__ __forceinline__ float base() const {
    if constexpr (kScalarM) return -negm;
    else return -negm[0];
  }
  __device__ __forceinline__ void set_neg_max(float nb) {
    if constexpr (kScalarM) {
      negm = nb;
    } else {
#pragma unroll
      for (int i = 0; i < 16; i++) negm[i] = nb;
    }
  }
  float m;             // base of the weights: at or near the running max of the scaled scores
  float l;             // running sum of the bf16-rounded P over this lane's keys
};

// A key/value block is processed in steps of HK_ keys (S^T: HK_/32 groups of 32 keys per wave): 64 in
// the pair engine (two halves at block 128, the whole block at block 64), half a block in the split
// engine.  Every step updates the online-softmax statistics on its own.
template <int D, int BLK, int HK_ = 64>
struct Half {
  static constexpr int HK = HK_;              // keys per step
  static constexpr int KT = HK / 32;          // 32-key groups of S^T per half
  static constexpr int KC = HK / 16;          // 16-key chunks per half
};

// S^T = K Q^T for keys [k0, k0 + HK) of the block (K rows from LDS).
template <int D, int BLK, int HK = 64>
__device__ __forceinline__ void qk_half(const WaveState<D, BLK>& st,
                                        f32x16 (&s)[Half<D, BLK, HK>::KT], const uint8_t* sk, int k0,
                                        int lane) {
  using T = Tile<D, BLK>;
  using H = Half<D, BLK, HK>;
  const int h = lane >> 5;
  const int krow0 = k0 + key_perm(lane & 31);
  const int ksw = swz<T::CPR>(krow0);   // identical for krow0 + 32 kt
  // The K operands of step cc + 1 are read while the MFMAs of step cc run.
  bf16x8 a[2][H::KT];
#pragma unroll
  for (int kt = 0; kt < H::KT; kt++)
    a[0][kt] = *(const bf16x8*)(sk + (krow0 + 32 * kt) * T::RB + ((h ^ ksw) << 4));
#pragma unroll
  for (int cc = 0; cc < T::DC; cc++) {
    if (cc + 1 < T::DC) {
#pragma unroll
      for (int kt = 0; kt < H::KT; kt++)
        a[(cc + 1) & 1][kt] =
            *(const bf16x8*)(sk + (krow0 + 32 * kt) * T::RB + (((2 * (cc + 1) + h) ^ ksw) << 4));
    }
    __builtin_amdgcn_sched_barrier(0);      // keep the reads ahead of this step's MFMAs
#pragma unroll
    for (int kt = 0; kt < H::KT; kt++)
      s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cc & 1][kt], st.q[cc], cc == 0 ? st.neg_max() : s[kt], 0, 0, 0);
  }
}

// Mask (tail: the block reaches past the sequence end), online-softmax statistics, P^T chunk by
// chunk and O^T += V^T P^T, for keys [k0, k0 + HK) of block kb.
//  * The base m of the weights moves only when a weight would exceed 2^8 (then to the row's maximum),
//    at head dim 64 when one reaches 2 (then to 2^6 above the maximum).  Any base is exact up to the
//    rounding of the weights, which is relative.
//  * Accumulator elements 8*(j&1)..+7 of S^T group j/2 are keys 16j + 8h + 0..7: the B operand
//    of 16-key chunk j.
//  * V^T operand: within each 16-lane group, source lane 4r+c reads V[key0 + r][d0 + 4c .. +3];
//    the transpose read hands lane i the four keys key0..key0+3 at head-dim d0 + i.
//  * Masked keys: past the sequence end (one-dimensional blocks: only the last block), or, in
//    the PSABlock-centric layout (PAD), every position whose bit in the tile's validity words
//    (lo: positions 0..63, hi: 64..127) is clear -- 3D padding and the end of the sequence.
template <int D, int BLK, bool PAD, int HK = 64>
__device__ __forceinline__ void softmax_pv_half(WaveState<D, BLK>& st,
                                                f32x16 (&s)[Half<D, BLK, HK>::KT], const uint8_t* sv,
                                                int kb, int k0, int n, bool tail, uint64_t lo,
                                                uint64_t hi, int lane, int& fresh) {
  using T = Tile<D, BLK>;
  using H = Half<D, BLK, HK>;
  const int h = lane >> 5, g = lane >> 4, j16 = lane & 15;
  if (tail) {
    asm volatile("" ::: "memory");        // keep the mask a branch taken only by partial tiles
    int hh = h;
    if constexpr (D == 64) asm volatile("" : "+v"(hh));       // formed here, not kept in a register
    if constexpr (PAD) {
#pragma unroll
      for (int kt = 0; kt < H::KT; kt++) {
        // This lane's keys of group kt are positions r0 + {0..7, 16..23}: one 64-bit word.
        const int r0 = k0 + 32 * kt + 8 * hh;
        const uint32_t win = (uint32_t)((BLK == 64 || r0 < 64 ? lo : hi) >> (r0 & 63));
#pragma unroll
        for (int i = 0; i < 16; i++)
          if (!((win >> (16 * (i >> 3) + (i & 7))) & 1u)) s[kt][i] = -__builtin_inff();
      }
    } else {
      const int kbase = kb * BLK + k0 + 8 * hh;
#pragma unroll
      for (int kt = 0; kt < H::KT; kt++)
#pragma unroll
        for (int i = 0; i < 16; i++)
          if (kbase + kt * 32 + 16 * (i >> 3) + (i & 7) >= n) s[kt][i] = -__builtin_inff();
    }
  }

  // s holds S - base with base = -negm (m, or 0 before the first kept key).
  // The softmax and its P V form the longest dependent chain of a block; while a wave runs it,
  // it issues ahead of the other wave on its SIMD, whose Q K^T MFMAs fill the gaps (measured:
  // 3 % faster sparse, 2-4 % dense).
  __builtin_amdgcn_s_setprio(1);
  if constexpr (D == 64) {
    // Head dim 64: the weights come first and their bits tell whether the base was too low.  A
    // weight of 2 or more has bit 14 set (bf16, sign 0), so one OR over the packed weights takes
    // the place of the maximum over the scores: 10 instructions instead of 27, of 131 per step,
    // and off the dependent chain between the two products.  Only a step that trips the test, or
    // has a row without a base yet (fresh), finds the maximum; the new base is 2^6 above it, so
    // that later steps rarely trip it again.  bf16 weights keep their relative precision at any
    // base.  Measured 3-4 % faster than the maximum first (878 -> 851 us at 32 heads x 17776
    // tokens); at head dim 128 the same order is equal or up to 4 % slower.
    const int vkey = k0 + 8 * h + (j16 >> 2);
    const int vsw0 = swz<T::CPR>(vkey), vsw1 = swz<T::CPR>(vkey + 4);   // identical for vkey + 16 j
    bf16x8 va[2][T::DT];
    auto read_v = [&](int j) {
#pragma unroll
      for (int dt = 0; dt < T::DT; dt++) {
        const int dd = dt * 32 + 16 * (g & 1) + 4 * (j16 & 3);
        const int lchunk = dd >> 3, inoff = (dd & 7) * 2;
        const uint8_t* a0 = sv + (vkey + 16 * j) * T::RB + ((lchunk ^ vsw0) << 4) + inoff;
        const uint8_t* a1 = sv + (vkey + 16 * j + 4) * T::RB + ((lchunk ^ vsw1) << 4) + inoff;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((PSA_LDS s16x4*)a0);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((PSA_LDS s16x4*)a1);
        va[j & 1][dt] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
    };
    bf16x8 p[H::KC];
    auto weights = [&]() {
#pragma unroll
      for (int j = 0; j < H::KC; j++) {
        f32x8 e;
#pragma unroll
        for (int x = 0; x < 8; x++) e[x] = __builtin_amdgcn_exp2f(s[j >> 1][8 * (j & 1) + x]);
        p[j] = __builtin_convertvector(e, bf16x8);
      }
    };
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    weights();
    uint32_t any = 0;
#pragma unroll
    for (int j = 0; j < H::KC; j++) {
      const u32x4 w = __builtin_bit_cast(u32x4, p[j]);
      any |= w[0] | w[1] | w[2] | w[3];
    }
    if (fresh || __builtin_amdgcn_ballot_w64((any & 0x40004000u) != 0)) {
      asm volatile("" ::: "memory");        // keep this rare path a branch
      float m4[4] = {-__builtin_inff(), -__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
#pragma unroll
      for (int kt = 0; kt < H::KT; kt++)
#pragma unroll
        for (int i = 0; i < 16; i++) m4[i & 3] = fmaxf(m4[i & 3], s[kt][i]);
      const float mx = fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]));
      const float base = st.base();
      const float ms = pair_max(mx) + base;
      const bool need = ms > st.m + 0.5f;
      const float up = ms + 6.0f;
      const float alpha = need ? __builtin_amdgcn_exp2f(st.m - up) : 1.0f;
      const float shift = need ? up - base : 0.0f;
      st.m = need ? up : st.m;
      st.l *= alpha;
#pragma unroll
      for (int dt = 0; dt < T::DT; dt++) st.o[dt] *= alpha;
#pragma unroll
      for (int kt = 0; kt < H::KT; kt++) s[kt] -= shift;
      st.set_neg_max(st.m == -__builtin_inff() ? 0.0f : -st.m);
      fresh = __builtin_amdgcn_ballot_w64(st.m == -__builtin_inff()) != 0;
      weights();
    }
    read_v(0);
#pragma unroll
    for (int j = 0; j < H::KC; j++) {
      if (j + 1 < H::KC) read_v(j + 1);
      __builtin_amdgcn_sched_barrier(0);      // keep the reads ahead of this chunk's MFMAs
      st.l = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p[j], p[j], 0, 1), ones, st.l, false);
      st.l = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p[j], p[j], 2, 3), ones, st.l, false);
      st.l = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p[j], p[j], 4, 5), ones, st.l, false);
      st.l = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p[j], p[j], 6, 7), ones, st.l, false);
#pragma unroll
      for (int dt = 0; dt < T::DT; dt++)
        st.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[j & 1][dt], p[j], st.o[dt], 0, 0, 0);
    }
  } else {
    // Row max as four independent chains, then combined (a short dependent chain).
    float m4[4] = {-__builtin_inff(), -__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
#pragma unroll
    for (int kt = 0; kt < H::KT; kt++)
#pragma unroll
      for (int i = 0; i < 16; i++) m4[i & 3] = fmaxf(m4[i & 3], s[kt][i]);
    const float mx = fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]));
    const float base = st.base();
    const float ms = pair_max(mx) + base;
    const bool need = ms - st.m > 8.0f;     // false for -inf - -inf (NaN)
    if (__builtin_amdgcn_ballot_w64(need)) {
      asm volatile("" ::: "memory");        // keep this rare path a branch
      const float alpha = need ? __builtin_amdgcn_exp2f(st.m - ms) : 1.0f;
      const float shift = need ? ms - base : 0.0f;
      st.m = need ? ms : st.m;
      st.l *= alpha;
#pragma unroll
      for (int dt = 0; dt < T::DT; dt++) st.o[dt] *= alpha;
#pragma unroll
      for (int kt = 0; kt < H::KT; kt++) s[kt] -= shift;
      const float nb = st.m == -__builtin_inff() ? 0.0f : -st.m;
      st.set_neg_max(nb);
    }

    const int vkey = k0 + 8 * h + (j16 >> 2);
    const int vsw0 = swz<T::CPR>(vkey), vsw1 = swz<T::CPR>(vkey + 4);   // identical for vkey + 16 j
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int j = 0; j < H::KC; j++) {
      // The V^T operands of this chunk are read ahead of its exponentials, which hide the LDS
      // latency.
      bf16x8 va[T::DT];
#pragma unroll
      for (int dt = 0; dt < T::DT; dt++) {
        const int dd = dt * 32 + 16 * (g & 1) + 4 * (j16 & 3);
        const int lchunk = dd >> 3, inoff = (dd & 7) * 2;
        const uint8_t* a0 = sv + (vkey + 16 * j) * T::RB + ((lchunk ^ vsw0) << 4) + inoff;
        const uint8_t* a1 = sv + (vkey + 16 * j + 4) * T::RB + ((lchunk ^ vsw1) << 4) + inoff;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((PSA_LDS s16x4*)a0);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((PSA_LDS s16x4*)a1);
        va[dt] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
      __builtin_amdgcn_sched_barrier(0);      // keep the reads ahead of the exponentials
      f32x8 e;
#pragma unroll
      for (int x = 0; x < 8; x++) e[x] = __builtin_amdgcn_exp2f(s[j >> 1][8 * (j & 1) + x]);
      const bf16x8 p = __builtin_convertvector(e, bf16x8);
      // Row sum of the rounded weights, two per instruction: the normaliser matches the P that
      // multiplies V.
      st.l = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p, p, 0, 1), ones, st.l, false);
      st.l = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p, p, 2, 3), ones, st.l, false);
      st.l = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p, p, 4, 5), ones, st.l, false);
      st.l = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p, p, 6, 7), ones, st.l, false);
#pragma unroll
      for (int dt = 0; dt < T::DT; dt++)
        st.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[dt], p, st.o[dt], 0, 0, 0);
    }
  }
  __builtin_amdgcn_s_setprio(0);
}

// Whether a workspace holds a finished plan for exactly the sizes of this launch.
__device__ __forceinline__ bool plan_matches(const PlanHeader& h, const PlanHeader& e) {
  return h.magic == e.magic && h.n_bh == e.n_bh && h.n_heads == e.n_heads && h.nb == e.nb &&
         h.block == e.block && h.n == e.n && h.frames == e.frames && h.height == e.height &&
         h.width == e.width && h.n_text == e.n_text && h.pbt == e.pbt && h.pbh == e.pbh &&
         h.pbw == e.pbw;
}

// Pops the next work item of the persistent schedule (one lane): from queue `queue` first, then
// from the others in turn; -1 once every queue is exhausted.  Queue x holds the SUB parts of list
// positions queues[x] .. queues[x + 1] - 1; the item at position i is order[i] (i itself without
// an order), its part r is returned as SUB item + r.  Counters only grow: a value at or past a
// queue's end is final, so an exhausted queue is recognised with a load and costs no atomic.
template <int SUB>
__device__ __forceinline__ int32_t pop_item(int32_t* __restrict__ queues,
                                            const int32_t* __restrict__ order, int& queue,
                                            int& exhausted) {
  while (exhausted < kNumQueues) {
    const int32_t start = queues[queue], len = (queues[queue + 1] - start) * SUB;
    int32_t* ctr = &queues[kQueueCounters + queue * kCounterStride];
    int32_t idx = len;
    if (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < len) idx = atomicAdd(ctr, 1);
    if (idx < len) {
      const int32_t i = start + idx / SUB;
      return (order ? order[i] : i) * SUB + idx % SUB;
    }
    queue = (queue + 1) % kNumQueues;
    exhausted++;
  }
  return -1;
}

// Arms the queues of a dense call: n_items work items in their natural order, cut into
// kNumQueues contiguous ranges of (nearly) equal length, counters at zero.
__global__ __launch_bounds__(64) void psa_dense_arm_kernel(int32_t* __restrict__ queues,
                                                           int32_t n_items) {
  const int t = threadIdx.x;
  if (t <= kNumQueues) queues[t] = (int32_t)((int64_t)n_items * t / kNumQueues);
  if (t < kNumQueues) queues[kQueueCounters + t * kCounterStride] = 0;
}

// Re-arms the plan's queue counters before each run (a workspace without a matching plan is
// left alone).
__global__ __launch_bounds__(64) void psa_rearm_kernel(int32_t* __restrict__ queues,
                                                       const PlanHeader* __restrict__ header,
                                                       PlanHeader expect) {
  if (!plan_matches(*header, expect)) return;
  if (threadIdx.x < kNumQueues) queues[kQueueCounters + threadIdx.x * kCounterStride] = 0;
}

// ---------------------------------------------------------------------------------------------
// Pair engine: a workgroup of 2 BLK/32 waves.  The first half of the waves takes one query block of
// BLK rows, the second half another (each wave 32 rows, the per-wave tile engine above).  The two
// rows share one stream of K/V blocks -- the union of their kept sets, each entry marked with the
// rows that keep it -- double-buffered in LDS with one barrier per block and every block's loads
// issued during the block before (K after its barrier, V after its first Q K^T); a row skips the
// blocks it does not keep.
// The plan pairs rows with equal kept sets, so a K/V block is loaded once for two query blocks
// and most entries are used by both rows.  Each row visits each of its own kept blocks once;
// at block 128 the stream runs cyclically from a block the plan chooses (psa_starts_kernel), and
// from block 0 for pairs that keep every block; at block 64 it is ascending.
//
// Shapes (PairShape), by what bounds them:
//   * head dim 128, block 128: eight waves, one workgroup per CU: 128 KB of buffers, 256 registers
//     per wave, two waves per SIMD.
//   * head dim 128, block 64: four waves, two workgroups per CU (64 KB + key list each), so two
//     waves per SIMD as well, and one workgroup's barriers are covered by the other.  Before, one
//     query block had a workgroup of two waves, two of those shared a CU -- one wave per SIMD -- and
//     steps were 32 keys: 12 heads x 32760 tokens took 2.77 ms against 1.79 ms, the Wan 2.1 14B rate
//     on large grids is 1.09 PFLOP/s against 0.68.
//   * head dim 64: half the MFMA work per score for the same softmax.  No unit alone bounds it (of the
//     cycles VALU 0.64, LDS 0.51, half of that bank conflicts, MFMA 0.50), so waves matter more than
//     registers: four per SIMD (128 registers each, 32 KB + list per workgroup).  32 heads x 17776
//     tokens, block 64: 1.57 ms with one wave per SIMD, 0.95 with two, 0.90 with three, 0.85 with
//     four.  Where there is enough work per CU (halves_pay) block 128 runs on the same four-wave
//     workgroups (SUB = 2): a work item of the plan's pairs is two parts, one query block each, whose
//     halves are the two groups' rows and whose 128-key blocks are two entries of 64 keys.
//   * head dim 64, block 128, eight waves: one workgroup per CU (two waves per SIMD at 167 registers;
//     four waves mean 128 and spill 37, 1.5 times as long), where there is not, and for dense calls of
//     few items (launch_dense).
// ---------------------------------------------------------------------------------------------

// Direct global->LDS loads of a whole K or V block by the waves of a workgroup: wave w
// loads the 1 KB slots w S .. w S + S - 1.  Slot j covers LDS bytes [1024 j, +1024) of the block;
// lane l writes bytes [1024 j + 16 l, +16): row (64 j + l) / CPR, physical chunk (64 j + l) % CPR,
// which holds logical chunk (physical ^ swz(row)).  The loads are issued from inline assembly (SGPR
// base + 32-bit lane offset, M0 = LDS destination); the compiler does not track them, so every
// consumer first waits with wait_dma<N>() and a barrier.
template <int D, int BLK>
struct DmaPlan {
  using T = Tile<D, BLK>;
  static constexpr int W = 2 * T::kWaves;              // waves of a workgroup
  static constexpr int S = T::BYTES / (1024 * W);      // slots per wave per tensor
  static_assert(S >= 1 && T::BYTES % (1024 * W) == 0, "tile shape");
  uint32_t off[S];
  int wave, lane;

  __device__ __forceinline__ void init(int wave_, int lane_) {
    wave = wave_;
    lane = lane_;
#pragma unroll
    for (int i = 0; i < S; i++) off[i] = offset(i, BLK);
  }

  // Byte offset in the block of the 16 bytes this lane loads for slot i; rows at or past `rows`
  // are clamped to row rows - 1 (their scores are masked).
  __device__ __forceinline__ uint32_t offset(int i, int rows) const {
    int l = lane;
    // Head dim 64 has no registers to keep the addresses of partial blocks in across the block
    // loop: they are formed where they are used.
    if constexpr (D == 64) asm volatile("" : "+v"(l));
    const int p = (wave * S + i) * 64 + l;
    const int row = p / T::CPR;
    const int chunk = (p % T::CPR) ^ swz<T::CPR>(row);
    return (uint32_t)(min(row, rows - 1) * T::RB + chunk * 16);
  }
};

// Loads block kb of one tensor into its LDS buffer.  Rows past the sequence end are clamped to the
// last row: their scores are masked to -inf, so they are never weighted.
template <int D, int BLK>
__device__ __forceinline__ void issue_block(const DmaPlan<D, BLK>& plan, const __bf16* xh,
                                            uint32_t lds, int kb, int n) {
  using P = DmaPlan<D, BLK>;
  kb = __builtin_amdgcn_readfirstlane(kb);
  const int rows = n - kb * BLK;
  const void* base = (const void*)(xh + (size_t)kb * BLK * D);
  const uint32_t l0 = __builtin_amdgcn_readfirstlane(lds + (uint32_t)(plan.wave * P::S) * 1024u);
  if (rows >= BLK) {
#pragma unroll
    for (int i = 0; i < P::S; i++) dma16(l0 + i * 1024u, plan.off[i], base);
  } else {
#pragma unroll
    for (int i = 0; i < P::S; i++) dma16(l0 + i * 1024u, plan.offset(i, rows), base);
  }
}

// O = O^T / l of a finished row block (rows past the end are not stored), LSE if asked.
template <int D, int BLK>
__device__ __forceinline__ void store_rows(const WaveState<D, BLK>& st, __bf16* __restrict__ oh,
                                           float* __restrict__ lseh, int row, int n, int lane) {
  using T = Tile<D, BLK>;
  const int h = lane >> 5;
  const float lsum = pair_sum(st.l);
  const float inv = lsum > 0.0f ? 1.0f / lsum : 0.0f;
  if (row < n) {
    __bf16* dst = oh + (size_t)row * D + 4 * h;
#pragma unroll
    for (int dt = 0; dt < T::DT; dt++)
#pragma unroll
      for (int a = 0; a < 4; a++) {
        const f32x4 v = {st.o[dt][4 * a] * inv, st.o[dt][4 * a + 1] * inv,
                         st.o[dt][4 * a + 2] * inv, st.o[dt][4 * a + 3] * inv};
        *(bf16x4*)(dst + dt * 32 + 8 * a) = __builtin_convertvector(v, bf16x4);
      }
    if (lseh && h == 0)
      lseh[row] = lsum > 0.0f ? (st.m + __builtin_log2f(lsum)) * 0.69314718055994530942f
                              : -__builtin_inff();
  }
}

// The same through LDS: the wave's 32 rows are staged row-major in `stage` (32 x 2D bytes of LDS
// no other wave touches; 16-byte chunks XOR-swizzled by the row), then stored as whole rows, 16
// bytes per lane, so that each store covers 64 x 16 contiguous bytes of O instead of 8 bytes in
// each of 32 rows.  row0 = the wave's first row; lane l holds row row0 + (l & 31).
template <int D, int BLK>
__device__ __forceinline__ void store_rows_staged(const WaveState<D, BLK>& st, __bf16* __restrict__ oh,
                                                  float* __restrict__ lseh, int row0, int n, int lane,
                                                  uint32_t stage) {
  using T = Tile<D, BLK>;
  constexpr int RB = 2 * D;                   // bytes per row
  constexpr int C16 = RB / 16;                // 16-byte chunks per row
  // The lane's addresses are formed here, not hoisted out of the item loop into registers that
  // would stay live across the block loop.
  asm volatile("" : "+v"(lane));
  const int h = lane >> 5, r = lane & 31;
  const float lsum = pair_sum(st.l);
  const float inv = lsum > 0.0f ? 1.0f / lsum : 0.0f;
#pragma unroll
  for (int dt = 0; dt < T::DT; dt++)
#pragma unroll
    for (int a = 0; a < 4; a++) {
      const f32x4 v = {st.o[dt][4 * a] * inv, st.o[dt][4 * a + 1] * inv,
                       st.o[dt][4 * a + 2] * inv, st.o[dt][4 * a + 3] * inv};
      const int chunk = (4 * dt + a) ^ (r & (C16 - 1));        // columns 8 (4 dt + a) + 4 h ...
      *(PSA_LDS bf16x4*)(uintptr_t)(stage + r * RB + chunk * 16 + 8 * h) = __builtin_convertvector(v, bf16x4);
    }
#pragma unroll 2
  for (int j = 0; j < 32 * C16 / 64; j++) {
    const int idx = 64 * j + lane, rr = idx / C16, c = idx % C16;
    const u32x4 val = *(PSA_LDS u32x4*)(uintptr_t)(stage + rr * RB + ((c ^ (rr & (C16 - 1))) * 16));
    if (row0 + rr < n) *(u32x4*)(oh + (size_t)(row0 + rr) * D + 8 * c) = val;
  }
  if (lseh && h == 0 && row0 + r < n)
    lseh[row0 + r] = lsum > 0.0f ? (st.m + __builtin_log2f(lsum)) * 0.69314718055994530942f
                                 : -__builtin_inff();
}

// Entry i of a pair's block stream: key block in bits 0-12, kept by the first row (bit 13) and
// by the second row (bit 14).
constexpr int kEntryRowShift = 13;
constexpr int kEntryBlockMask = (1 << kEntryRowShift) - 1;
static_assert(PSA_MAX_BLOCKS <= (1 << kEntryRowShift), "block index fits the entry");

// One work item of the pair engine: this wave's row (block of BLK query rows, -1: none) of one
// (batch, head) and nu stream entries (SPARSE: in `list`; dense: every block, kept by both rows).
// Block i sits in buffer i & 1; after one barrier (its loads, issued a block earlier, have landed
// and block i - 1 is no longer read) the loads of block i + 1 go out and each row that keeps block
// i runs it: Q K^T, softmax and P V for each step of 64 keys.
template <int D, int BLK, int SUB, bool SPARSE, bool PAD>
__device__ __forceinline__ void process_pair(const DmaPlan<D, BLK>& plan, int grp,
                                             const __bf16* __restrict__ qh,
                                             const __bf16* __restrict__ kh,
                                             const __bf16* __restrict__ vh,
                                             __bf16* __restrict__ oh, float* __restrict__ lseh,
                                             int n, int my_row, int nu, int first,
                                             const uint16_t* list, float c,
                                             uint8_t (*sk)[Tile<D, BLK>::BYTES],
                                             uint8_t (*sv)[Tile<D, BLK>::BYTES],
                                             const uint64_t* masks) {
  using T = Tile<D, BLK>;
  using H = Half<D, BLK>;
  const int tid = threadIdx.x, lane = tid & 63, gw = (tid >> 6) & (T::kWaves - 1);
  const int h = lane >> 5, r32 = lane & 31;
  const int row = my_row * BLK + gw * 32 + r32;

  // Entry i of the stream: list entry first + i, cyclically (SUB = 2: half i % 2 of list entry
  // first + i / 2, kept by both groups).  Dense: block i, kept by both rows, in a word that numbers any
  // number of blocks (its streams can be longer than a list).
  constexpr int kRowShift = SPARSE ? kEntryRowShift : 30;
  auto entry = [&](int i) {
    if constexpr (SPARSE) {
      int j = i / SUB + first;
      const int len = nu / SUB;
      j = j >= len ? j - len : j;
      const int x = (int)__builtin_amdgcn_readfirstlane(list[j]);
      return SUB == 1 ? x : (x & kEntryBlockMask) * SUB + i % SUB;
    } else {
      return (int)((uint32_t)i | (3u << kRowShift));
    }
  };
  auto block_of = [](int x) { return SUB == 1 ? x & ((1 << kRowShift) - 1) : x; };
  // The second half of the sequence's last block may lie past the end altogether; it is loaded
  // from the last half that does not, and masked.
  auto from = [&](int kb) { return SUB == 1 ? kb : min(kb, (n - 1) / BLK); };
  auto issue_k = [&](int buf, int kb) { issue_block<D, BLK>(plan, kh, lds_address(sk[buf]), from(kb), n); };
  auto issue_v = [&](int buf, int kb) { issue_block<D, BLK>(plan, vh, lds_address(sv[buf]), from(kb), n); };
  int e = 0;
  // Sparse: the first block's loads go out before the Q loads, so that the two latencies overlap
  // at the start of the item (dense: after them; the other order measured slower there).
  if constexpr (SPARSE) {
    if (nu > 0) {
      e = entry(0);
      issue_k(0, block_of(e));
      issue_v(0, block_of(e));
    }
  }

  WaveState<D, BLK> st;
  if (my_row >= 0) {
    const bf16x8* src = (const bf16x8*)(qh + (size_t)min(row, n - 1) * D) + h;
#pragma unroll
    for (int cc = 0; cc < T::DC; cc++) st.q[cc] = src[2 * cc];
#pragma unroll
    for (int cc = 0; cc < T::DC; cc++)
      st.q[cc] = __builtin_convertvector(__builtin_convertvector(st.q[cc], f32x8) * c, bf16x8);
#pragma unroll
    for (int cc = 0; cc < T::DC; cc++) asm volatile("" ::"v"(st.q[cc]));
  }
  st.m = -__builtin_inff();
  st.l = 0.0f;
  st.set_neg_max(0.0f);
  int fresh = 1;
#pragma unroll
  for (int dt = 0; dt < T::DT; dt++) st.o[dt] = (f32x16){};

  if constexpr (!SPARSE) {
    if (nu > 0) {
      e = entry(0);
      issue_k(0, block_of(e));
      issue_v(0, block_of(e));
    }
  }
  // The validity words of a block (one word per 64 positions) are read when its loads are issued, a block
  // ahead: read where they are needed they put a scalar load into the chain of every block.  Not with
  // SUB = 2, whose four waves per SIMD hide that load and have no registers left.
  uint64_t lo_next = ~0ull, hi_next = ~0ull;
  auto read_masks = [&](int kb) {
    if constexpr (PAD) {
      lo_next = masks[SUB == 1 ? 2 * kb : kb];
      if constexpr (BLK > 64) hi_next = masks[2 * kb + 1];
    }
  };
  if (SUB == 1 && nu > 0) read_masks(block_of(e));
  // Where the loop's instructions lie within the fetch lines moves the dense kernel of head dim 128 by up
  // to 1.5 % (75600 tokens, 40 heads: 98.0 to 99.3 ms over 13 offsets); this is the best one measured.
  if constexpr (!SPARSE && D == 128 && BLK == 128) asm volatile(".p2align 8\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
  for (int i = 0; i < nu; i++) {
    const int kb = block_of(e);
    const bool mine = my_row >= 0 && (SUB > 1 || ((e >> (kRowShift + grp)) & 1));
    if constexpr (SUB > 1) read_masks(kb);
    const uint64_t lo = lo_next, hi = hi_next;
    const bool tail = PAD ? (BLK > 64 ? lo & hi : lo) != ~0ull : (kb + 1) * BLK > n;
    wait_dma<0>();                                        // block i, issued a block ago
    __syncthreads();                                      // ... by every wave; block i-1 read
    // The next block's K goes out right after the barrier and its V after this block's first
    // Q K^T half: a wave stalls while it issues, and a single burst of all its loads after the
    // barrier, where every wave issues at once, keeps the MFMA pipes idle for longer (measured:
    // sparse 0.5-1.3 % and dense 0.4-3 % faster on two boxes, same bits).
    const bool more = i + 1 < nu;
    int kbn = 0;
    if (more) {
      e = entry(i + 1);
      kbn = block_of(e);
      if constexpr (SUB == 1) read_masks(kbn);
      issue_k((i + 1) & 1, kbn);
    }
    if (mine) {
      const uint8_t* skb = sk[i & 1];
      const uint8_t* svb = sv[i & 1];
      f32x16 s[H::KT];
      qk_half<D, BLK>(st, s, skb, 0, lane);
      if (more) issue_v((i + 1) & 1, kbn);
      softmax_pv_half<D, BLK, PAD>(st, s, svb, kb, 0, n, tail, lo, hi, lane, fresh);
      if constexpr (BLK > H::HK) {
        qk_half<D, BLK>(st, s, skb, H::HK, lane);
        softmax_pv_half<D, BLK, PAD>(st, s, svb, kb, H::HK, n, tail, lo, hi, lane, fresh);
      }
    } else if (more) {
      issue_v((i + 1) & 1, kbn);
    }
  }
  if constexpr (SPARSE) {
    // The buffer of block nu - 2 (every wave passed the barrier of block nu - 1) stages the
    // output: 8 KB per wave, K half for group 0, V half for group 1.
    if (my_row >= 0) {
      static_assert(T::kWaves * 32 * 2 * D <= T::BYTES, "a wave's rows fit its share of a free buffer");
      const uint32_t stage = lds_address(grp == 0 ? sk[nu & 1] : sv[nu & 1]) + gw * (32 * 2 * D);
      store_rows_staged<D, BLK>(st, oh, lseh, my_row * BLK + gw * 32, n, lane, stage);
    }
  } else {
    if (my_row >= 0) store_rows<D, BLK>(st, oh, lseh, row, n, lane);
  }
}

// SPARSE: persistent, workgroups popping pair items (SUB parts each) from the plan's queues.  Dense:
// the pairs (2 p, 2 p + 1) of the flattened (batch*head, pair) list, either popped from armed queues
// by a persistent grid (queues given) or one per workgroup, consecutive workgroups of one XCD taking
// consecutive ones.
// Byte offsets of the plan's sections in the workspace handed to the pair engine (a workspace of
// up to 4 GiB: one base pointer and 32-bit offsets keep fewer kernel arguments live in scalar
// registers than one pointer per section).
struct PlanView {
  uint32_t params, coords, order, queues, masks, pairs, starts;
};

// Waves per SIMD the kernel is compiled for, and the workgroups (of 2 BLK / 32 waves) per CU that
// gives.  See the shapes above.
template <int D, int BLK>
struct PairShape {
  static constexpr int kWavesPerSimd = D == 64 && BLK == 64 ? 4 : 2;
  static constexpr int kPerCu = kWavesPerSimd * 64 / BLK;
};

template <int D, int BLK, int SUB, bool SPARSE, bool PAD>
__global__ __launch_bounds__(BLK * 4) __attribute__((amdgpu_waves_per_eu(PairShape<D, BLK>::kWavesPerSimd, PairShape<D, BLK>::kWavesPerSimd))) void psa_pair_kernel(
    const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
    __bf16* __restrict__ o, float* __restrict__ lse, const uint8_t* __restrict__ ws, PlanView pv,
    PlanHeader expect, float c) {
  using T = Tile<D, BLK>;
  const PlanHeader* header = (const PlanHeader*)ws;
  const psa_stripe_t* params = (const psa_stripe_t*)(ws + pv.params);
  const int2* coords = (const int2*)(ws + pv.coords);
  const int32_t* order = (const int32_t*)(ws + pv.order);
  int32_t* queues = ws ? (int32_t*)(ws + pv.queues) : nullptr;
  const uint64_t* masks = (const uint64_t*)(ws + pv.masks);
  const int2* pairs = (const int2*)(ws + pv.pairs);
  const int32_t* starts = (const int32_t*)(ws + pv.starts);
  constexpr int W = 2 * T::kWaves;            // waves of the workgroup
  __shared__ __attribute__((aligned(1024))) uint8_t sk[2][T::BYTES];
  __shared__ __attribute__((aligned(1024))) uint8_t sv[2][T::BYTES];
  // SPARSE: the key list.  Head dim 64 takes only the nb entries it needs (dynamic LDS), which lets
  // four workgroups share a CU; at head dim 128 registers allow no more than the largest list does,
  // and the fixed address measured 0.4 % faster.
  extern __shared__ uint16_t dynamic_list[];
  __shared__ uint16_t static_list[SPARSE && D == 128 ? PSA_MAX_BLOCKS : 1];
  uint16_t* const list = D == 128 ? static_list : dynamic_list;
  __shared__ int32_t misc[24];

  if constexpr (SPARSE) {
    // A workspace without a finished plan for exactly these sizes is left alone.
    if (!plan_matches(*header, expect)) return;
    // Of the two shapes of head dim 64 at block 128 the plan has chosen one.
    if (D == 64 && BLK * SUB == 128 && (queues[kHalvesWord] != 0) != (SUB == 2)) return;
  }
  const int32_t n_heads = expect.n_heads, n = expect.n, nb = expect.nb;
  const int32_t np = pairs_per_head(nb), n_items = expect.n_bh * np;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int grp = __builtin_amdgcn_readfirstlane(wave / T::kWaves);
  DmaPlan<D, BLK> plan;
  plan.init(__builtin_amdgcn_readfirstlane(wave), lane);
  int queue = blockIdx.x % kNumQueues, exhausted = 0;
  for (int round = 0;; round++) {
    int32_t item;
    if constexpr (SPARSE) {
      // two slots in turn: an item may end without a barrier after this one
      if (tid == 0) misc[14 + (SUB > 1 ? round & 1 : 1)] = pop_item<SUB>(queues, order, queue, exhausted);
      __syncthreads();
      item = __builtin_amdgcn_readfirstlane(misc[14 + (SUB > 1 ? round & 1 : 1)]);
      if (item < 0) break;
    } else if (queues) {
      // Dense, persistent: items from the armed queues in their natural order.
      if (tid == 0) misc[14 + (SUB > 1 ? round & 1 : 1)] = pop_item<SUB>(queues, nullptr, queue, exhausted);
      __syncthreads();
      item = __builtin_amdgcn_readfirstlane(misc[14 + (SUB > 1 ? round & 1 : 1)]);
      if (item < 0) break;
    } else {
      // Dense, one item per workgroup, consecutive workgroups of one XCD on consecutive items.
      if (round > 0) break;
      const int32_t per_xcd = gridDim.x / kNumQueues;
      item = (blockIdx.x % kNumQueues) * per_xcd + blockIdx.x / kNumQueues;
      if (item >= n_items * SUB) break;
    }
    const int part = item % SUB;
    item /= SUB;
    const int32_t bh = item / np, p = item - bh * np, h = bh % n_heads;
    int2 pr;
    if constexpr (SPARSE) {
      pr = pairs[(int64_t)h * np + p];
    } else {
      pr = make_int2(2 * p, 2 * p + 1 < nb ? 2 * p + 1 : -1);
    }
    int my_row;
    if constexpr (SUB == 1) {
      my_row = __builtin_amdgcn_readfirstlane(grp == 0 ? pr.x : pr.y);
    } else {
      // One query block of the pair; the groups take its halves.
      const int q = part == 0 ? pr.x : pr.y;
      if (q < 0) continue;
      pr = make_int2(q, -1);
      my_row = __builtin_amdgcn_readfirstlane(q * SUB + grp);
    }

    int32_t nu = SUB == 1 ? nb : (n + BLK - 1) / BLK, first = 0;
    if constexpr (SPARSE) {
      // In-kernel decode of the union of the two rows' kept key blocks (ascending), and the
      // number of them below the block the plan starts this item's stream at (the stream then
      // runs cyclically from there).
      const psa_stripe_t m = params[h];
      const int2 ca = coords[pr.x];
      const int2 cb = pr.y >= 0 ? coords[pr.y] : make_int2(kDeadTile, 0);
      const int32_t start = BLK * SUB == 128 ? starts[item] : 0;
      nu = 0;
      for (int32_t base = 0; base < nb; base += W * 64) {
        const int32_t kb = base + tid;
        const int2 ck = kb < nb ? coords[kb] : make_int2(kDeadTile, 0);
        const bool ka = tile_keep(m, ca, ck), kbk = tile_keep(m, cb, ck);
        const bool keep = ka || kbk;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(keep);
        const uint64_t below = __builtin_amdgcn_ballot_w64(keep && kb < start);
        if (lane == 0) {
          misc[wave] = __builtin_popcountll(mask);
          misc[16 + wave] = __builtin_popcountll(below);
        }
        __syncthreads();
        int32_t pos = nu, total = 0;
#pragma unroll
        for (int w = 0; w < W; w++) {
          pos += w < wave ? misc[w] : 0;
          total += misc[w];
          first += misc[16 + w];
        }
        pos += __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                         __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
        if (keep)
          list[pos] = (uint16_t)(kb | ((ka ? 1 : 0) << kEntryRowShift) | ((kbk ? 1 : 0) << (kEntryRowShift + 1)));
        nu += total;
        __syncthreads();
      }
      first = __builtin_amdgcn_readfirstlane(first < nu ? first : 0);
      nu *= SUB;
    }
    const size_t off = (size_t)bh * n * D;
    process_pair<D, BLK, SUB, SPARSE, PAD>(plan, grp, q + off, k + off, v + off, o + off,
                                      lse ? lse + (size_t)bh * n : nullptr, n, my_row, nu, first, list,
                                      c, sk, sv, masks);
  }
}

// ---------------------------------------------------------------------------------------------
// Split engine: for problems of so few query blocks that the pair engine's items leave CUs idle.  A
// workgroup of the pair engine's shape takes ONE query block; its two groups of waves hold the same
// rows and take half of every key block each (64 keys at block 128, 32 at block 64), and the two
// online-softmax states are merged through LDS at the end.  One workgroup per query block, all
// resident at once up to 256 of them (512 at block 64), so nothing is scheduled: the time is that of
// the longest query block, half of what it is as half of a pair.  It needs no pairs and no order from
// the plan.  Up to twice as many run in two rounds; the one thing known of their lengths is that text
// rows keep every key block, so they start first (3 heads x 17776 tokens with 226 of text, block 64
// and head dim 64: 269 us in the order of the blocks, 197 with text first).
// Measured (plan and attention, before the pair engine's plan): 2 heads x 1024 x 64, block 64 35 us ->
// 28; 2 heads x 4672 x 128, block 128 79 -> 42; 18 dense heads of 1116 x 64 24 -> 17; 1.5 times over
// 24 drawn calls of this size.
// ---------------------------------------------------------------------------------------------

// Key blocks of the longest sequence the split engine takes (split_sparse: one head of 1024 blocks at block 64).
constexpr int kSplitBlocks = 1024;

template <int D, int BLK, bool SPARSE, bool PAD>
__global__ __launch_bounds__(BLK * 4) __attribute__((amdgpu_waves_per_eu(2, 2))) void psa_split_kernel(
    const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
    __bf16* __restrict__ o, float* __restrict__ lse, const uint8_t* __restrict__ ws, PlanView pv,
    PlanHeader expect, float c) {
  using T = Tile<D, BLK>;
  constexpr int HK = BLK / 2, W = 2 * T::kWaves, DH = T::DT / 2;
  using H = Half<D, BLK, HK>;
  __shared__ __attribute__((aligned(1024))) uint8_t sk[2][T::BYTES];
  __shared__ __attribute__((aligned(1024))) uint8_t sv[2][T::BYTES];
  __shared__ uint16_t list[SPARSE ? kSplitBlocks : 1];
  __shared__ int32_t found[W];
  __shared__ float2 stat[W][32];              // (m, l) of every wave's rows

  if constexpr (SPARSE) {
    // A workspace without a finished plan for exactly these sizes is left alone.  If only the density
    // differs, the pair engine is launched next: its queue counters are set here.
    if (!plan_matches(*(const PlanHeader*)ws, expect)) {
      PlanHeader dense = expect;
      dense.magic |= kPlanFull;
      if (blockIdx.x == 0 && threadIdx.x < kNumQueues &&
          plan_matches(*(const PlanHeader*)ws, dense))
        ((int32_t*)(ws + pv.queues))[kQueueCounters + threadIdx.x * kCounterStride] = 0;
      return;
    }
  }
  const int32_t n_heads = expect.n_heads, n = expect.n, nb = expect.nb;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, gw = wave & (T::kWaves - 1);
  const int grp = __builtin_amdgcn_readfirstlane(wave / T::kWaves);
  const int h = lane >> 5, r32 = lane & 31;
  // The rows of text keep every key block: all of them first, then the others head by head.  (One
  // division and no branch: behind one, the loads of the arguments below wait for it.)
  const int32_t local = SPARSE && expect.n_text > 0 ? (n - expect.n_text) / BLK : nb;
  const int32_t first = expect.n_bh * (nb - local);
  const bool text = (int32_t)blockIdx.x < first;
  const int32_t rank = text ? blockIdx.x : blockIdx.x - first, rows = text ? nb - local : local;
  const int32_t bh = rank / rows, qb = (text ? local : 0) + rank - bh * rows;
  const size_t off = (size_t)bh * n * D;
  const __bf16 *kh = k + off, *vh = v + off;
  const int row = qb * BLK + gw * 32 + r32;

  // The kept key blocks, ascending.
  int32_t nu = nb;
  if constexpr (SPARSE) {
    const psa_stripe_t m = ((const psa_stripe_t*)(ws + pv.params))[bh % n_heads];
    const int2* coords = (const int2*)(ws + pv.coords);
    const int2 cq = coords[qb];
    nu = 0;
    for (int32_t base = 0; base < nb; base += W * 64) {
      const int32_t kb = base + tid;
      const bool keep = kb < nb && tile_keep(m, cq, coords[kb]);
      const uint64_t mask = __builtin_amdgcn_ballot_w64(keep);
      if (lane == 0) found[wave] = __builtin_popcountll(mask);
      __syncthreads();
      int32_t pos = nu;
#pragma unroll
      for (int w = 0; w < W; w++) {
        pos += w < wave ? found[w] : 0;
        nu += found[w];
      }
      if (keep) list[pos + __builtin_popcountll(mask & ((1ull << lane) - 1))] = (uint16_t)kb;
      __syncthreads();
    }
  }
  auto entry = [&](int i) { return SPARSE ? (int)__builtin_amdgcn_readfirstlane(list[i]) : i; };

  DmaPlan<D, BLK> plan;
  plan.init(__builtin_amdgcn_readfirstlane(wave), lane);
  int kb = 0;
  if (nu > 0) {
    kb = entry(0);
    issue_block<D, BLK>(plan, kh, lds_address(sk[0]), kb, n);
    issue_block<D, BLK>(plan, vh, lds_address(sv[0]), kb, n);
  }
  WaveState<D, BLK> st;
  {
    const bf16x8* src = (const bf16x8*)(q + off + (size_t)min(row, n - 1) * D) + h;
#pragma unroll
    for (int cc = 0; cc < T::DC; cc++) st.q[cc] = src[2 * cc];
#pragma unroll
    for (int cc = 0; cc < T::DC; cc++)
      st.q[cc] = __builtin_convertvector(__builtin_convertvector(st.q[cc], f32x8) * c, bf16x8);
#pragma unroll
    for (int cc = 0; cc < T::DC; cc++) asm volatile("" ::"v"(st.q[cc]));
  }
  st.m = -__builtin_inff();
  st.l = 0.0f;
  st.set_neg_max(0.0f);
  int fresh = 1;
#pragma unroll
  for (int dt = 0; dt < T::DT; dt++) st.o[dt] = (f32x16){};

  const int k0 = grp * HK;
  const uint64_t* masks = (const uint64_t*)(ws + pv.masks);
  uint64_t lo_next = ~0ull, hi_next = ~0ull;              // a block ahead, as in the pair engine
  auto read_masks = [&](int b) {
    if constexpr (PAD) {
      lo_next = masks[2 * b];
      if constexpr (BLK > 64) hi_next = masks[2 * b + 1];
    }
  };
  if (nu > 0) read_masks(kb);
  for (int i = 0; i < nu; i++) {
    const uint64_t lo = lo_next, hi = hi_next;
    const bool tail = PAD ? (lo & hi) != ~0ull : (kb + 1) * BLK > n;
    wait_dma<0>();                                        // block i, issued a block ago
    __syncthreads();                                      // ... by every wave; block i-1 read
    const int cur = kb;
    const bool more = i + 1 < nu;
    if (more) {
      kb = entry(i + 1);
      read_masks(kb);
      issue_block<D, BLK>(plan, kh, lds_address(sk[(i + 1) & 1]), kb, n);
    }
    f32x16 s[H::KT];
    qk_half<D, BLK, HK>(st, s, sk[i & 1], k0, lane);
    if (more) issue_block<D, BLK>(plan, vh, lds_address(sv[(i + 1) & 1]), kb, n);
    softmax_pv_half<D, BLK, PAD, HK>(st, s, sv[i & 1], cur, k0, n, tail, lo, hi, lane, fresh);
  }

  // Merge: both groups scale their O to the common base; group g finishes columns 32 DH g .., adding
  // what the other group holds of them.
  const float mine = pair_sum(st.l);
  if (h == 0) stat[wave][r32] = make_float2(st.m, mine);
  __syncthreads();                                        // (also: the buffers are no longer read)
  const float2 other = stat[(1 - grp) * T::kWaves + gw][r32];
  const float top = fmaxf(st.m, other.x);
  const float alpha = st.m == -__builtin_inff() ? 0.0f : __builtin_amdgcn_exp2f(st.m - top);
  const float beta = other.x == -__builtin_inff() ? 0.0f : __builtin_amdgcn_exp2f(other.x - top);
  const float lsum = mine * alpha + other.y * beta;
  const float inv = lsum > 0.0f ? 1.0f / lsum : 0.0f;
  static_assert(W * DH * 4096 <= 4 * T::BYTES, "a wave's half of O fits its share of the buffers");
  constexpr int kPer = T::BYTES / (DH * 4096);            // waves per buffer
  auto slot = [&](int w) { return (f32x4*)((w / kPer < 2 ? sk[w / kPer] : sv[w / kPer - 2]) + (w % kPer) * DH * 4096) + lane; };
  f32x4* out = slot(wave);
#pragma unroll
  for (int j = 0; j < DH; j++)
#pragma unroll
    for (int a = 0; a < 4; a++) {
      const f32x16& x = st.o[j], &y = st.o[DH + j];
      const int e = 4 * a;
      const f32x4 lower = {x[e], x[e + 1], x[e + 2], x[e + 3]}, upper = {y[e], y[e + 1], y[e + 2], y[e + 3]};
      out[(j * 4 + a) * 64] = (grp == 0 ? upper : lower) * alpha;
    }
  __syncthreads();
  const f32x4* in = slot((1 - grp) * T::kWaves + gw);
  __bf16* dst = o + off + (size_t)row * D + 32 * DH * grp + 4 * h;
#pragma unroll
  for (int j = 0; j < DH; j++)
#pragma unroll
    for (int a = 0; a < 4; a++) {
      const f32x16& x = st.o[j], &y = st.o[DH + j];
      const int e = 4 * a;
      const f32x4 lower = {x[e], x[e + 1], x[e + 2], x[e + 3]}, upper = {y[e], y[e + 1], y[e + 2], y[e + 3]};
      const f32x4 sum = ((grp == 0 ? lower : upper) * alpha + in[(j * 4 + a) * 64]) * inv;
      if (row < n) *(bf16x4*)(dst + 32 * j + 8 * a) = __builtin_convertvector(sum, bf16x4);
    }
  if (lse && grp == 0 && h == 0 && row < n)
    lse[(size_t)bh * n + row] = lsum > 0.0f ? (top + __builtin_log2f(lsum)) * 0.69314718055994530942f
                                            : -__builtin_inff();
}

// Workgroups of a persistent grid over n_items work items: as many as fit the device at once (the
// key list, 2 nb bytes of LDS, can allow fewer than the registers do), but no more than there are
// items -- beyond one workgroup per CU the dispatcher stacks them, and of two stacked workgroups
// both may find an item where another CU then stays idle.  A multiple of kNumQueues.
template <int D, int BLK>
static int32_t pair_grid(int32_t cus, int32_t n_items, int32_t list_bytes) {
  constexpr int32_t kLds = 160 * 1024, kFixed = 4 * Tile<D, BLK>::BYTES + 128;
  // (the fixed list of head dim 128 fits kPerCu workgroups)
  const int32_t per_cu = max(1, min((int32_t)PairShape<D, BLK>::kPerCu, kLds / (kFixed + list_bytes)));
  const int32_t grid = min(cus * per_cu, max(cus, n_items));
  return (grid + kNumQueues - 1) / kNumQueues * kNumQueues;
}

template <int D, int BLK, int SUB, bool PAD>
static hipError_t launch_pairs(const void* q, const void* k, const void* v, void* o, float* lse,
                               const PlanHeader& expect, float c, const char* ws, const PlanView& pv, int32_t cus,
                               hipStream_t stream) {
  const int32_t list_bytes = D == 64 ? (2 * expect.nb + 15) & ~15 : 0;
  const int32_t grid = pair_grid<D, BLK>(cus, expect.n_bh * pairs_per_head(expect.nb) * SUB, list_bytes);
  hipLaunchKernelGGL((psa_pair_kernel<D, BLK, SUB, true, PAD>), dim3(grid), dim3(4 * BLK), list_bytes, stream,
                     (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (__bf16*)o, lse,
                     (const uint8_t*)ws, pv, expect, c);
  return hipGetLastError();
}

template <int D, int BLOCK, bool PAD>
static hipError_t launch_sparse_t(const void* q, const void* k, const void* v, void* o,
                                  float* lse, const PlanHeader& sizes, float c,
                                  void* workspace, const WorkspaceLayout& wl, int32_t cus,
                                  hipStream_t stream, int32_t full) {
  char* ws = (char*)workspace;
  static_assert(sizeof(PlanHeader) <= 256, "the plan header is the workspace's first section");
  const PlanView pv = {(uint32_t)wl.params, (uint32_t)wl.coords, (uint32_t)wl.order, (uint32_t)wl.queues,
                       (uint32_t)(PAD ? wl.masks : 0), (uint32_t)wl.pairs, (uint32_t)wl.starts};
  PlanHeader expect = sizes;
  bool rearm = full < 0;
  const bool by_density = split_by_density(expect.n_bh, expect.nb, BLOCK);
  if (split_any(expect.n_bh, expect.nb, BLOCK) || (by_density && full != 1)) {
    hipLaunchKernelGGL((psa_split_kernel<D, BLOCK, true, PAD>), dim3(expect.n_bh * expect.nb), dim3(4 * BLOCK), 0,
                       stream, (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (__bf16*)o, lse,
                       (const uint8_t*)ws, pv, expect, c);
    const hipError_t e = hipGetLastError();
    // Of a run, whose plan's density only the device knows, both engines are launched where it
    // decides, and the one that does not fit the plan returns at once (PSABlock plans are never full).
    if (e != hipSuccess || !by_density || full == 0 || PAD) return e;
    rearm = false;
  }
  if (by_density) expect.magic |= kPlanFull;
  if (rearm) {
    hipLaunchKernelGGL(psa_rearm_kernel, dim3(1), dim3(64), 0, stream, (int32_t*)(ws + wl.queues),
                       (const PlanHeader*)(ws + wl.header), expect);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if constexpr (D == 64 && BLOCK == 128) {
    // The plan's work decides, which only the device knows: where the sizes leave it open both shapes
    // are launched, and the other one returns at once.
    const hipError_t e = launch_pairs<64, 128, 1, PAD>(q, k, v, o, lse, expect, c, ws, pv, cus, stream);
    if (e != hipSuccess || !halves_possible(BLOCK, (int64_t)expect.n_bh * pairs_per_head(expect.nb), expect.nb))
      return e;
    return launch_pairs<64, 64, 2, PAD>(q, k, v, o, lse, expect, c, ws, pv, cus, stream);
  } else {
    return launch_pairs<D, BLOCK, 1, PAD>(q, k, v, o, lse, expect, c, ws, pv, cus, stream);
  }
}

template <bool PAD>
static hipError_t launch_sparse_pad(const void* q, const void* k, const void* v, void* o, float* lse,
                                    int32_t head_dim, int32_t block, const PlanHeader& e, float c, void* workspace,
                                    const WorkspaceLayout& wl, int32_t cus, hipStream_t stream, int32_t full) {
  if (head_dim == 128 && block == 128)
    return launch_sparse_t<128, 128, PAD>(q, k, v, o, lse, e, c, workspace, wl, cus, stream, full);
  if (head_dim == 64 && block == 64)
    return launch_sparse_t<64, 64, PAD>(q, k, v, o, lse, e, c, workspace, wl, cus, stream, full);
  if (head_dim == 128 && block == 64)
    return launch_sparse_t<128, 64, PAD>(q, k, v, o, lse, e, c, workspace, wl, cus, stream, full);
  if (head_dim == 64 && block == 128)
    return launch_sparse_t<64, 128, PAD>(q, k, v, o, lse, e, c, workspace, wl, cus, stream, full);
  return hipErrorInvalidValue;
}

hipError_t launch_sparse(const void* q, const void* k, const void* v, void* o, float* lse,
                         int32_t batch, int32_t n_heads, int32_t head_dim, const Geometry& g,
                         float c, void* workspace, const WorkspaceLayout& wl, int32_t cus,
                         hipStream_t stream, int32_t full) {
  const PlanHeader e = plan_header(g, batch, n_heads);
  return g.pbt > 0 ? launch_sparse_pad<true>(q, k, v, o, lse, head_dim, g.block, e, c, workspace, wl, cus, stream, full)
                   : launch_sparse_pad<false>(q, k, v, o, lse, head_dim, g.block, e, c, workspace, wl, cus, stream, full);
}

// Dense attention.  With queues (a dense workspace) a one-thread-group kernel arms them and a
// persistent grid takes the items; without, one workgroup per item.  The items are pairs of BLK-row
// blocks; every block is kept, so BLK changes neither the keys of a row nor their order, and all
// shapes give the same bits.
template <int D, int BLK>
static hipError_t launch_dense_t(const void* q, const void* k, const void* v, void* o, float* lse,
                                 int32_t n_bh, int32_t n, float c, int32_t* queues, int32_t cus,
                                 hipStream_t stream) {
  PlanHeader e = {};
  e.nb = (n + BLK - 1) / BLK;
  e.n = n;
  const int32_t np = pairs_per_head(e.nb);
  if (queues) {
    hipLaunchKernelGGL(psa_dense_arm_kernel, dim3(1), dim3(64), 0, stream, queues, n_bh * np);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  const PlanView pv = {0, 0, 0, 0, 0, 0, 0};      // the dense workspace is the queue area
  // A launch takes fewer than 2^32 threads: with one workgroup per item, as many heads at a time.
  constexpr int32_t kItems = (int32_t)((((int64_t)1 << 32) - 1) / (4 * BLK) - kNumQueues);
  const int32_t slice = queues ? n_bh : max(1, min(n_bh, kItems / np));
  for (int32_t bh = 0; bh < n_bh; bh += slice) {
    e.n_bh = e.n_heads = min(slice, n_bh - bh);
    const int32_t n_items = e.n_bh * np, per_xcd = (n_items + kNumQueues - 1) / kNumQueues;
    const int32_t grid = queues ? pair_grid<D, BLK>(cus, n_items, 0) : per_xcd * kNumQueues;
    const size_t off = (size_t)bh * n * D;
    hipLaunchKernelGGL((psa_pair_kernel<D, BLK, 1, false, false>), dim3(grid), dim3(4 * BLK), 0, stream,
                       (const __bf16*)q + off, (const __bf16*)k + off, (const __bf16*)v + off, (__bf16*)o + off,
                       lse ? lse + (size_t)bh * n : nullptr, (const uint8_t*)queues, pv, e, c);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

// Longest sequence of the short dense calls below.
constexpr int32_t kDenseShort = 512;

hipError_t launch_dense(const void* q, const void* k, const void* v, void* o, float* lse,
                        int32_t batch, int32_t n_heads, int32_t head_dim, int32_t n_tokens,
                        int32_t block, float c, int32_t* queues, int32_t cus, hipStream_t stream) {
  const int32_t n_bh = batch * n_heads;
  const int32_t nb = (n_tokens + block - 1) / block;
  if (split_any(n_bh, nb, block)) {
    PlanHeader e = {};
    e.n_bh = n_bh;
    e.n_heads = n_bh;
    e.nb = nb;
    e.n = n_tokens;
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(n_bh * nb), dim3(4 * block), 0, stream, (const __bf16*)q, (const __bf16*)k,
                         (const __bf16*)v, (__bf16*)o, lse, (const uint8_t*)nullptr, PlanView{}, e, c);
      return hipGetLastError();
    };
    if (block == 128)
      return head_dim == 128 ? go(psa_split_kernel<128, 128, false, false>) : go(psa_split_kernel<64, 128, false, false>);
    return head_dim == 128 ? go(psa_split_kernel<128, 64, false, false>) : go(psa_split_kernel<64, 64, false, false>);
  }
  // Short sequences take 64-row pairs and a fixed grid: of a 128-row pair half and more would lie past
  // their end, and a pop of the queues costs as much as their items.  Heads x tokens, 128-row pairs
  // and queues -> this: head dim 64 4096 x 64 123 -> 28 us, 4096 x 256 197 -> 141, 4096 x 512 419 ->
  // 374; head dim 128 4096 x 64 105 -> 58, 4096 x 256 273 -> 260, 4096 x 512 739 -> 733, 128 x 384
  // 22.5 -> 19.3.  On longer ones 128-row pairs read K and V half as often (3 to 10 % faster at head
  // dim 128), and the queues level the XCDs.
  if (n_tokens <= kDenseShort) {
    if (head_dim == 128) return launch_dense_t<128, 64>(q, k, v, o, lse, n_bh, n_tokens, c, nullptr, cus, stream);
    if (head_dim == 64) return launch_dense_t<64, 64>(q, k, v, o, lse, n_bh, n_tokens, c, nullptr, cus, stream);
    return hipErrorInvalidValue;
  }
  if (head_dim == 128)
    return launch_dense_t<128, 128>(q, k, v, o, lse, n_bh, n_tokens, c, queues, cus, stream);
  if (head_dim == 64) {
    // No more 256-row items than CUs: one round of them at two waves per SIMD, where the four-wave
    // shape's 128-row items fill the CUs unevenly (48 heads x 1024 tokens 27.4 -> 24.1 us, 12 x 3600
    // 71 -> 61, 6 x 7800 141 -> 117; beyond the line 128 x 768 would take 37.6 against 31.8).
    if ((int64_t)n_bh * pairs_per_head((n_tokens + 127) / 128) <= cus)
      return launch_dense_t<64, 128>(q, k, v, o, lse, n_bh, n_tokens, c, queues, cus, stream);
    return launch_dense_t<64, 64>(q, k, v, o, lse, n_bh, n_tokens, c, queues, cus, stream);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------------------------
// Static scratch of psa_attention_fwd_noalloc: the plan of a call lives in this array instead of
// a caller's workspace.  Every GPU the library runs on holds its own copy, from the time the
// library's code is loaded on it until the process ends.  In host code `scratch` names a host-side
// stand-in, not a device address: the kernels only ever get the address scratch_pointer() looked
// up for the current device.
// ---------------------------------------------------------------------------------------------

static __device__ __align__(256) uint8_t scratch[PSA_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 256;
std::mutex g_scratch_lock;
void* g_scratch_address[kMaxDevices];      // per device, once looked up
}  // namespace

hipError_t scratch_pointer(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_lock);
  if (!g_scratch_address[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));       // device `dev` is current
    if (e != hipSuccess) return e;
    if (!p || ((uintptr_t)p & 255) != 0) return hipErrorInvalidSymbol;
    g_scratch_address[dev] = p;
  }
  *out = g_scratch_address[dev];
  return hipSuccess;
}

}  // namespace psa
