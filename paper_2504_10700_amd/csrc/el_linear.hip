// Per-order channel-mixing linear (see include/el.h): Y[i,k',(l,m)] = sum_k W[l,k,k'] X[i,k,(l,m)]
// (Section 4.1 of arXiv 2504.10700, the linear combination between the pooling and the
// symmetric contraction), forward and backward, on the matrix cores.
//
// One MFMA 16x16x4 multiplies a 16x4 by a 4x16 block; lane L supplies A[i = L%16][kk = L/16]
// and B[kk = L/16][j = L%16] and receives four entries of column j = L%16 of the 16x16 result
// (rows 4*(L/16)+r in fp32, 4*r + L/16 in fp64; r = 0..3).
//
// Forward (and dX, which is the same product on W transposed): rows = 16 atoms, reduction =
// input channels, columns = 16 output channels, one accumulator block per component (l,m); the
// 2l+1 components of an order share their B operand.  With the layout X[atom][channel][lm]
// the A operands of all components of one (atom, channel) are 64 contiguous bytes, and a lane
// ends up with whole 64-byte rows of the result.  Kernels: mfma_forward_bf16_kernel (fp32, l_max = 3,
// reduction channels a multiple of 32: every value as the exact sum of three bfloat16 values),
// mfma_forward_lds_kernel (fp32, l_max = 3, others:
// X staged through LDS once per workgroup, B through a buffer descriptor, result
// rows stored as whole lines through an LDS transpose; the product lives in el_tile.h and is
// shared with the fused linear + contraction kernel) and mfma_forward_kernel (every other
// shape: operands straight from global memory through a four-deep register pipeline).
// dW: rows = 16 input channels, columns = 16 output channels, reduction = atoms (four per
// MFMA) and the components of the order; A and B operands are again 64 contiguous bytes per
// lane.  The atoms are cut into ranges, every range writes a partial dW (mfma_dw_lds_kernel:
// both operands through a ring in LDS; mfma_dw_kernel: every other shape), a
// second kernel adds the partials in a fixed order (no atomics).
// Channel counts outside these tilings: split_forward_kernel and split_dw_kernel (fp64 products and sums); both in one launch
// for the backward of small batches of any channel count (split_backward_kernel).
#include <algorithm>
#include <atomic>
#include <string>
#include <type_traits>
#include <utility>

#include "../../include/el.h"
#include "el_tile.h"
#include "sc_internal.h"

namespace el {
namespace {

using sc::DeviceGuard;
using sc::misaligned;
using sc::set_error;

// ---- work that rides in another launch of the backward (a launch of its own costs 5 to 9 us): W transposed in the dW
// launch, for the dX that follows it; the sum of the partial dW in the dX launch.

// Wt[l][j][k] = W[l][k][j]: the dX product then reads its B operands along rows like the forward.
template <typename T>
struct Transpose {
  const T* W;
  T* Wt;
  int n_l, k_in, k_out;
  int blocks;                                  // workgroups that do it, before those of the launch itself: a multiple of 8 (XCDs), 0: none
};

template <typename T>
__device__ __forceinline__ void transpose_role(const Transpose<T>& t, int block) {
  const int64_t n = static_cast<int64_t>(t.n_l) * t.k_in * t.k_out;
  for (int64_t i = block * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n; i += static_cast<int64_t>(t.blocks) * blockDim.x) {
    const int k = static_cast<int>(i % t.k_in), j = static_cast<int>(i / t.k_in % t.k_out);
    const int l = static_cast<int>(i / (static_cast<int64_t>(t.k_in) * t.k_out));
    t.Wt[i] = t.W[(static_cast<size_t>(l) * t.k_in + k) * t.k_out + j];
  }
}

// dW[i] = sum of part[r][i] over the ranges r, a slice of 64 lanes x 16 bytes at a time.  Four waves share a slice; wave
// q adds the q-th quarter of the ranges (eight sums in turn, sixteen requests in flight, combined in a fixed tree), the four quarter
// sums are added in wave order: a fixed order altogether, so the result is bitwise reproducible.
template <typename T>
struct RangeSum {
  const T* part;
  T* dW;
  int64_t elems;                               // a multiple of kSlice
  int ranges;                                  // 0: nothing to add
  static constexpr int V = 16 / sizeof(T), kSlice = 64 * V;
};

// The slices first, first + stride, ...; quarter: 4 x kSlice elements of LDS per four waves.  Called by all waves of the workgroup.
template <typename T>
__device__ __forceinline__ void add_ranges(const RangeSum<T>& s, int64_t first, int64_t stride, T* quarter) {
  constexpr int V = RangeSum<T>::V, kSlice = RangeSum<T>::kSlice, U = 8;
  typedef T Vec __attribute__((ext_vector_type(V)));
  const int lane = threadIdx.x % kLanes, q = threadIdx.x / kLanes % 4, team = threadIdx.x / 256, teams = blockDim.x / 256;
  const int ra = s.ranges * q / 4, rb = s.ranges * (q + 1) / 4;
  T* const mine = quarter + team * 4 * kSlice;
  for (int64_t s0 = first * teams; s0 * kSlice < s.elems; s0 += stride * teams) {
    const int64_t i = (s0 + team) * kSlice + lane * V;
    const bool live = i < s.elems;
    Vec a[U];
#pragma unroll
    for (int k = 0; k < U; ++k)
#pragma unroll
      for (int v = 0; v < V; ++v) a[k][v] = T(0);
    if (live) {
      const T* src = s.part + i;
      int r = ra;
      for (; r + 2 * U <= rb; r += 2 * U) {
        Vec x[2 * U];
#pragma unroll
        for (int k = 0; k < 2 * U; ++k) x[k] = *reinterpret_cast<const Vec*>(src + static_cast<size_t>(r + k) * s.elems);
#pragma unroll
        for (int k = 0; k < 2 * U; ++k) a[k % U] += x[k];
      }
      for (; r + U <= rb; r += U) {
        Vec x[U];
#pragma unroll
        for (int k = 0; k < U; ++k) x[k] = *reinterpret_cast<const Vec*>(src + static_cast<size_t>(r + k) * s.elems);
#pragma unroll
        for (int k = 0; k < U; ++k) a[k] += x[k];
      }
      for (; r < rb; ++r) a[0] += *reinterpret_cast<const Vec*>(src + static_cast<size_t>(r) * s.elems);
    }
#pragma unroll
    for (int w = U / 2; w >= 1; w /= 2)
#pragma unroll
      for (int k = 0; k < w; ++k) a[k] += a[k + w];
    *reinterpret_cast<Vec*>(mine + q * kSlice + lane * V) = a[0];
    __syncthreads();
    if (q == 0 && live) {
      Vec y = a[0];
#pragma unroll
      for (int w = 1; w < 4; ++w) y += *reinterpret_cast<const Vec*>(mine + w * kSlice + lane * V);
      *reinterpret_cast<Vec*>(s.dW + i) = y;
    }
    __syncthreads();
  }
}

// Y[n][j][c] = sum_k X[n][k][c] * W[l(c)][k][j], W is [L][k_red][k_cols] (the dX product of the
// backward passes W transposed, so that both read their B operands along rows of W).
// One row tile = 16 atoms; wave w owns the column tiles w, w+4, ... and works on CT of them
// at a time.  The grid is persistent: every workgroup walks the row tiles blockIdx.x,
// blockIdx.x + gridDim.x, ...  With one workgroup resident per CU (the accumulators and the
// operand pipeline fill the register file) a grid of one workgroup per row tile would pay the
// launch of a workgroup, the first loads and the drain of the stores once per tile with
// nothing to overlap them (measured 27 us per workgroup against 15 us of matrix time).
// k_red % (4 * kDepth) == 0, k_cols % (64 * CT) == 0.
constexpr int kDepth = 4;  // operand sets of the forward kernel's software pipeline

template <typename T, int LMAX, int CT>
__global__ __launch_bounds__(kThreads) void mfma_forward_kernel(int64_t n_nodes, int k_red, int k_cols,
                                                                const T* __restrict__ X, const T* __restrict__ W,
                                                                T* __restrict__ Y) {
  constexpr int NC = (LMAX + 1) * (LMAX + 1), L = LMAX + 1;
  typedef typename Mma<T>::acc_t acc_t;
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int kq = lane / 16;                    // position inside the reduction step
  const int steps = k_red / 4;
  const int tiles_per_wave = k_cols / (16 * kWaves);
  const int64_t row_tiles = (n_nodes + 15) / 16;
  for (int64_t tile = blockIdx.x; tile < row_tiles; tile += gridDim.x)
  for (int g = 0; g < tiles_per_wave; g += CT) {
    const int64_t n0 = tile * 16;
    int64_t na = n0 + (lane & 15);             // the atom whose A operands this lane supplies
    if (na >= n_nodes) na = n_nodes - 1;       // rows past the end compute on a valid atom and are not stored
    const T* xrow = X + (static_cast<size_t>(na) * k_red + kq) * NC;
    int jc[CT];                                // this lane's column in every tile of the group
#pragma unroll
    for (int t = 0; t < CT; ++t) jc[t] = ((g + t) * kWaves + wave) * 16 + (lane & 15);
    acc_t acc[NC][CT];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int t = 0; t < CT; ++t) acc[c][t] = acc_t{0, 0, 0, 0};

    auto load = [&](int s, T (&a)[NC], T (&b)[L][CT]) {
      load_row<T, NC>(xrow + static_cast<size_t>(s) * 4 * NC, a);
      const int k = s * 4 + kq;
#pragma unroll
      for (int l = 0; l < L; ++l)
#pragma unroll
        for (int t = 0; t < CT; ++t)
          b[l][t] = W[(static_cast<size_t>(l) * k_red + k) * k_cols + jc[t]];
    };
    auto multiply = [&](const T (&a)[NC], const T (&b)[L][CT]) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int t = 0; t < CT; ++t) acc[c][t] = Mma<T>::mma(a[c], b[order_of(c)][t], acc[c][t]);
    };
    // kDepth operand sets in turn: the loads of step s + kDepth - 1 are issued before the
    // products of step s, so that kDepth - 1 steps of matrix work cover the load latency.
    // The loop body has no branch (steps is a multiple of kDepth; prefetches past the end
    // re-read the last step): with branches inside, the compiler's wait-count bookkeeping
    // falls back to waiting for every outstanding load at each step, which serialises the
    // pipeline (measured: 33 us instead of 15 us of matrix time per workgroup).  The scheduling
    // barriers keep the instruction scheduler from regrouping the loads of several steps, which
    // has the same effect (a wait for the newest loads at the top of every iteration).
    T a[kDepth][NC], b[kDepth][L][CT];
#pragma unroll
    for (int q = 0; q < kDepth - 1; ++q) load(q < steps ? q : steps - 1, a[q], b[q]);
    for (int s = 0; s < steps; s += kDepth) {
#pragma unroll
      for (int q = 0; q < kDepth; ++q) {
        const int nxt = s + q + kDepth - 1;
        load(nxt < steps ? nxt : steps - 1, a[(q + kDepth - 1) % kDepth], b[(q + kDepth - 1) % kDepth]);
        __builtin_amdgcn_sched_barrier(0);   // keep the loads ahead of this step's products ...
        multiply(a[q], b[q]);
        __builtin_amdgcn_sched_barrier(0);   // ... and the next step's loads behind them
      }
    }
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t n = n0 + Mma<T>::row(lane, r);
        if (n < n_nodes) {
          T y[NC];
#pragma unroll
          for (int c = 0; c < NC; ++c) y[c] = acc[c][t][r];
          store_row<T, NC>(Y + (static_cast<size_t>(n) * k_cols + jc[t]) * NC, y);
        }
      }
  }
}

// fp32, l_max = 3: the LDS-staged product of el_tile.h.  A full work unit = a row tile x 128
// columns (two column tiles per wave, 128 accumulator registers); see UnitSchedule for the halves.
template <int CT>
__device__ __forceinline__ void forward_lds_unit(int64_t n_nodes, int64_t n0, int g, int k_red, int k_cols,
                                                 const float* __restrict__ X, const float* __restrict__ W,
                                                 float* __restrict__ Y, float* xs) {
  constexpr int NC = 16;
  Mma<float>::acc_t acc[NC][CT];
  int jc[CT];
  lds_tile_product<CT>(n_nodes, n0, g, k_red, k_cols, X, W, xs, acc, jc);
  // (the product ends with a workgroup barrier: its buffers are free for the store stages)
  static_assert(kWaves * kStoreStageFloats <= kBuffers * 16 * kRowPad, "the store stages reuse the product's buffers");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  store_tile_coalesced<CT>(Y, n_nodes, n0, k_cols, jc, acc, xs + wave * kStoreStageFloats);
}

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void mfma_forward_lds_kernel(
    int64_t n_nodes, int k_red, int k_cols, const float* __restrict__ X, const float* __restrict__ W,
    float* __restrict__ Y) {
  __shared__ __attribute__((aligned(16))) float xs[kBuffers * 16 * kRowPad];
  const int groups = k_cols / 128;                       // full units per row tile
  const UnitSchedule u = unit_schedule((n_nodes + 15) / 16 * groups, true);
  if (u.has_half)
    forward_lds_unit<1>(n_nodes, u.half_unit / groups * 16, static_cast<int>(u.half_unit % groups) * 2 + u.half, k_red,
                        k_cols, X, W, Y, xs);
  for (int64_t unit = blockIdx.x; unit < u.n_full; unit += gridDim.x)
    forward_lds_unit<2>(n_nodes, unit / groups * 16, static_cast<int>(unit % groups) * 2, k_red, k_cols, X, W, Y, xs);
}

// The same product on the bfloat16 matrix cores (SplitPass), k_red % 32 == 0: one workgroup of eight waves per CU (256 registers, 12 bytes a lane spilled outside the loop of a step), which
// walks its share of the row tiles of its 128 columns, two tiles a pass.  What bounds it at 8192 atoms and 128 -> 128 channels (two tiles per
// CU, 41 us): 29 us for the rows at the rate of a large copy, 15 us of products, 8 us of stores at the end of the pass with nothing left to
// overlap them.  Forward on inputs from memory, us, before (two workgroups per CU, each with one tile and its own split of
// W; at 10 000 and 12 288 atoms mfma_forward_lds_kernel) -> this: 128 -> 128 channels, 4096 atoms 26.9 -> 23.1, 8192
// 42.3 -> 40.6, 10 000 60.8 -> 55.5, 12 288 65.0 -> 58.3, 24 000 119 -> 113; 256 -> 256, 6000 atoms 99.9 -> 95.4; 256 -> 128, 4096 atoms
// 47.2 -> 37.7; 512 -> 128, 3000 atoms 75 -> 58.  The pairs of X split in the first half of a step, right behind their requests: 4096
// atoms 24.2, 10 000 56.6.  One tile a pass with requests two steps ahead: 24.2 and 55.3, 256 -> 256 6000 atoms 96.6.  Error against 64 bits
// (2-norm, relative), 128 / 256 / 512 channels summed: 0.73e-7, 1.0e-7, 1.5e-7 where the fp32 instruction gives 2.0e-7, 2.9e-7,
// 4.0e-7 (32 products per rounding of the sum); of one nonzero weight per column, largest: 5.98e-8 and 5.96e-8; of
// two, four, six, eight, 2-norm: 3.7e-8 and 3.1e-8, 4.6e-8 and 4.0e-8, 4.9e-8 and 4.7e-8, 5.2e-8 and 5.4e-8.
// kTrans: W is [L][k_cols][k_red], dX reads the weights of the forward as they are.
template <bool kTrans, int G>
__device__ __forceinline__ void split_passes(const SplitArgs& p, int64_t t0, int64_t t1, int j0, unsigned* lds, int* x_bad) {
  int64_t t = t0;
  for (; t + kSplitRows <= t1; t += kSplitRows) SplitPass<kSplitRows, kTrans, G>::run(p, t * 16, j0, lds, x_bad);
  if (t < t1) SplitPass<1, kTrans, G>::run(p, t * 16, j0, lds, x_bad);
}

// sum: partial dW to add up, after the row tiles: by the workgroups that have one tile less than others and would wait for them (16 us
// at 128 channels, more than their share of the sum takes), if they are a quarter of all or more, and by all otherwise.
template <bool kTrans>
__global__ __launch_bounds__(kSplitThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void mfma_forward_bf16_kernel(
    int64_t n_nodes, int k_red, int k_cols, const float* __restrict__ X, const float* __restrict__ W,
    float* __restrict__ Y, RangeSum<float> sum) {
  __shared__ __attribute__((aligned(16))) unsigned lds[2 * kSplitSlot];
  __shared__ int x_bad[kSplitRows];
  const int groups = k_cols / 128, ranges = gridDim.x / groups;
  const int group = blockIdx.x % groups, range = blockIdx.x / groups;
  const int64_t tiles = (n_nodes + 15) / 16;
  const int64_t t0 = tiles * range / ranges, t1 = tiles * (range + 1) / ranges;
  const SplitArgs p{n_nodes, k_red, k_cols, X, W, Y};
  if (__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x)) < kSplitThreads / 2)
    split_passes<kTrans, 0>(p, t0, t1, group * 128, lds, x_bad);
  else
    split_passes<kTrans, 1>(p, t0, t1, group * 128, lds, x_bad);
  if constexpr (kTrans) {
    if (sum.ranges == 0) return;
    const int64_t few = tiles / ranges;
    const int less = static_cast<int>(ranges - tiles % ranges);              // ranges with `few` tiles (all, if they divide evenly)
    static_assert(8 * RangeSum<float>::kSlice <= 2 * kSplitSlot, "the quarter sums reuse the planes");
    float* const quarter = reinterpret_cast<float*>(lds);
    if (4 * less < ranges) add_ranges(sum, blockIdx.x, gridDim.x, quarter);
    else if (t1 - t0 == few) add_ranges(sum, (range - (t0 - range * few)) * groups + group, static_cast<int64_t>(less) * groups, quarter);
  }
}

// The same products with a workgroup per row tile and two of them on a CU (128 registers), each with its own split of W: where hardly more
// tiles than CUs would leave most workgroups of the kernel above with one tile and let all wait for those with two (pair_pays).
__global__ __launch_bounds__(kSplitThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void mfma_forward_bf16_pair_kernel(
    int64_t n_nodes, int k_red, int k_cols, const float* __restrict__ X, const float* __restrict__ W, float* __restrict__ Y) {
  __shared__ __attribute__((aligned(16))) unsigned planes[3 * kPairPlane];
  static_assert(kSplitWaves * kStoreStageFloats <= 3 * kPairPlane, "the store stages reuse the planes");
  const int groups = k_cols / 128;
  const int64_t n0 = blockIdx.x / groups * int64_t(16);
  const int j0 = static_cast<int>(blockIdx.x % groups) * 128;
  // What is computed again is what a pass computes again (32 columns and two orders, or all for a value of X), so that a result does not
  // depend on which of the kernels it is from.
  __shared__ int bad[4][2];
  if (threadIdx.x < 8) (&bad[0][0])[threadIdx.x] = 0;         // (the product begins with a barrier)
  Mma<float>::acc_t acc[16][1];
  bool x_served, redo[2];
  split_tile_product(n_nodes, n0, j0, k_red, k_cols, X, W, planes, acc, x_served, redo);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int jc[1] = {j0 + wave * 16 + static_cast<int>(threadIdx.x % 16)};
  if (redo[0]) bad[wave / 2][0] = 1;
  if (redo[1]) bad[wave / 2][1] = 1;
  const bool all = __syncthreads_or(!x_served);               // (also the barrier after which the planes are free)
  if (all || bad[wave / 2][0] != 0) plain_tile_product<0>(n_nodes, n0, jc[0], k_red, k_cols, X, W, acc);
  if (all || bad[wave / 2][1] != 0) plain_tile_product<1>(n_nodes, n0, jc[0], k_red, k_cols, X, W, acc);
  store_tile_coalesced<1>(Y, n_nodes, n0, k_cols, jc, acc, reinterpret_cast<float*>(planes) + wave * kStoreStageFloats);
}

// Partial dW of a range of atoms: part[range][l][k][j] = sum_{n in range} sum_{m in l} X[n][k][c] dY[n][j][c].
// Workgroup = (range, group of 4 row tiles, group of NT column tiles); wave w owns row tile
// 4*kgroup + w.  k_in % 64 == 0, k_out % (16 * NT) == 0, nodes_per_range % 4 == 0.
template <typename T, int LMAX, int NT>
__global__ __launch_bounds__(kThreads) void mfma_dw_kernel(int64_t n_nodes, int nodes_per_range, int k_in, int k_out,
                                                           const T* __restrict__ X, const T* __restrict__ dY,
                                                           T* __restrict__ part, Transpose<T> tr) {
  constexpr int NC = (LMAX + 1) * (LMAX + 1), L = LMAX + 1;
  typedef typename Mma<T>::acc_t acc_t;
  if (static_cast<int>(blockIdx.x) < tr.blocks) return transpose_role(tr, static_cast<int>(blockIdx.x));
  const int block = static_cast<int>(blockIdx.x) - tr.blocks;
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int jgroups = k_out / (16 * NT), kgroups = k_in / 64;
  const int jg = block % jgroups;
  const int kg = (block / jgroups) % kgroups;
  const int64_t range = block / (jgroups * kgroups);
  const int64_t r0 = range * nodes_per_range;
  const int64_t r1 = (r0 + nodes_per_range < n_nodes) ? r0 + nodes_per_range : n_nodes;
  const int k = (kg * kWaves + wave) * 16 + (lane & 15);   // row (input channel) of this lane's A operands
  const int j0 = jg * NT * 16 + (lane & 15);               // column of this lane in the group's first tile
  acc_t acc[L][NT];
#pragma unroll
  for (int l = 0; l < L; ++l)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[l][t] = acc_t{0, 0, 0, 0};
  for (int64_t n4 = r0; n4 < r1; n4 += 4) {
    const int64_t n = n4 + lane / 16;          // the atom of this lane's position in the reduction step
    const bool valid = n < r1;
    const int64_t nc = valid ? n : r1 - 1;
    T a[NC];
    load_row<T, NC>(X + (static_cast<size_t>(nc) * k_in + k) * NC, a);
    if (!valid) {
#pragma unroll
      for (int c = 0; c < NC; ++c) a[c] = T(0);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      T b[NC];
      load_row<T, NC>(dY + (static_cast<size_t>(nc) * k_out + j0 + t * 16) * NC, b);
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[order_of(c)][t] = Mma<T>::mma(a[c], b[c], acc[order_of(c)][t]);
    }
  }
  T* out = part + static_cast<size_t>(range) * L * k_in * k_out;
  const int kt = (kg * kWaves + wave) * 16;
#pragma unroll
  for (int l = 0; l < L; ++l)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        out[(static_cast<size_t>(l) * k_in + kt + Mma<T>::row(lane, r)) * k_out + j0 + t * 16] = acc[l][t][r];
}

// The same partial dW for fp32, l_max = 3 and k_in a multiple of 128.  A workgroup of eight waves owns 128 input x 64 output channels, a
// wave 32 x 32 of them with all orders (64 accumulator registers; the 32x32x2 instruction: lane L supplies row L % 32 and atom
// L / 32).  X and dY reach the matrix cores through LDS, written there by the memory path itself (loads straight to LDS, no
// registers) in a ring of chunks of four atoms, two of them under way; the operands of two atoms are read before the products of
// the two before them.  One workgroup per CU.
// What bounds it at 10 000 atoms, 128 -> 128 channels (62 us): 34 us of products at 2.4 GHz, which these products do not hold (54 us where
// all values are zero), 5 us for the partial results, 6 us until the first rows are there.  Four waves with X straight in registers and dY
// through them to LDS needed the range in steps of 16 atoms: backward, us, that -> this: 40 atoms 28.0 -> 26.7, 2100 53.8 -> 47.0,
// 10 000 121.1 -> 120.3; 256 -> 128, 2100 atoms 81.2 -> 74.0, 24 000 456 -> 458.
// Error of dW against 64 bits (2-norm, relative), the 16x16x4 instruction (four atoms) / this one (two): 128 -> 128 channels, 40 atoms 1.61e-7 / 1.61e-7,
// 2100 1.96e-7 / 1.95e-7, 10 000 3.78e-7 / 3.78e-7, 100 000 1.153e-6 / 1.155e-6; 256 -> 256, 10 000 7.28e-7 / 7.29e-7; positive values, 10 000, 5.28e-8 /
// 5.29e-8: it does not depend on how many products an instruction takes.
constexpr int kDwRingWaves = 8;
constexpr int kDwRingThreads = kDwRingWaves * kLanes;
constexpr int kDwSlots = 3, kDwChunk = 4;                     // chunks of the ring, atoms of a chunk
constexpr int kDwIn = 128, kDwOut = 64;                       // channels of a workgroup
constexpr int kDwAtom = (kDwIn + kDwOut) * 16;                // floats of an atom in LDS: rows of X, then of dY

__global__ __launch_bounds__(kDwRingThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void mfma_dw_lds_kernel(
    int64_t n_nodes, int nodes_per_range, int k_in, int k_out, const float* __restrict__ X,
    const float* __restrict__ dY, float* __restrict__ part, Transpose<float> tr) {
  typedef float V4 __attribute__((ext_vector_type(4)));
  typedef float V16 __attribute__((ext_vector_type(16)));
  constexpr int L = 4;
  __shared__ __attribute__((aligned(16))) float ring[kDwSlots * kDwChunk * kDwAtom];
  const int lane = threadIdx.x % kLanes;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kLanes);
  const int jgroups = k_out / kDwOut, kgroups = k_in / kDwIn;
  // (the workgroups of a range, which read the same rows, on one XCD: they meet in its L2)
  if (static_cast<int>(blockIdx.x) < tr.blocks) return transpose_role(tr, static_cast<int>(blockIdx.x));
  const int own = static_cast<int>(gridDim.x) - tr.blocks, at = static_cast<int>(blockIdx.x) - tr.blocks;
  const int per_xcd = own / 8, extra = own % 8, xcd = at % 8;
  const int block = xcd * per_xcd + (xcd < extra ? xcd : extra) + at / 8;
  const int j0 = block % jgroups * kDwOut;
  const int k0 = block / jgroups % kgroups * kDwIn;
  const int64_t range = block / (jgroups * kgroups);
  const int64_t r0 = range * nodes_per_range;
  const int64_t r1 = (r0 + nodes_per_range < n_nodes) ? r0 + nodes_per_range : n_nodes;
  const int chunks = static_cast<int>((r1 - r0 + kDwChunk - 1) / kDwChunk);   // at least one

  // A chunk: per wave half an atom, four KB of X (16 channels each) and two of dY.  The four 16-byte pieces of a row are permuted
  // by its channel so that the operand reads meet no bank twice.
  const int piece = (lane / 4) * 64 + ((lane % 4) ^ (lane / 16)) * 16;
  auto request = [&](int chunk, int slot) {                    // (past the end: the last chunk again)
    int64_t n = r0 + kDwChunk * static_cast<int64_t>(chunk < chunks ? chunk : chunks - 1) + wave / 2;
    if (n >= r1) n = r1 - 1;                                   // an atom past the end is a copy that is zeroed when it is read
    float* const to = ring + (slot * kDwChunk + wave / 2) * kDwAtom;
    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(X + (static_cast<size_t>(n) * k_in + k0) * 16), 0, kDwIn * 64, 0x00020000);
    const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(dY + (static_cast<size_t>(n) * k_out + j0) * 16), 0, kDwOut * 64, 0x00020000);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int block = wave % 2 * 4 + i;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(xrs, (__attribute__((address_space(3))) void*)(to + block * 256), 16, piece, block * 1024, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int block = wave % 2 * 2 + i;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(yrs, (__attribute__((address_space(3))) void*)(to + kDwIn * 16 + block * 256), 16, piece,
                                               block * 1024, 0, 0);
    }
  };
  constexpr int kRequests = 6;

  const int i32 = lane % 32, h = lane / 32, wi = wave / 2, wj = wave % 2;
  struct Operands {
    V4 a[4], b[4];
  };
  int aoff[4];                                                 // floats; the columns of the wave lie at a constant distance
#pragma unroll
  for (int p = 0; p < 4; ++p) aoff[p] = h * kDwAtom + i32 * 16 + (p ^ (i32 / 4 % 4)) * 4;
  auto read = [&](int slot, int chunk, int half, Operands& o) {
    const float* const s = ring + (slot * kDwChunk + half * 2) * kDwAtom;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      o.a[p] = *reinterpret_cast<const V4*>(s + wi * 512 + aoff[p]);
      o.b[p] = *reinterpret_cast<const V4*>(s + (kDwIn / 32 + wj) * 512 + aoff[p]);
    }
    const int64_t n = r0 + kDwChunk * static_cast<int64_t>(chunk) + half * 2;
    if (n + 1 >= r1 && n + h >= r1) {
#pragma unroll
      for (int p = 0; p < 4; ++p) o.a[p] = o.b[p] = V4{0, 0, 0, 0};
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  V16 acc[L];
#pragma unroll
  for (int l = 0; l < L; ++l)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[l][r] = 0;
  auto multiply = [&](const Operands& o) {
#pragma unroll
    for (int c = 0; c < 16; ++c)
      acc[order_of(c)] = __builtin_amdgcn_mfma_f32_32x32x2f32(o.a[c / 4][c % 4], o.b[c / 4][c % 4], acc[order_of(c)], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // All but the requests of one chunk of this wave are served, its reads are done, and every wave is here.
  auto meet = [&]() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kRequests) : "memory"); };

  Operands o0, o1;
  request(0, 0);
  request(1, 1);
  meet();
  request(2, 2);
  read(0, 0, 0, o0);
  int slot = 0;
  for (int c = 0; c < chunks; ++c) {
    read(slot, c, 1, o1);
    multiply(o0);
    meet();                                                    // chunk c + 1 is here, chunk c has been read by all
    request(c + kDwSlots, slot);
    slot = slot == kDwSlots - 1 ? 0 : slot + 1;
    read(slot, c + 1, 0, o0);
    multiply(o1);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // no request may reach LDS after the workgroup has given it back
  float* out = part + static_cast<size_t>(range) * L * k_in * k_out;
#pragma unroll
  for (int l = 0; l < L; ++l)
#pragma unroll
    for (int r = 0; r < 16; ++r)                               // rows 8 (r / 4) + 4 (lane / 32) + r % 4 of the 32 x 32 result
      out[(static_cast<size_t>(l) * k_in + k0 + wi * 32 + r / 4 * 8 + h * 4 + r % 4) * k_out + j0 + wj * 32 + i32] = acc[l][r];
}

// The sum of the partial dW as a launch of its own.
template <typename T>
__global__ __launch_bounds__(256) void dw_reduce_kernel(RangeSum<T> sum) {
  __shared__ __attribute__((aligned(16))) T quarter[4 * RangeSum<T>::kSlice];
  add_ranges(sum, blockIdx.x, gridDim.x, quarter);
}

// ---- the products cut along the reduction: any channel count, and batches of few row tiles (split_small)
//
// A workgroup owns 16 atoms x 16 columns with all components and its four waves take every fourth step of the
// reduction; the four partial tiles meet in LDS (fixed order) and leave as whole lines.  TA = type of the products
// and sums: double for channel counts that the kernels above do not tile (their rows may be fp32: the fp64 matrix
// rate is half the fp32 one, and these shapes are far from it), the storage type where only the batch is small.
// What bounds it: small batches the chain of one wave (load -> products -> LDS -> store), large ones the matrix
// cores.  Against one thread per (atom, column) in fp64, us: forward 100 -> 128 channels 155 atoms 198 -> 10, 4000 508 -> 46.
// k_red and k_cols are free: positions past the end supply zeros, columns past the end are not stored.
template <typename TA>
struct SplitRow {   // elements per row of a partial tile in LDS: the four rows that one instruction writes meet no bank twice
  static constexpr int stride = sizeof(TA) == 4 ? 20 : 16;
};

// blockIdx -> logical block such that an XCD's blocks are one contiguous range (the column tiles of a row tile read
// the same rows of X: they meet in one L2).  blocks is a multiple of kXcds.
constexpr int kXcds = 8;
__device__ __forceinline__ int64_t xcd_contiguous_block(unsigned block, unsigned blocks) {
  const int64_t per = blocks / kXcds;
  return (block % kXcds) * per + block / kXcds;
}

// Calls launch(first tile, workgroups) until all tiles (a workgroup of so many threads each) are served: a grid holds
// less than 2^32 threads.  A grid is a multiple of kXcds.
template <typename F>
hipError_t for_all_tiles(int64_t n_tiles, int threads, F&& launch) {
  const int64_t most = (int64_t(1) << 31) / threads;
  for (int64_t tile0 = 0; tile0 < n_tiles; tile0 += most) {
    const int64_t blocks = std::min(n_tiles - tile0, most);
    launch(tile0, static_cast<unsigned>((blocks + kXcds - 1) / kXcds * kXcds));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// The tile at atom n0 and column j0.  kTrans: W is [L][k_cols][k_red] (the dX product reads the weights of the forward as they are).
template <typename TS, typename TA, int LMAX, bool kTrans>
struct SplitTile {
  static constexpr int NC = (LMAX + 1) * (LMAX + 1), L = LMAX + 1;
  static constexpr int CG = NC < 4 ? NC : 4;                 // components per round through LDS
  static constexpr int RS = SplitRow<TA>::stride;
  typedef typename Mma<TA>::acc_t acc_t;
  // in LDS, as two arrays (as one structure the reads of the sums wait for the writes of the result): the partial tiles, the tile
  typedef TA Partial[kWaves][CG][16 * RS];
  typedef TS Out[16][16 * NC];
  static __device__ __forceinline__ void run(int64_t n0, int j0, int64_t n_nodes, int k_red, int k_cols, const TS* X, const TS* W, TS* Y,
                                             Partial& red, Out& out) {
    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    const int kq = lane / 16, i16 = lane & 15;
    const int64_t na = n0 + i16 < n_nodes ? n0 + i16 : n_nodes - 1;
    const int j = j0 + i16 < k_cols ? j0 + i16 : k_cols - 1;
    const int steps = (k_red + 3) / 4;
    const TS* xrow = X + static_cast<size_t>(na) * k_red * NC;
    acc_t acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = acc_t{0, 0, 0, 0};

    auto load = [&](int s, TS (&a)[NC], TS (&b)[L]) {
      const int k = s * 4 + kq, kc = k < k_red ? k : k_red - 1;
      load_unaligned<TS, NC>(xrow + static_cast<size_t>(kc) * NC, a);
#pragma unroll
      for (int l = 0; l < L; ++l)
        b[l] = kTrans ? W[(static_cast<size_t>(l) * k_cols + j) * k_red + kc] : W[(static_cast<size_t>(l) * k_red + kc) * k_cols + j];
    };
    auto multiply = [&](int s, const TS (&a)[NC], const TS (&b)[L]) {
      const bool live = s * 4 + kq < k_red;                    // both operands are zeroed: the row re-read may hold a NaN
#pragma unroll
      for (int c = 0; c < NC; ++c)
        acc[c] = Mma<TA>::mma(live ? static_cast<TA>(a[c]) : TA(0), live ? static_cast<TA>(b[order_of(c)]) : TA(0), acc[c]);
    };
    if (wave < steps) {
      TS a[2][NC], b[2][L];
      load(wave, a[0], b[0]);
      // No request stands under a condition, and steps past the end multiply zeros: behind a condition the compiler puts the requests of W, and
      // every step of a small batch lasts one memory latency more.  Left alone it also moves the requests behind the products that they are to overlap;
      // only the fp64 forward it orders better by itself.  Forward, us, left alone / pinned: 128 -> 128 channels, 40 atoms 9.5 / 7.1, 300 10.0 / 7.5,
      // 2000 22.9 / 22.0; 256 -> 256, 100 17.1 / 11.5; l_max = 2, 300 8.0 / 6.4; 100 -> 128, 1500 23.7 / 21.5; fp64, 128 -> 128, 350 14.8 / 15.4, 3000 67.5 /
      // 68.9, 192 -> 128, 2500 79.0 / 83.9.  Backward in fp64, whose dX reads W strided: 256 -> 128, 199 39.0 / 37.8, 256 -> 256, 150 61.0 / 59.5.
      constexpr bool kPin = sizeof(TS) == 4 || kTrans;
      auto pin = [] {
        if constexpr (kPin) __builtin_amdgcn_sched_barrier(0);
      };
      for (int s = wave; s < steps; s += 2 * kWaves) {
        const int s1 = s + kWaves, s2 = s + 2 * kWaves;
        load(s1 < steps ? s1 : s, a[1], b[1]);
        pin();
        multiply(s, a[0], b[0]);
        pin();
        load(s2 < steps ? s2 : s, a[0], b[0]);
        pin();
        multiply(s1, a[1], b[1]);
      }
    }
    const int er = threadIdx.x / 16, ec = threadIdx.x % 16;    // the entry that this thread sums
#pragma unroll
    for (int c0 = 0; c0 < NC; c0 += CG) {
      if (c0 > 0) __syncthreads();                             // the previous round has been read
#pragma unroll
      for (int c = c0; c < c0 + CG && c < NC; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][c - c0][Mma<TA>::row(lane, r) * RS + i16] = acc[c][r];
      __syncthreads();
#pragma unroll
      for (int c = c0; c < c0 + CG && c < NC; ++c) {
        TA y = red[0][c - c0][er * RS + ec];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) y += red[w][c - c0][er * RS + ec];
        out[er][ec * NC + c] = static_cast<TS>(y);
      }
    }
    __syncthreads();
    constexpr int V = NC % 4 == 0 ? 16 / sizeof(TS) : 1;       // rows of X and Y are whole 16-byte pieces, or not
    typedef TS Vec __attribute__((ext_vector_type(V)));
    constexpr int kPieces = 16 * NC / V;                       // per atom
    const int live = (k_cols - j0 < 16 ? k_cols - j0 : 16) * NC / V;
    for (int q = threadIdx.x; q < 16 * kPieces; q += kThreads) {
      const int r = q / kPieces, p = q % kPieces;
      if (n0 + r < n_nodes && p < live)
        *reinterpret_cast<Vec*>(Y + (static_cast<size_t>(n0 + r) * k_cols + j0) * NC + p * V) =
            *reinterpret_cast<const Vec*>(&out[r][p * V]);
    }
  }
};

// kSum: workgroups from `blocks` on add partial dW.
template <typename TS, typename TA, int LMAX, bool kTrans, bool kSum>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void split_forward_kernel(
    int64_t tile0, unsigned blocks, int64_t n_nodes, int k_red, int k_cols, const TS* __restrict__ X, const TS* __restrict__ W,
    TS* __restrict__ Y, RangeSum<TS> sum) {
  typedef SplitTile<TS, TA, LMAX, kTrans> Tile;
  __shared__ __attribute__((aligned(16))) typename Tile::Partial red;
  __shared__ __attribute__((aligned(16))) typename Tile::Out out;
  const int col_tiles = (k_cols + 15) / 16;
  if constexpr (kSum) {
    if (blockIdx.x >= blocks) {
      static_assert(sizeof(red) >= 4 * RangeSum<TS>::kSlice * sizeof(TS), "the quarter sums reuse the partial tiles");
      return add_ranges(sum, blockIdx.x - blocks, gridDim.x - blocks, reinterpret_cast<TS*>(red));
    }
  }
  const int64_t tile = tile0 + xcd_contiguous_block(blockIdx.x, blocks);
  if (tile >= (n_nodes + 15) / 16 * col_tiles) return;       // the same for the whole workgroup
  Tile::run(tile / col_tiles * 16, static_cast<int>(tile % col_tiles) * 16, n_nodes, k_red, k_cols, X, W, Y, red, out);
}

// The same product where the tiles would be mostly padding (few_channels): one thread per (atom, column), fp64 products
// and sums.  Bound by the bytes of X and Y (l_max = 3, one channel, 200 000 atoms: 8 us for 26 MB).
template <typename TS, int LMAX, bool kTrans>
__global__ __launch_bounds__(kThreads) void few_channels_kernel(int64_t block0, int64_t n_nodes, int k_red, int k_cols,
                                                                const TS* __restrict__ X, const TS* __restrict__ W,
                                                                TS* __restrict__ Y) {
  constexpr int NC = (LMAX + 1) * (LMAX + 1);
  const int64_t i = (block0 + blockIdx.x) * kThreads + threadIdx.x;
  if (i >= n_nodes * k_cols) return;
  const int64_t n = i / k_cols;
  const int j = static_cast<int>(i % k_cols);
  double y[NC] = {};
  for (int k = 0; k < k_red; ++k) {
    TS x[NC];
    load_unaligned<TS, NC>(X + (static_cast<size_t>(n) * k_red + k) * NC, x);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int l = order_of(c);
      y[c] += static_cast<double>(x[c]) *
              static_cast<double>(kTrans ? W[(static_cast<size_t>(l) * k_cols + j) * k_red + k] : W[(static_cast<size_t>(l) * k_red + k) * k_cols + j]);
    }
  }
  TS out[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) out[c] = static_cast<TS>(y[c]);
  store_row<TS, NC>(Y + static_cast<size_t>(i) * NC, out);
}

// dW for any channel count: a workgroup owns 16 x 16 entries of one order, its sixteen waves take every sixteenth
// reduction step (4 atoms); their sums meet in LDS and are added in wave order.  Products and sums in fp64; no
// workspace.  The highest orders, which have the most components, come first in the grid.  Bound by the vector cache
// (four SIMDs ask for 512 lines per 28 products of theirs).  Against one thread per entry, us: 100 -> 128 channels, 155
// atoms 143 -> 7, 4000 3980 -> 120; 96 -> 96, 3000 atoms 2962 -> 75.
constexpr int kDwWaves = 16;

template <typename TS, int ORDER, int kDwWaves>
__device__ __forceinline__ void split_dw_order(int64_t n_nodes, int nc, int k_in, int k_out, const TS* __restrict__ X,
                                               const TS* __restrict__ dY, TS* __restrict__ dW, int k0, int j0,
                                               double (*red)[256]) {
  constexpr int M = 2 * ORDER + 1;
  typedef Mma<double>::acc_t acc_t;
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int nq = lane / 16, i16 = lane & 15;
  const int k = k0 + i16 < k_in ? k0 + i16 : k_in - 1, j = j0 + i16 < k_out ? j0 + i16 : k_out - 1;
  const TS* xcol = X + static_cast<size_t>(k) * nc + ORDER * ORDER;
  const TS* ycol = dY + static_cast<size_t>(j) * nc + ORDER * ORDER;
  acc_t acc{0, 0, 0, 0};
  const int64_t steps = (n_nodes + 3) / 4;
  auto load = [&](int64_t s, TS (&a)[M], TS (&b)[M]) {
    const int64_t n = s * 4 + nq;
    const size_t nc_ = static_cast<size_t>(n < n_nodes ? n : n_nodes - 1);
    load_unaligned<TS, M>(xcol + nc_ * k_in * nc, a);
    load_unaligned<TS, M>(ycol + nc_ * k_out * nc, b);
  };
  auto multiply = [&](int64_t s, const TS (&a)[M], const TS (&b)[M]) {
    const bool live = s * 4 + nq < n_nodes;                  // both operands are zeroed: the row re-read may hold a NaN
#pragma unroll
    for (int c = 0; c < M; ++c)
      acc = Mma<double>::mma(live ? static_cast<double>(a[c]) : 0.0, live ? static_cast<double>(b[c]) : 0.0, acc);
  };
  if (wave < steps) {
    TS a[2][M], b[2][M];
    load(wave, a[0], b[0]);
    // Requests before the products that they overlap, as in SplitTile, where the steps of a wave are few (split_backward_kernel; 40 atoms, 256 -> 256
    // channels 35 -> 22 us); sixteen waves of long sums are better left alone (fp64, 96 -> 96, 300 atoms 21 against 24).
    constexpr bool kPin = kDwWaves == kWaves;
    for (int64_t s = wave; s < steps; s += 2 * kDwWaves) {
      const int64_t s1 = s + kDwWaves, s2 = s + 2 * kDwWaves;
      load(s1 < steps ? s1 : s, a[1], b[1]);
      if constexpr (kPin) {
        __builtin_amdgcn_sched_barrier(0);
        multiply(s, a[0], b[0]);
        __builtin_amdgcn_sched_barrier(0);
        load(s2 < steps ? s2 : s, a[0], b[0]);
        __builtin_amdgcn_sched_barrier(0);
        multiply(s1, a[1], b[1]);
      } else {
        multiply(s, a[0], b[0]);
        if (s1 < steps) {
          load(s2 < steps ? s2 : s1, a[0], b[0]);
          multiply(s1, a[1], b[1]);
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][Mma<double>::row(lane, r) * 16 + i16] = acc[r];
  __syncthreads();
  const int e = threadIdx.x, ko = k0 + e / 16, jo = j0 + e % 16;
  if (e >= 256 || ko >= k_in || jo >= k_out) return;
  double y = red[0][e];
#pragma unroll
  for (int w = 1; w < kDwWaves; ++w) y += red[w][e];
  dW[(static_cast<size_t>(ORDER) * k_in + ko) * k_out + jo] = static_cast<TS>(y);
}

// Tile `tile` of order l_max - `rank`.  red: kW partial tiles of LDS.
template <typename TS, int kW>
__device__ __forceinline__ void split_dw_tile(int64_t tile, int rank, int64_t n_nodes, int l_max, int k_in, int k_out, const TS* __restrict__ X,
                                              const TS* __restrict__ dY, TS* __restrict__ dW, double (*red)[256]) {
  const int jtiles = (k_out + 15) / 16, nc = (l_max + 1) * (l_max + 1);
  if (tile >= static_cast<int64_t>((k_in + 15) / 16) * jtiles) return;   // the grid is rounded up; the whole workgroup
  const int j0 = static_cast<int>(tile % jtiles) * 16, k0 = static_cast<int>(tile / jtiles) * 16;
  switch (l_max - rank) {
    case 0: return split_dw_order<TS, 0, kW>(n_nodes, nc, k_in, k_out, X, dY, dW, k0, j0, red);
    case 1: return split_dw_order<TS, 1, kW>(n_nodes, nc, k_in, k_out, X, dY, dW, k0, j0, red);
    case 2: return split_dw_order<TS, 2, kW>(n_nodes, nc, k_in, k_out, X, dY, dW, k0, j0, red);
    default: return split_dw_order<TS, 3, kW>(n_nodes, nc, k_in, k_out, X, dY, dW, k0, j0, red);
  }
}

template <typename TS>
__global__ __launch_bounds__(kDwWaves * kLanes) void split_dw_kernel(int64_t tile0, int64_t n_nodes, int l_max, int k_in,
                                                                     int k_out, const TS* __restrict__ X, const TS* __restrict__ dY,
                                                                     TS* __restrict__ dW) {
  __shared__ double red[kDwWaves][256];
  split_dw_tile<TS, kDwWaves>(tile0 + blockIdx.x, static_cast<int>(blockIdx.y), n_nodes, l_max, k_in, k_out, X, dY, dW, red);
}

// The backward of a small batch as one launch (backward_together): workgroups [0, dx_tiles) own tiles of dX, the others tiles of dW, dw_tiles per
// order, the highest first (both numbers are multiples of kXcds).  dW with four waves a tile for sixteen: both kinds last as long as the chain of
// one wave, and run beside each other.
template <typename TS, typename TA, int LMAX>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void split_backward_kernel(
    unsigned dx_tiles, unsigned dw_tiles, int64_t n_nodes, int k_in, int k_out, const TS* __restrict__ X, const TS* __restrict__ W,
    const TS* __restrict__ dY, TS* __restrict__ dX, TS* __restrict__ dW) {
  typedef SplitTile<TS, TA, LMAX, true> Tile;
  typedef double DwPartial[kWaves][256];
  __shared__ __attribute__((aligned(16))) unsigned char partial[std::max(sizeof(typename Tile::Partial), sizeof(DwPartial))];
  __shared__ __attribute__((aligned(16))) typename Tile::Out out;
  if (blockIdx.x >= dx_tiles) {
    const unsigned block = blockIdx.x - dx_tiles;
    return split_dw_tile<TS, kWaves>(xcd_contiguous_block(block % dw_tiles, dw_tiles), static_cast<int>(block / dw_tiles), n_nodes, LMAX, k_in, k_out,
                                     X, dY, dW, *reinterpret_cast<DwPartial*>(partial));
  }
  const int col_tiles = (k_in + 15) / 16;
  const int64_t tile = xcd_contiguous_block(blockIdx.x, dx_tiles);
  if (tile >= (n_nodes + 15) / 16 * col_tiles) return;       // the same for the whole workgroup
  Tile::run(tile / col_tiles * 16, static_cast<int>(tile % col_tiles) * 16, n_nodes, k_out, k_in, dY, W, dX,
            *reinterpret_cast<typename Tile::Partial*>(partial), out);
}

__global__ void zero_kernel(unsigned int* p, size_t n_words) {
  for (size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; i < n_words;
       i += static_cast<size_t>(gridDim.x) * blockDim.x)
    p[i] = 0u;
}

template <typename T>
__global__ void transpose_w_kernel(Transpose<T> t) {
  transpose_role(t, static_cast<int>(blockIdx.x));
}

// ---- host side

size_t elem_size(const el_config* c) { return c->dtype == SC_F64 ? 8 : 4; }

sc_status check_config(const char* fn, const el_config* cfg, int64_t n) {
  if (!cfg) return set_error(SC_ERR_INVALID_ARG, std::string(fn) + ": cfg is NULL");
  if (cfg->struct_size != static_cast<int32_t>(sizeof(el_config)))
    return set_error(SC_ERR_INVALID_ARG, std::string(fn) + ": struct_size does not match this library's el_config");
  if (cfg->k_in < 1 || cfg->k_out < 1) return set_error(SC_ERR_INVALID_ARG, std::string(fn) + ": k_in or k_out < 1");
  if (cfg->l_max < 0 || cfg->l_max > SC_MAX_L) return set_error(SC_ERR_UNSUPPORTED, std::string(fn) + ": l_max outside 0..3");
  if (cfg->dtype != SC_F32 && cfg->dtype != SC_F64) return set_error(SC_ERR_INVALID_ARG, std::string(fn) + ": bad dtype");
  if (n < 0 || n > (int64_t(1) << 30)) return set_error(SC_ERR_INVALID_ARG, std::string(fn) + ": n_nodes outside 0..2^30");
  return SC_OK;
}

// Compute units of the current device (asked once per device).
int compute_units() {
  static std::atomic<int> cached[64];   // zero-initialised; any thread may fill an entry, all with the same value
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

// Is the product with k_red reduction channels and k_cols output channels served by the MFMA kernel?
bool mfma_forward_ok(int k_red, int k_cols) { return k_red % (4 * kDepth) == 0 && k_cols % 64 == 0; }
bool mfma_dw_ok(const el_config* c) { return c->k_in % 64 == 0 && c->k_out % 64 == 0; }

// Does split_forward_kernel take a product that the other kernels tile as well?  Up to about one round of its
// resident workgroups (a workgroup per 16 atoms x 16 columns, four of them per CU in fp32), where the others leave
// most of the chip idle and run the whole reduction in one wave.  Forward, us, 128 -> 128 channels, other / split: fp32
// l_max = 3, 61 atoms 34.4 / 10.2, 1000 23.6 / 14.2, 2000 26.7 / 25.5, 4000 30.0 / 43.2; l_max = 2, 1000 atoms
// 17.0 / 10.8, 2000 18.5 / 18.6; 256 -> 128, 2000 atoms 47.7 / 40.1, 4000 52.2 / 71.3; fp64 (whose other kernel has
// one wave per SIMD) 61 atoms 77.7 / 16.2, 2000 85.8 / 48.7, 4000 91.9 / 84.7.  Columns that take the other kernel several
// turns of 64 (192): backward of 192 -> 128, 2000 atoms 99.9 / 72.1, 4000 130 / 123.
bool split_small(size_t elem, int64_t n, int k_cols) {
  const bool long_other = elem == 8 || (k_cols > 64 && k_cols % 128 != 0);
  return (n + 15) / 16 * (k_cols / 16) <= static_cast<int64_t>(long_other ? 8 : 4) * compute_units();
}

// Does few_channels_kernel take a product of untiled channel counts?  A tile pads them to 4 x 16.  Forward of 200 000 atoms, us,
// split_forward_kernel / few_channels_kernel: l_max = 3, 1 -> 1 channels 93 / 8, 3 -> 2 97 / 18; l_max = 2, 2 -> 8 63 / 19; l_max = 1,
// 3 -> 8 22 / 9, 1 -> 128 196 / 91; l_max = 0, 5 -> 8 10.5 / 6.  Up to 20 000 atoms the calls take what a launch takes, 4 to 9 us, either way.
bool few_channels(int l_max, int k_red, int k_cols) {
  return (k_red <= 5 && k_cols <= 8 && k_red * k_cols * (l_max + 1) <= 64) || (l_max == 1 && k_red <= 2);
}

// Does dX read W as it is?  Its strided reads of W save the launch that transposes W and cost less than it as long
// as there is no more than one workgroup per CU.  Backward, us, 128 -> 128 channels, W as it is / transposed: fp32 61 atoms
// 27.9 / 29.2, 500 31.8 / 33.4, 1000 44.3 / 39.8, 2000 73.1 / 55.3; fp64 500 atoms 41.8 / 44.5, 2000 117 / 113.
bool dx_reads_w_as_is(int64_t n, int k_cols) { return (n + 15) / 16 * (k_cols / 16) <= compute_units(); }

// Is the product served by mfma_forward_bf16_kernel, beyond the batches of split_forward_kernel?  (Its 31-bit offsets into W
// go through a buffer descriptor.)  With up to 64 channels summed a pass is mostly the split of its W and its stores: beyond two row tiles
// per CU not with 32 channels, and with 64 not where less than half of the CUs get one more of two to five (forward, 32 -> 128 channels, us,
// mfma_forward_lds_kernel / this kernel: 10 000 atoms 27.7 / 31.1, 48 000 104 / 114; 64 -> 128, 10 000 atoms 38.5 / 40.3, 20 000 70 / 69).
bool bf16_parts_ok(size_t elem, int l_max, int64_t n, int k_red, int k_cols) {
  if (!(elem == 4 && l_max == 3 && k_cols % 128 == 0 && k_red % kSplitChunk == 0 && mfma_forward_ok(k_red, k_cols) &&
        static_cast<int64_t>(k_red) * k_cols < (int64_t(1) << 26) && !split_small(elem, n, k_cols)))
    return false;
  const int64_t cus = compute_units(), units = (n + 15) / 16 * (k_cols / 128), more = units % cus;
  if (units <= 2 * cus || k_red > 64) return true;
  return k_red == 64 && (units > 5 * cus || more == 0 || more > cus / 2);
}

// ... and with W read along its rows (not dX, whose launch also adds the partial dW) by the kernel with two workgroups on a CU?  Up to a quarter
// more row tiles than CUs, with fewer channels summed up to five eighths more and twice as many, because the second tile of a pass costs more of it
// there; 64 channels also beyond five tiles per CU, where a pass is mostly its stores.  Forward, us, one / two workgroups on a CU: 128 -> 128
// channels, 4097 atoms 33.3 / 28.6, 4448 34.5 / 31.5, 5000 34.4 / 32.1, 6000 34.4 / 35.2; 256 -> 128, 4100 54.8 / 50.4; 256 -> 256, 2100 55.9 / 53.5, 3000 55.2 /
// 56.2; 96 -> 128, 4100 27.5 / 23.9, 6400 29.4 / 27.8; 64 -> 128, 4100 22.8 / 19.2, 6400 23.9 / 23.2, 20 640 75.9 / 70.1, 40 000 123 / 119; 32 -> 128, 2100
// 10.8 / 9.8, 5000 18.5 / 14.9, 8192 21.7 / 21.2.
bool pair_pays(int64_t n, int k_red, int k_cols) {
  const int64_t cus = compute_units(), units = (n + 15) / 16 * (k_cols / 128);
  if (k_red <= 32) return true;                // (up to two per CU: bf16_parts_ok)
  if (k_red == 64 && units > 5 * cus && units < (int64_t(1) << 22)) return true;   // (a workgroup each: the grid's limit)
  return units > cus && units <= cus + (k_red <= 96 ? cus * 5 / 8 : cus / 4);
}

// ... whose dX reads W as it is: a lane's channels are contiguous there and the launch that transposes W is saved.  (Backward, us, with
// the kernel of two workgroups per CU, W transposed / as it is: 128 -> 128 channels, 2100 atoms 60.8 / 57.8, 8192 108 / 100, 20 480
// 237 / 226; 256 -> 128, 3000 atoms 87.4 / 83.5, 20 000 429 / 407; 256 -> 256, 20 000 atoms 716 / 714.)
bool dx_parts_read_w_as_is(const el_config* c, int64_t n) {
  return bf16_parts_ok(elem_size(c), c->l_max, n, c->k_out, c->k_in);
}

// Is the LDS-staged dW kernel the one for this configuration?
bool dw_lds_ok(const el_config* c) { return c->dtype == SC_F32 && c->l_max == 3 && c->k_in % 128 == 0 && c->k_out % 64 == 0; }

// Atoms per range of the dW kernel: enough ranges to fill the chip about once, a multiple of 4.
int nodes_per_range(const el_config* cfg, int64_t n) {
  const int groups = (dw_lds_ok(cfg) ? cfg->k_in / 128 : cfg->k_in / 64) * (cfg->k_out / 64);
  int64_t ranges = std::max<int64_t>(1, 256 / std::max(1, groups));
  int64_t per = (n + ranges - 1) / ranges;
  per = std::max<int64_t>(16, (per + 3) / 4 * 4);
  return static_cast<int>(std::min<int64_t>(per, int64_t(1) << 20));
}

// ride: partial dW that the launch may add up (it then sets ride->ranges to 0); NULL: none.
template <typename T, typename TA, int LMAX, bool kTrans>
hipError_t launch_split(int64_t n, int k_red, int k_cols, const void* X, const void* W, void* Y, RangeSum<T>* ride, hipStream_t stream) {
  return for_all_tiles((n + 15) / 16 * ((k_cols + 15) / 16), kThreads, [&](int64_t tile0, unsigned grid) {
    const T *x = static_cast<const T*>(X), *w = static_cast<const T*>(W);
    T* y = static_cast<T*>(Y);
    if constexpr (sizeof(T) == sizeof(TA)) {
      if (ride && ride->ranges > 0) {
        const unsigned more = static_cast<unsigned>(std::min<int64_t>((ride->elems + ride->kSlice - 1) / ride->kSlice, compute_units()));
        hipLaunchKernelGGL((split_forward_kernel<T, TA, LMAX, kTrans, true>), dim3(grid + more), dim3(kThreads), 0, stream, tile0, grid,
                           n, k_red, k_cols, x, w, y, *ride);
        ride->ranges = 0;
        return;
      }
    }
    hipLaunchKernelGGL((split_forward_kernel<T, TA, LMAX, kTrans, false>), dim3(grid), dim3(kThreads), 0, stream, tile0, grid, n, k_red,
                       k_cols, x, w, y, RangeSum<T>{});
  });
}

template <typename T, int LMAX, bool kTrans>
hipError_t forward_l(int64_t n, int k_red, int k_cols, const void* X, const void* W, void* Y, RangeSum<T>* ride, hipStream_t stream) {
  if constexpr (sizeof(T) == 4 && LMAX == 3) {
    if (bf16_parts_ok(sizeof(T), LMAX, n, k_red, k_cols)) {
      const int groups = k_cols / 128;
      if constexpr (!kTrans) {
        if (pair_pays(n, k_red, k_cols)) {
          hipLaunchKernelGGL(mfma_forward_bf16_pair_kernel, dim3(static_cast<unsigned>((n + 15) / 16 * groups)), dim3(kSplitThreads), 0, stream,
                             n, k_red, k_cols, static_cast<const float*>(X), static_cast<const float*>(W), static_cast<float*>(Y));
          return hipGetLastError();
        }
      }
      const int64_t ranges = std::min<int64_t>((n + 15) / 16, std::max(1, compute_units() / groups));
      RangeSum<float> sum{};
      if (kTrans && ride) std::swap(sum, *ride);
      hipLaunchKernelGGL((mfma_forward_bf16_kernel<kTrans>), dim3(static_cast<unsigned>(ranges * groups)), dim3(kSplitThreads), 0, stream,
                         n, k_red, k_cols, static_cast<const float*>(X), static_cast<const float*>(W), static_cast<float*>(Y), sum);
      return hipGetLastError();
    }
  }
  if (mfma_forward_ok(k_red, k_cols) && (kTrans || split_small(sizeof(T), n, k_cols)))
    return launch_split<T, T, LMAX, kTrans>(n, k_red, k_cols, X, W, Y, ride, stream);
  // The tiled kernels below read B operands along rows of W (the backward hands them W transposed).
  if constexpr (!kTrans) {
    if (mfma_forward_ok(k_red, k_cols)) {
      const int64_t tiles = (n + 15) / 16;
      const unsigned grid = static_cast<unsigned>(std::min<int64_t>(tiles, compute_units()));
      // (the LDS-staged kernel addresses W through a buffer descriptor: its bytes must fit 31 bits)
      if (sizeof(T) == 4 && LMAX == 3 && k_cols % 128 == 0 && static_cast<int64_t>(k_red) * k_cols < (int64_t(1) << 26)) {
        if constexpr (sizeof(T) == 4 && LMAX == 3) {   // the LDS-staged variant: two workgroups fit a CU
          const int64_t units = tiles * (k_cols / 128);
          const unsigned grid2 = static_cast<unsigned>(std::min<int64_t>(units, 2 * compute_units()));
          hipLaunchKernelGGL(mfma_forward_lds_kernel, dim3(grid2), dim3(kThreads), 0, stream, n, k_red, k_cols,
                             static_cast<const float*>(X), static_cast<const float*>(W), static_cast<float*>(Y));
        }
      } else if (sizeof(T) == 4 && k_cols % 128 == 0) {
        // two column tiles at a time when the accumulators fit (fp32 and at least two tiles per wave)
        hipLaunchKernelGGL((mfma_forward_kernel<T, LMAX, 2>), dim3(grid), dim3(kThreads), 0, stream, n, k_red, k_cols,
                           static_cast<const T*>(X), static_cast<const T*>(W), static_cast<T*>(Y));
      } else {
        hipLaunchKernelGGL((mfma_forward_kernel<T, LMAX, 1>), dim3(grid), dim3(kThreads), 0, stream, n, k_red, k_cols,
                           static_cast<const T*>(X), static_cast<const T*>(W), static_cast<T*>(Y));
      }
      return hipGetLastError();
    }
  }
  if (few_channels(LMAX, k_red, k_cols))
    return for_all_tiles((n * k_cols + kThreads - 1) / kThreads, kThreads, [&](int64_t block0, unsigned grid) {
      hipLaunchKernelGGL((few_channels_kernel<T, LMAX, kTrans>), dim3(grid), dim3(kThreads), 0, stream, block0, n, k_red,
                         k_cols, static_cast<const T*>(X), static_cast<const T*>(W), static_cast<T*>(Y));
    });
  return launch_split<T, double, LMAX, kTrans>(n, k_red, k_cols, X, W, Y, nullptr, stream);
}

template <typename T, bool kTrans>
hipError_t forward_t(int l_max, int64_t n, int k_red, int k_cols, const void* X, const void* W, void* Y, RangeSum<T>* ride,
                     hipStream_t stream) {
  switch (l_max) {
    case 0: return forward_l<T, 0, kTrans>(n, k_red, k_cols, X, W, Y, ride, stream);
    case 1: return forward_l<T, 1, kTrans>(n, k_red, k_cols, X, W, Y, ride, stream);
    case 2: return forward_l<T, 2, kTrans>(n, k_red, k_cols, X, W, Y, ride, stream);
    default: return forward_l<T, 3, kTrans>(n, k_red, k_cols, X, W, Y, ride, stream);
  }
}

// The partial dW of the tiled kernels; returns in *sum what is left to add.
template <typename T, int LMAX>
hipError_t partial_dw_l(const el_config* cfg, int64_t n, const void* X, const void* dY, void* dW, void* ws, const Transpose<T>& tr,
                        RangeSum<T>* sum, hipStream_t stream) {
  const int per = nodes_per_range(cfg, n);
  const int ranges = static_cast<int>((n + per - 1) / per);
  *sum = RangeSum<T>{static_cast<const T*>(ws), static_cast<T*>(dW), static_cast<int64_t>(LMAX + 1) * cfg->k_in * cfg->k_out, ranges};
  if constexpr (sizeof(T) == 4 && LMAX == 3) {
    if (dw_lds_ok(cfg)) {
      const unsigned grid = static_cast<unsigned>(static_cast<int64_t>(ranges) * (cfg->k_in / kDwIn) * (cfg->k_out / kDwOut));
      hipLaunchKernelGGL(mfma_dw_lds_kernel, dim3(grid + tr.blocks), dim3(kDwRingThreads), 0, stream, n, per, cfg->k_in, cfg->k_out,
                         static_cast<const float*>(X), static_cast<const float*>(dY), static_cast<float*>(ws), tr);
      return hipGetLastError();
    }
  }
  // column tiles per workgroup: the accumulators (orders x tiles x 4 values) must fit the registers
  constexpr int NT = sizeof(T) == 4 ? 4 : 2;
  const unsigned grid = static_cast<unsigned>(static_cast<int64_t>(ranges) * (cfg->k_in / 64) * (cfg->k_out / (16 * NT)));
  hipLaunchKernelGGL((mfma_dw_kernel<T, LMAX, NT>), dim3(grid + tr.blocks), dim3(kThreads), 0, stream, n, per, cfg->k_in,
                     cfg->k_out, static_cast<const T*>(X), static_cast<const T*>(dY), static_cast<T*>(ws), tr);
  return hipGetLastError();
}

template <typename T>
hipError_t partial_dw(const el_config* cfg, int64_t n, const void* X, const void* dY, void* dW, void* ws, const Transpose<T>& tr,
                      RangeSum<T>* sum, hipStream_t stream) {
  switch (cfg->l_max) {
    case 0: return partial_dw_l<T, 0>(cfg, n, X, dY, dW, ws, tr, sum, stream);
    case 1: return partial_dw_l<T, 1>(cfg, n, X, dY, dW, ws, tr, sum, stream);
    case 2: return partial_dw_l<T, 2>(cfg, n, X, dY, dW, ws, tr, sum, stream);
    default: return partial_dw_l<T, 3>(cfg, n, X, dY, dW, ws, tr, sum, stream);
  }
}

// Is the backward one launch of split_backward_kernel?  Its workgroups all have a place at once and each lasts as long as its chain: the
// atoms in the four waves of a tile of dW, k_out in those of a tile of dX.  Of two launches (the tiled partial dW with 13 us for its first rows
// alone, or split_dw_kernel; then dX) each would have its own chain.  So the atoms are limited by the chain, atoms x tiles of dW by the places.
// Backward, us, two launches / one:
//   fp32   128 -> 128    40 atoms 24.0 / 13.5   300 26.2 / 17.4   500 28.0 / 21.8   800 32 / 36
//          192 -> 128    400 26.2 / 24.9        500 27.1 / 28.9 (the limit of atoms)
//          256 -> 256    40 31.7 / 20.6         160 35.9 / 26.2   250 40.6 / 39.4   300 40 / 49 (beyond the limit of places)
//          64 -> 64      300 18.0 / 10.2        l_max = 1, 128 -> 128  300 10.6 / 7.8   500 11.2 / 11.1
//   fp64   128 -> 128    160 34.2 / 19.5        300 35.3 / 28.6   400 36.7 / 38.8
// and for channel counts whose dW is not tiled:
//   fp32   96 -> 96      300 20.7 / 14.0        800 36.6 / 27.2   2000 71 / 101
//          100 -> 128    l_max = 2  800 30.4 / 22.2   2000 61 / 62        fp64, 96 -> 96  800 84.6 / 56.3
bool backward_together(const el_config* cfg, int64_t n) {
  if (few_channels(cfg->l_max, cfg->k_out, cfg->k_in)) return false;
  const int64_t tiles = static_cast<int64_t>((cfg->k_in + 15) / 16) * ((cfg->k_out + 15) / 16);
  if (!mfma_dw_ok(cfg)) return n <= 1024 && n * tiles <= 60000;
  return cfg->dtype == SC_F64 ? n <= 320 && n * tiles <= 24000 : n <= 448 && n * tiles <= 48000;
}

template <typename T, typename TA, int LMAX>
hipError_t launch_together(const el_config* cfg, int64_t n, const T* X, const T* W, const T* dY, T* dX, T* dW, hipStream_t stream) {
  const unsigned dw_tiles = static_cast<unsigned>(((cfg->k_in + 15) / 16 * ((cfg->k_out + 15) / 16) + kXcds - 1) / kXcds * kXcds);
  const unsigned dx_tiles = static_cast<unsigned>(((n + 15) / 16 * ((cfg->k_in + 15) / 16) + kXcds - 1) / kXcds * kXcds);
  hipLaunchKernelGGL((split_backward_kernel<T, TA, LMAX>), dim3(dx_tiles + (LMAX + 1) * dw_tiles), dim3(kThreads), 0, stream, dx_tiles,
                     dw_tiles, n, cfg->k_in, cfg->k_out, X, W, dY, dX, dW);
  return hipGetLastError();
}

template <typename T, int LMAX>
hipError_t together_l(const el_config* cfg, int64_t n, const void* X, const void* W, const void* dY, void* dX, void* dW, hipStream_t stream) {
  const T *x = static_cast<const T*>(X), *w = static_cast<const T*>(W), *dy = static_cast<const T*>(dY);
  T *dx = static_cast<T*>(dX), *dw = static_cast<T*>(dW);
  if (mfma_forward_ok(cfg->k_out, cfg->k_in)) return launch_together<T, T, LMAX>(cfg, n, x, w, dy, dx, dw, stream);
  return launch_together<T, double, LMAX>(cfg, n, x, w, dy, dx, dw, stream);
}

template <typename T>
hipError_t together_t(const el_config* cfg, int64_t n, const void* X, const void* W, const void* dY, void* dX, void* dW, hipStream_t stream) {
  switch (cfg->l_max) {
    case 0: return together_l<T, 0>(cfg, n, X, W, dY, dX, dW, stream);
    case 1: return together_l<T, 1>(cfg, n, X, W, dY, dX, dW, stream);
    case 2: return together_l<T, 2>(cfg, n, X, W, dY, dX, dW, stream);
    default: return together_l<T, 3>(cfg, n, X, W, dY, dX, dW, stream);
  }
}

// Does an output lie on an input?  With two launches dX may take X's place (tiled channel counts: dW has been summed over X by then), and dW that
// of W where the launch of dX reads W transposed; in one launch the workgroups that write either run beside those that still read.
bool written_in_place(const el_config* cfg, int64_t n, const void* X, const void* W, const void* dY, const void* dX, const void* dW) {
  const size_t row = static_cast<size_t>(n) * (cfg->l_max + 1) * (cfg->l_max + 1) * elem_size(cfg);
  const size_t x = row * cfg->k_in, y = row * cfg->k_out, w = static_cast<size_t>(cfg->l_max + 1) * cfg->k_in * cfg->k_out * elem_size(cfg);
  auto overlap = [](const void* p, size_t p_bytes, const void* q, size_t q_bytes) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
    return a < b + q_bytes && b < a + p_bytes;
  };
  return overlap(dX, x, X, x) || overlap(dX, x, W, w) || overlap(dX, x, dY, y) || overlap(dW, w, X, x) || overlap(dW, w, W, w) || overlap(dW, w, dY, y);
}

// Workspace: [ W transposed, rounded up to 256 bytes ][ partial dW per range of atoms ].
size_t wt_bytes(const el_config* cfg) {
  if (!mfma_forward_ok(cfg->k_out, cfg->k_in)) return 0;   // split_forward_kernel reads W as it is
  const size_t bytes = static_cast<size_t>(cfg->l_max + 1) * cfg->k_in * cfg->k_out * elem_size(cfg);
  return (bytes + 255) / 256 * 256;
}

size_t workspace_bytes(const el_config* cfg, int64_t n) {
  if (n == 0) return 256;
  size_t bytes = wt_bytes(cfg);
  if (mfma_dw_ok(cfg)) {
    const int per = nodes_per_range(cfg, n);
    const int64_t ranges = (n + per - 1) / per;
    bytes += static_cast<size_t>(ranges) * (cfg->l_max + 1) * cfg->k_in * cfg->k_out * elem_size(cfg);
  }
  return (bytes + 255) / 256 * 256 + 256;
}

// dX = dY times W transposed: reduction over the output channels, columns = input channels.  Beyond the smallest
// batches the kernels take W transposed once into the workspace (strided B operands cost a third more time for the fp32
// and fp64 instructions; the kernel of the bfloat16 parts reads W as it is).  With the tiled dW two launches: the partial dW
// and W transposed, then dX and the sum of the partial dW.  Backward, us, with a launch for each -> with two: 128 -> 128 channels, 40
// atoms 26.8 -> 25.1, 1000 41.3 -> 33.3, 10 000 120.3 -> 115.8, 16 384 170.8 -> 170.2; 64 -> 64, 1500 atoms 30.6 -> 24.5; l_max = 1,
// 256 -> 128, 300 atoms 17.4 -> 11.6; fp64 128 -> 128, 4000 atoms 206 -> 192.
template <typename T>
hipError_t backward_t(const el_config* cfg, int64_t n, const void* X, const void* W, const void* dY, void* dX, void* dW, void* ws,
                      hipStream_t stream) {
  if (backward_together(cfg, n) && !written_in_place(cfg, n, X, W, dY, dX, dW)) return together_t<T>(cfg, n, X, W, dY, dX, dW, stream);
  const bool transposed = mfma_forward_ok(cfg->k_out, cfg->k_in) && !dx_reads_w_as_is(n, cfg->k_in) && !dx_parts_read_w_as_is(cfg, n);
  Transpose<T> tr{static_cast<const T*>(W), static_cast<T*>(ws), cfg->l_max + 1, cfg->k_in, cfg->k_out, 0};
  if (transposed) {                            // about a thousand elements a workgroup
    const int64_t elems = static_cast<int64_t>(cfg->l_max + 1) * cfg->k_in * cfg->k_out;
    tr.blocks = static_cast<int>(std::min<int64_t>((elems + 8191) / 8192 * 8, 2048));
  }
  auto dx = [&](RangeSum<T>* ride) {
    return transposed ? forward_t<T, false>(cfg->l_max, n, cfg->k_out, cfg->k_in, dY, ws, dX, ride, stream)
                      : forward_t<T, true>(cfg->l_max, n, cfg->k_out, cfg->k_in, dY, W, dX, ride, stream);
  };
  if (mfma_dw_ok(cfg)) {
    RangeSum<T> sum{};
    hipError_t e = partial_dw<T>(cfg, n, X, dY, dW, static_cast<char*>(ws) + wt_bytes(cfg), tr, &sum, stream);
    if (e != hipSuccess) return e;
    e = dx(&sum);
    if (e != hipSuccess || sum.ranges == 0) return e;
    hipLaunchKernelGGL((dw_reduce_kernel<T>), dim3(static_cast<unsigned>(std::min<int64_t>((sum.elems + sum.kSlice - 1) / sum.kSlice, 1 << 16))),
                       dim3(256), 0, stream, sum);
    return hipGetLastError();
  }
  if (transposed) {
    hipLaunchKernelGGL((transpose_w_kernel<T>), dim3(tr.blocks), dim3(256), 0, stream, tr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const hipError_t e = dx(nullptr);
  if (e != hipSuccess) return e;
  const int64_t tiles = static_cast<int64_t>((cfg->k_in + 15) / 16) * ((cfg->k_out + 15) / 16);
  return for_all_tiles(tiles, kDwWaves * kLanes, [&](int64_t tile0, unsigned grid) {
    hipLaunchKernelGGL((split_dw_kernel<T>), dim3(grid, cfg->l_max + 1), dim3(kDwWaves * kLanes), 0, stream, tile0, n, cfg->l_max,
                       cfg->k_in, cfg->k_out, static_cast<const T*>(X), static_cast<const T*>(dY), static_cast<T*>(dW));
  });
}

}  // namespace
}  // namespace el

extern "C" {

sc_status el_forward(const el_config* cfg, int64_t n_nodes, const void* X, const void* W, void* Y, void* hip_stream) {
  using namespace el;
  sc_status st = check_config("el_forward", cfg, n_nodes);
  if (st != SC_OK) return st;
  if (n_nodes == 0) return SC_OK;
  if (!X || !W || !Y) return set_error(SC_ERR_INVALID_ARG, "el_forward: NULL tensor argument");
  if (misaligned(X, 16) || misaligned(W, 16) || misaligned(Y, 16))
    return set_error(SC_ERR_INVALID_ARG, "el_forward: tensor pointer not 16-byte aligned");
  DeviceGuard guard(cfg->device);
  if (!guard.ok) return set_error(SC_ERR_HIP, "el_forward: cannot make cfg->device current");
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const hipError_t e = cfg->dtype == SC_F64
                           ? forward_t<double, false>(cfg->l_max, n_nodes, cfg->k_in, cfg->k_out, X, W, Y, nullptr, stream)
                           : forward_t<float, false>(cfg->l_max, n_nodes, cfg->k_in, cfg->k_out, X, W, Y, nullptr, stream);
  if (e != hipSuccess) return set_error(SC_ERR_HIP, std::string("el_forward: kernel launch: ") + hipGetErrorString(e));
  return SC_OK;
}

sc_status el_workspace_bytes(const el_config* cfg, int64_t n_nodes, size_t* bytes) {
  using namespace el;
  sc_status st = check_config("el_workspace_bytes", cfg, n_nodes);
  if (st != SC_OK) return st;
  if (!bytes) return set_error(SC_ERR_INVALID_ARG, "el_workspace_bytes: bytes is NULL");
  *bytes = workspace_bytes(cfg, n_nodes);
  return SC_OK;
}

sc_status el_backward(const el_config* cfg, int64_t n_nodes, const void* X, const void* W, const void* dY, void* dX,
                      void* dW, void* workspace, size_t workspace_bytes_given, void* hip_stream) {
  using namespace el;
  sc_status st = check_config("el_backward", cfg, n_nodes);
  if (st != SC_OK) return st;
  if (!dW) return set_error(SC_ERR_INVALID_ARG, "el_backward: dW is NULL");
  if (misaligned(dW, 16)) return set_error(SC_ERR_INVALID_ARG, "el_backward: dW not 16-byte aligned");
  DeviceGuard guard(cfg->device);
  if (!guard.ok) return set_error(SC_ERR_HIP, "el_backward: cannot make cfg->device current");
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (n_nodes == 0) {
    const size_t words = elem_size(cfg) / 4 * static_cast<size_t>(cfg->l_max + 1) * cfg->k_in * cfg->k_out;
    hipLaunchKernelGGL(zero_kernel, dim3(64), dim3(256), 0, stream, static_cast<unsigned int*>(dW), words);
    const hipError_t e0 = hipGetLastError();
    if (e0 != hipSuccess) return set_error(SC_ERR_HIP, std::string("el_backward: fill launch: ") + hipGetErrorString(e0));
    return SC_OK;
  }
  if (!X || !W || !dY || !dX) return set_error(SC_ERR_INVALID_ARG, "el_backward: NULL tensor argument");
  if (misaligned(X, 16) || misaligned(W, 16) || misaligned(dY, 16) || misaligned(dX, 16))
    return set_error(SC_ERR_INVALID_ARG, "el_backward: tensor pointer not 16-byte aligned");
  if (!workspace || workspace_bytes_given < workspace_bytes(cfg, n_nodes))
    return set_error(SC_ERR_WORKSPACE, "el_backward: workspace missing or smaller than el_workspace_bytes()");
  if (misaligned(workspace, 256)) return set_error(SC_ERR_WORKSPACE, "el_backward: workspace not 256-byte aligned");
  const hipError_t e = cfg->dtype == SC_F64 ? backward_t<double>(cfg, n_nodes, X, W, dY, dX, dW, workspace, stream)
                                            : backward_t<float>(cfg, n_nodes, X, W, dY, dX, dW, workspace, stream);
  if (e != hipSuccess) return set_error(SC_ERR_HIP, std::string("el_backward: kernel launch: ") + hipGetErrorString(e));
  return SC_OK;
}

}  // extern "C"
