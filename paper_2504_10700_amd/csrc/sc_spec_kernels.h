// Skeleton of the specialised kernels: hand-written memory / scheduling skeleton around generated
// straight-line arithmetic (csrc/generated/*.inc, written by codegen/generate.py).
//
// Mapping (Algorithm 2 of arXiv 2504.10700 is independent per atom and channel):
//   lane      = channel (64 consecutive channels per wave: the A row of a node is read as
//               64 B per lane, a wave covers 4 KB of contiguous HBM; B/dB rows are 16 B per lane)
//   forward   workgroup = 4 waves = a tile of consecutive nodes of the batch x one 64-channel
//               block; a wave visits its share of the nodes grouped by element and reads the
//               folded weights of a run once
//   backward, second-order pass
//             workgroup = 4 waves = one tile of the grouping (nodes of ONE element) x one
//               64-channel block, the element's folded weights in registers; its waves add their
//               dW' rows through LDS, so one partial row set leaves per tile; the grid is
//               remapped so that each XCD (own L2) gets a contiguous range of tiles
// Per node the next node's rows are requested before the current one is evaluated
// (two register sets, ping-pong), so HBM latency hides behind ~300-800 VALU operations.
// kCM instances of the forward and backward kernels serve the component-major layout
// ([node][component][channel], SC_COMPONENT_MAJOR): same mapping and arithmetic, rows accessed
// through Cols instead of Row.
//
// One step (forward + backward of one batch) is four launches:
//   1 prepare   the weights of every (element, channel) folded into the internal basis once,
//               wf[element][channel block][kS][64]; other workgroups of the same launch count the
//               elements of z (first half of the grouping) and, for larger batches, order every
//               window of 1024 nodes by element (the order of the forward's visits)
//   2 forward   nodes in batch order, inside a window by element (no grouping needed: every node
//               reads the folded weights of its element from wf, which stays in L2, once per run
//               of an element): consecutive workgroups stream the same stretch of memory.  Other
//               workgroups of the same launch finish the grouping (scatter + tile table), which
//               only the backward needs
//   3 backward  nodes grouped by element (tiles), weights of the tile's element in registers,
//               dW' summed per tile without atomics
//   4 finalize  per (element, channel block): sum of the per-tile dW' rows in a fixed order
//               (fp64) and the map to the external paths
//
// Arguments.  The first 14 words of a kernel's arguments (scalars and pointers, up to the first structure) come with the wave in
// scalar registers (-amdgpu-kernarg-preload-count); the rest it loads, which is one memory latency at the head of every launch.
// So what the head of a kernel needs stands first: sizes, the tile table, the order of the nodes.  Before / with, us a step,
// 128 channels, 0e+1o: 3072 atoms 32.4 / 31.0, 10 000 74.7 / 72.8 (bfloat16 rows 56.4 / 55.2), 2731 atoms of l_max = 2 in
// fp64 31.7 / 30.6; from 50 000 atoms on no difference.
//
// Included by the files that hold the generated programs; each makes table entries of them (Entry below).
#pragma once
#include <type_traits>

#include "sc_group_split.h"
#include "sc_spec.h"

namespace sc {
namespace {

// what the generated programs call
__device__ __forceinline__ float sc_fma(float x, float y, float z) { return __builtin_fmaf(x, y, z); }
__device__ __forceinline__ double sc_fma(double x, double y, double z) { return __builtin_fma(x, y, z); }

constexpr int kSpecWaves = 4;
constexpr int kSpecThreads = kSpecWaves * kLanes;
constexpr int kXcds = 8;

__device__ __forceinline__ int wave_of_thread() { return __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes); }

// Row of N elements of T at p (p is aligned to the row size if that is a multiple of 16 B,
// else only to sizeof(T)): 16-byte accesses plus a scalar tail.
template <typename T, int N>
struct Row {
  static constexpr int V = 16 / sizeof(T);
  static constexpr int kAlign = (N * sizeof(T)) % 16 == 0 ? 16 : sizeof(T);
  typedef T Vec __attribute__((ext_vector_type(V), aligned(kAlign)));

  static __device__ __forceinline__ void load(const T* __restrict__ p, T (&v)[N]) {
#pragma unroll
    for (int i = 0; i + V <= N; i += V) {
      const Vec x = *reinterpret_cast<const Vec*>(p + i);
#pragma unroll
      for (int k = 0; k < V; ++k) v[i + k] = x[k];
    }
#pragma unroll
    for (int i = N / V * V; i < N; ++i) v[i] = p[i];
  }
  static __device__ __forceinline__ void store(T* __restrict__ p, const T (&v)[N]) {
#pragma unroll
    for (int i = 0; i + V <= N; i += V) {
      Vec x;
#pragma unroll
      for (int k = 0; k < V; ++k) x[k] = v[i + k];
      // A row of one 16-byte piece makes the wave's store one contiguous KB: streamed past the
      // cache (measured faster).  Longer rows are written by several instructions that each touch
      // a part of every line: left to the L2 to merge (streaming them measured slower).
      if constexpr (N * sizeof(T) == 16) __builtin_nontemporal_store(x, reinterpret_cast<Vec*>(p + i));
      else *reinterpret_cast<Vec*>(p + i) = x;
    }
#pragma unroll
    for (int i = N / V * V; i < N; ++i) p[i] = v[i];
  }
};

// Store of a wave's rows (N elements per lane, lane rows N elements apart = one contiguous
// block of 64*N elements) as fully coalesced instructions: each lane's row goes through an
// LDS block of the same layout and comes back transposed, so that store instruction k
// writes the k-th contiguous 1 KB of the block instead of 64 scattered 16-byte pieces
// (four times fewer, four times larger write requests to L2; measured -10% on the whole
// backward kernel; the same trick on the loads of A gained nothing).  stage: 64*N elements
// of LDS owned by this wave; block: where lane 0's row goes (16-byte aligned); live_lanes: the
// lanes whose rows exist (fewer than 64 in the last channel block of a channel count that is not
// a multiple of 64).
// kStream: non-temporal stores (the rows are not read again soon and each instruction writes
// whole lines).  Measured on one box, library against library: forward 28.4 -> 27.0 us at 10k
// nodes (neutral at 200k), second-order kernel 78.7 -> 77.5 us; a wash for the backward's dA
// at 10k nodes and 1% slower at 200k, so the backward leaves it off.
template <typename T, int N, bool kStream = true>
__device__ __forceinline__ void store_rows_coalesced(T* __restrict__ block, T* stage, int lane, const T (&v)[N],
                                                     int live_lanes = kLanes) {
  constexpr int V = 16 / sizeof(T);
  typedef T Vec __attribute__((ext_vector_type(V)));
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // earlier reads of the stage are done
  __builtin_amdgcn_wave_barrier();
  if constexpr (N % V == 0) {
#pragma unroll
    for (int j = 0; j < N / V; ++j) {
      Vec x;
#pragma unroll
      for (int k = 0; k < V; ++k) x[k] = v[j * V + k];
      *reinterpret_cast<Vec*>(stage + lane * N + j * V) = x;
    }
  } else {  // rows that are not a whole number of 16-byte pieces (e.g. 9 components)
#pragma unroll
    for (int j = 0; j < N; ++j) stage[lane * N + j] = v[j];
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // other lanes' pieces are visible
  __builtin_amdgcn_wave_barrier();
  // 16-byte pieces of the block: 64*N/V of them, fewer if the last channel block is not full
  // (live_lanes * N is a multiple of V: channel counts are multiples of four)
  constexpr int kPieces = kLanes * N / V;
  const int pieces = live_lanes * N / V;
#pragma unroll
  for (int q0 = 0; q0 < kPieces; q0 += kLanes) {
    const int q = q0 + lane;
    if ((live_lanes == kLanes && q0 + kLanes <= kPieces) || q < pieces) {   // the first test is a constant for full blocks
      const Vec x = *reinterpret_cast<const Vec*>(stage + q * V);
      if constexpr (kStream) __builtin_nontemporal_store(x, reinterpret_cast<Vec*>(block + q * V));
      else *reinterpret_cast<Vec*>(block + q * V) = x;
    }
  }
}

// Storage type TS of the per-node rows (A, B, dB, dA, H, ...) when it differs from the arithmetic
// type T: bfloat16 (SC_BF16: rows in bfloat16, arithmetic, weights and dW in fp32) or fp32 under
// fp64 arithmetic (Types below).  Widening is exact, narrowing rounds to nearest, ties to even (the
// chip's own conversion instructions).
typedef __bf16 bf16_bits;

// Rows of N elements stored as TS, handled as T.  TS == T is Row<T, N> itself.
template <typename T, typename TS, int N>
struct RowIO {
  typedef TS Vec8 __attribute__((ext_vector_type(N * sizeof(TS) == 8 ? N : 2), aligned(8)));   // an 8-byte row in one access
  static __device__ __forceinline__ void load(const TS* __restrict__ p, T (&v)[N]) {
    TS raw[N];
    if constexpr (N * sizeof(TS) == 8) {
      const Vec8 x = *reinterpret_cast<const Vec8*>(p);
#pragma unroll
      for (int i = 0; i < N; ++i) raw[i] = x[i];
    } else {
      Row<TS, N>::load(p, raw);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = static_cast<T>(raw[i]);
  }
  static __device__ __forceinline__ void store(TS* __restrict__ p, const T (&v)[N]) {
    TS raw[N];
#pragma unroll
    for (int i = 0; i < N; ++i) raw[i] = static_cast<TS>(v[i]);
    if constexpr (N * sizeof(TS) == 8) {
      Vec8 x;
#pragma unroll
      for (int i = 0; i < N; ++i) x[i] = raw[i];
      *reinterpret_cast<Vec8*>(p) = x;
    } else {
      Row<TS, N>::store(p, raw);
    }
  }
};
template <typename T, int N>
struct RowIO<T, T, N> : Row<T, N> {};

// Component-major rows (SC_COMPONENT_MAJOR: tensors laid out [node][component][channel]): the N
// components of one (node, channel) lie K elements apart, and a wave's access to one component
// covers 64 consecutive channels - coalesced as it is, loads and stores alike, so nothing passes
// through LDS.  p points at component 0 of the lane's channel.
template <typename T, int N>
struct Cols {
  static __device__ __forceinline__ void load(const T* __restrict__ p, int K, T (&v)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = p[static_cast<size_t>(i) * K];
  }
  template <bool kStream>
  static __device__ __forceinline__ void store(T* __restrict__ p, int K, const T (&v)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if constexpr (kStream) __builtin_nontemporal_store(v[i], p + static_cast<size_t>(i) * K);
      else p[static_cast<size_t>(i) * K] = v[i];
    }
  }
};

// store_rows_coalesced for rows stored as TS; `stage` is this wave's LDS block of 64*N elements of T
// (large enough for TS, which is never wider).
template <typename T, typename TS, int N, bool kStream>
struct RowsOut {
  static __device__ __forceinline__ void store(TS* __restrict__ block, T* stage, int lane, const T (&v)[N], int live_lanes) {
    TS raw[N];
#pragma unroll
    for (int i = 0; i < N; ++i) raw[i] = static_cast<TS>(v[i]);
    store_rows_coalesced<TS, N, kStream>(block, reinterpret_cast<TS*>(stage), lane, raw, live_lanes);
  }
};
template <typename T, int N, bool kStream>
struct RowsOut<T, T, N, kStream> {
  static __device__ __forceinline__ void store(T* __restrict__ block, T* stage, int lane, const T (&v)[N], int live_lanes) {
    store_rows_coalesced<T, N, kStream>(block, stage, lane, v, live_lanes);
  }
};
#define store_rows_as RowsOutCall
template <typename T, typename TS, int N, bool kStream = true>
__device__ __forceinline__ void RowsOutCall(TS* __restrict__ block, T* stage, int lane, const T (&v)[N],
                                            int live_lanes = kLanes) {
  RowsOut<T, TS, N, kStream>::store(block, stage, lane, v, live_lanes);
}

// blockIdx -> logical work item such that the blocks an XCD receives (round-robin by
// blockIdx) form one contiguous range.  gridDim.x is a multiple of kXcds.
__device__ __forceinline__ int xcd_contiguous_block() {
  const int per = gridDim.x / kXcds;
  return (blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
}

// Folded weights: wf[element][channel block][kS][64 channels]: every internal row of an
// (element, channel block) is 256 contiguous bytes (fp32), so a wave reads it with one fully
// coalesced instruction.  (Rows per lane - [element][channel][kS] read as 16-byte pieces - make
// every load instruction touch 64 cache lines; with the weights read per node that bound the
// natural-order forward by the tag rate of the vector cache: 614 us instead of 440 at 200k nodes.)
template <typename T, typename G>
__device__ __forceinline__ void load_folded(const T* __restrict__ wf, int z, int chblocks, int cb, int lane,
                                            T (&w)[G::kS]) {
  const T* src = wf + (static_cast<size_t>(z) * chblocks + cb) * G::kS * kLanes + lane;
#pragma unroll
  for (int s = 0; s < G::kS; ++s) w[s] = src[s * kLanes];
}

// The internal rows kPart, kPart + kParts, ... of one (element, 64 channels): what they need is requested before the first
// value is used (one memory latency, not one per few rows); what belongs to other rows is not computed.
template <typename T, typename G, typename TW, int kPart, int kParts>
__device__ __forceinline__ void fold_part(const TW* __restrict__ src, int K, T* __restrict__ dst) {
  T w[G::kS];
  TW wz[G::kP];
#pragma unroll
  for (int p = 0; p < G::kP; ++p) wz[p] = src[static_cast<size_t>(p) * K];
  asm volatile("" ::: "memory");
  G::fold(wz, 1, w);
#pragma unroll
  for (int s = kPart; s < G::kS; s += kParts) dst[s * kLanes] = w[s];
}

// The fold role folds W[element, :, 64 channels] into wf, a workgroup per such pair and a quarter of the rows per wave: bound by one memory
// latency and by what one compute unit can request.  A wave for all rows, four pairs a workgroup (45 of the 256 units at 89 elements, 128
// channels) -> this, us a launch: 0e+1o, 3072 nodes 4.1 -> 2.9; l_max = 2 in fp64, 2731 nodes 4.1 -> 2.9; 10 000 nodes, whose launch waits for
// memory that has left the caches, 5.3 either way.
// kWaves = 1: a wave for all rows, for the launches that also evaluate, with the few rows of a small basis: there the workgroups of this
// role stand before those of the nodes, and fewer of them hold those up less.  us, four waves / one: l_max = 2 in fp64 1398 nodes 7.7 / 7.3, 2000
// 8.1 / 7.8; l_max = 3, nu = 2, 0e in fp32 2000 7.7 / 7.5; the 86 rows of 0e+1o 2000 9.1 / 9.2, 0e+1o+2e 9.8 / 10.8.
template <typename G>
constexpr int direct_fold_waves() { return G::kP > 64 ? kSpecWaves : 1; }

template <typename T, typename G, typename TW, int kWaves>
__device__ __forceinline__ void fold_role(int wg, int Z, int K, int chblocks, const TW* __restrict__ W, T* __restrict__ wf) {
  static_assert(kSpecWaves == 4 && (kWaves == 1 || kWaves == 4), "a part per wave");
  const int lane = threadIdx.x & (kLanes - 1), wave = wave_of_thread();
  const int pair = kWaves == 1 ? wg * kSpecWaves + wave : wg;
  if (pair >= Z * chblocks) return;
  const int z = pair / chblocks, cb = pair % chblocks;   // pair = element * chblocks + channel block
  const int live = K - cb * kLanes < kLanes ? K - cb * kLanes : kLanes;
  const int ch = cb * kLanes + (lane < live ? lane : live - 1);   // dead lanes repeat the last channel
  const TW* src = W + static_cast<size_t>(z) * G::kP * K + ch;
  T* dst = wf + static_cast<size_t>(pair) * G::kS * kLanes + lane;
  if constexpr (kWaves == 1) return fold_part<T, G, TW, 0, 1>(src, K, dst);
  switch (wave) {
    case 0: return fold_part<T, G, TW, 0, kSpecWaves>(src, K, dst);
    case 1: return fold_part<T, G, TW, 1, kSpecWaves>(src, K, dst);
    case 2: return fold_part<T, G, TW, 2, kSpecWaves>(src, K, dst);
    default: return fold_part<T, G, TW, 3, kSpecWaves>(src, K, dst);
  }
}

// Launch 1.  Workgroups [0, window_wgs): window role (order of the forward pass); the next
// count_wgs: count role of the grouping.  The others: fold role.
template <typename T, typename G, typename TW>
__global__ __launch_bounds__(kSpecThreads) void spec_prepare_kernel(const int32_t* __restrict__ z, int n, int Z, int window_wgs,
                                                                    int count_wgs, const TW* __restrict__ W, T* __restrict__ wf,
                                                                    int K, int chblocks, SplitGroupArgs ga) {
  extern __shared__ unsigned char lds_raw[];
  ga.z = z;
  ga.n = n;
  ga.Z = Z;
  if (static_cast<int>(blockIdx.x) < window_wgs) {   // the longest role first
    split_window_role(ga, blockIdx.x, reinterpret_cast<int32_t*>(lds_raw));
    return;
  }
  if (static_cast<int>(blockIdx.x) < window_wgs + count_wgs) {
    split_count_role(ga, blockIdx.x - window_wgs, reinterpret_cast<int32_t*>(lds_raw));
    return;
  }
  fold_role<T, G, TW, kSpecWaves>(static_cast<int>(blockIdx.x) - window_wgs - count_wgs, Z, K, chblocks, W, wf);
}

// The grouping alone (a backward pass that cannot reuse a forward's grouping): scatter and table roles.
__global__ __launch_bounds__(kSpecThreads) void spec_scatter_kernel(SplitGroupArgs ga, int scatter_wgs) {
  extern __shared__ unsigned char lds_raw[];
  if (static_cast<int>(blockIdx.x) < scatter_wgs) split_scatter_role(ga, blockIdx.x, reinterpret_cast<int32_t*>(lds_raw));
  else split_table_role(ga, reinterpret_cast<int32_t*>(lds_raw));
}

// Launch 2.  Workgroups [0, scatter_wgs): scatter role; the next `table` (0 or 1): table role;
// the others: forward of `tile` consecutive nodes x one 64-channel block, a
// contiguous quarter of the nodes per wave.  A node whose element index is outside [0, Z) is
// skipped (its row of B is left untouched), as the grouped kernels do.
// kDirect: the weights of a run are folded from W (external paths) by the wave itself instead of
// being read from the folded table, so that no launch has to come before this one.
template <typename T, typename G, typename TS, typename TW, bool kCM, bool kDirect>
__global__ __launch_bounds__(kSpecThreads) void spec_forward_kernel(const int32_t* __restrict__ wnode,
                                                                    const int32_t* __restrict__ elements, int scatter_wgs,
                                                                    int table, int chblocks, int tile, int n, int Z, int K,
                                                                    int fold_wgs, const TS* __restrict__ A,
                                                                    const T* __restrict__ wf, const TW* __restrict__ W,
                                                                    TS* __restrict__ B, SplitGroupArgs ga) {
  extern __shared__ unsigned char lds_raw[];
  int block = blockIdx.x;
  const bool clamp = kDirect && fold_wgs < 0;   // (a word of its own would be one of the first 14 too many)
  if constexpr (kDirect) {   // no launch came before: the roles count for themselves, the fold role is here
    if (block < scatter_wgs + table) {
      int32_t* counts = reinterpret_cast<int32_t*>(lds_raw) + split_group_lds_bytes(Z) / sizeof(int32_t);
      split_count_all(ga, counts);
      ga.counts = counts;
    } else if (block < scatter_wgs + table + fold_wgs) {
      fold_role<T, G, TW, direct_fold_waves<G>()>(block - scatter_wgs - table, Z, K, chblocks, W, const_cast<T*>(wf));   // read by nobody in this launch
      return;
    }
  }
  if (block < scatter_wgs) {
    split_scatter_role(ga, block, reinterpret_cast<int32_t*>(lds_raw));
    return;
  }
  if (block < scatter_wgs + table) {
    split_table_role(ga, reinterpret_cast<int32_t*>(lds_raw));
    return;
  }
  block -= scatter_wgs + table;
  if constexpr (kDirect) block -= clamp ? 0 : fold_wgs;
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = wave_of_thread();
  T* stage = reinterpret_cast<T*>(lds_raw) + wave * kLanes * G::kNLM;  // [64][kNLM] per wave (if used)
  constexpr bool kStageB = G::kNLM * sizeof(TS) != 16;  // 16-byte rows are coalesced as they are
  const int t = block / chblocks, cb = block % chblocks;
  const int s0 = t * tile;
  const int in_tile = (n - s0 < tile) ? n - s0 : tile;
  const int j0 = s0 + in_tile * wave / kSpecWaves, j1 = s0 + in_tile * (wave + 1) / kSpecWaves;
  if (j0 >= j1) return;
  const int live = K - cb * kLanes < kLanes ? K - cb * kLanes : kLanes;   // channels of this block
  const int ch = cb * kLanes + (lane < live ? lane : live - 1);           // dead lanes repeat the last channel
  // This wave's nodes (at most 64: one per lane) are visited grouped by element - a stable sort of
  // their element indices inside the wave - so that a run of nodes of one element reads the
  // folded weights once (they are re-read per node otherwise: 61 of 432 us at 200k nodes).  The
  // indices are read at once, which also takes them off the per-node chain of dependent loads.
  // Nodes with an element index outside [0, Z) sort last and are skipped (clamp: take the nearest element's weights).  (A third row buffer, i.e.
  // the rows of node p+2 requested while node p is evaluated, measured the same at 10k nodes and 3%
  // slower at 200k.)
  // With the window order of the prepare launch (ga.wnode) the wave's positions hold nodes of a
  // 1024-node window that are ordered by element already, so the runs are long: 0.2 instead of 0.8
  // reads of the weights per node with 89 elements of skewed frequency, which is what the forward
  // gains from a batch ordered by element (427 -> 385 us at 200k nodes; the weights are L2 hits, but
  // 2.4 GB of them per launch next to 1.6 GB of A).  The sort inside the wave stays: it moves nodes
  // with an invalid index to the end and joins runs across a window boundary.
  const int cnt = j1 - j0;
  int key = Z, mine = j0 + lane;   // the lane's node and its element index
  if (lane < cnt) {
    const int e = elements[j0 + lane];
    if (wnode) {   // positions follow the window order written by the count role (uniform)
      mine = wnode[j0 + lane];
      mine = mine < 0 ? 0 : (mine >= n ? n - 1 : mine);
    }
    key = (e >= 0 && e < Z) ? e : !clamp ? Z : e < 0 ? 0 : Z - 1;
  }
  int rank = lane;   // lanes past the last node keep their own slot
  if (lane < cnt) rank = 0;
  for (int k = 0; k < cnt; ++k) {   // uniform trip count
    const int zk = __builtin_amdgcn_readlane(key, k);
    if (lane < cnt && (zk < key || (zk == key && k < lane))) ++rank;
  }
  const int order = __builtin_amdgcn_ds_permute(rank << 2, lane);   // order[p] = lane of the node visited p-th
  auto visit = [&](int p, int& node, int& e) {
    const int idx = __builtin_amdgcn_readlane(order, p);
    e = __builtin_amdgcn_readlane(key, idx);
    node = __builtin_amdgcn_readlane(mine, idx);
  };
  // Rows: two register sets in turn (the next node's row is requested before the current node is
  // evaluated).  Weights: ONE register set, reloaded from the folded table (L2) right before a node of
  // another element is evaluated - a second set for prefetching them costs 29-68 registers and with
  // them a wave per SIMD, which hides that latency better than the prefetch does.
  T a0[G::kNlm], a1[G::kNlm], w[G::kS], b[G::kNLM];
  static_assert(!kCM || std::is_same<T, TS>::value, "component-major rows are stored in the arithmetic type");
  auto load_a = [&](int node, T (&a)[G::kNlm]) {
    if constexpr (kCM) Cols<TS, G::kNlm>::load(A + static_cast<size_t>(node) * G::kNlm * K + ch, K, a);
    else RowIO<T, TS, G::kNlm>::load(A + (static_cast<size_t>(node) * K + ch) * G::kNlm, a);
  };
  auto store_b = [&](int node) {
    if constexpr (kCM) {
      if (lane < live) Cols<TS, G::kNLM>::template store<true>(B + static_cast<size_t>(node) * G::kNLM * K + ch, K, b);
    } else if constexpr (kStageB) {
      store_rows_as<T, TS, G::kNLM>(B + (static_cast<size_t>(node) * K + cb * kLanes) * G::kNLM, stage, lane, b, live);
    } else if (lane < live) {
      RowIO<T, TS, G::kNLM>::store(B + (static_cast<size_t>(node) * K + ch) * G::kNLM, b);
    }
  };
  // (The table is read where it is needed and not in here: behind a call the compiler waits for nearly all weights before
  // the arithmetic of a node starts.  Step, us, bfloat16 rows, 128 channels, here / through a call: 10 000 nodes 59.5 / 59.0,
  // 20 000 100.8 / 101.8, 50 000 218 / 221.)
  auto fold_w = [&](int e) {
    TW wz[G::kP];   // all rows are requested before the first is used, as in the prepare launch
    const TW* src = W + static_cast<size_t>(e) * G::kP * K + ch;
#pragma unroll
    for (int q = 0; q < G::kP; ++q) wz[q] = src[static_cast<size_t>(q) * K];
    G::fold(wz, 1, w);
    // finished values here, as where they come from the table: left open, the compiler fuses the fold's last
    // multiplications into the arithmetic of the node, and the bits differ from the table's
#pragma unroll
    for (int i = 0; i < G::kS; ++i) asm volatile("" : "+v"(w[i]));
  };
  // The loop takes two nodes per trip and every load in it is issued without a condition of its
  // own, in a fixed order: the weights of a new element first, then the rows of the next node, then
  // the arithmetic of the current node, which waits for its own operands only.  (A request under
  // a condition makes the compiler wait for ALL outstanding loads at the join, the request just
  // issued included, before the arithmetic it is meant to overlap; the scheduling barrier keeps the
  // compiler from moving the request down into that arithmetic to save registers.)  The last trip
  // of an even share requests its last node's rows once more; an odd share ends with a single node.
  const int valid = __builtin_popcountll(__ballot(key < Z));   // they come first in the visiting order
  if (valid == 0) return;   // no valid node in this wave's share
  int n0, e0, n1, e1, e_w = -1;
  visit(0, n0, e0);
  load_a(n0, a0);
  int p = 0;
  for (; p + 1 < valid; p += 2) {
    if (e0 != e_w) {
      if constexpr (kDirect) fold_w(e0);
      else load_folded<T, G>(wf, e0, chblocks, cb, lane, w);
      e_w = e0;
    }
    visit(p + 1, n1, e1);
    load_a(n1, a1);
    __builtin_amdgcn_sched_barrier(0);
    G::forward(a0, w, b);
    store_b(n0);
    if (e1 != e_w) {
      if constexpr (kDirect) fold_w(e1);
      else load_folded<T, G>(wf, e1, chblocks, cb, lane, w);
      e_w = e1;
    }
    visit(p + 2 < valid ? p + 2 : valid - 1, n0, e0);
    load_a(n0, a0);
    __builtin_amdgcn_sched_barrier(0);
    G::forward(a1, w, b);
    store_b(n1);
  }
  if (p < valid) {
    if (e0 != e_w) {
      if constexpr (kDirect) fold_w(e0);
      else load_folded<T, G>(wf, e0, chblocks, cb, lane, w);
    }
    G::forward(a0, w, b);
    store_b(n0);
  }
}

// kOcc = waves per SIMD the kernel is held to (0: the compiler's choice, which every launch uses now).
// The fp32 kernel of the small basis needs 171 registers if left alone, three over the limit for
// three waves per SIMD; held to 168 (two values go to scratch) it ran three workgroups per CU
// instead of two, which paid while small batches were cut into many equal tiles (51.1 -> 49.3 us
// at 10k nodes).  With tiles processed largest first, as many whole ones as fill two workgroups per CU once,
// the third workgroup is rarely resident, and the unconstrained kernel is faster (step 82.8 -> 80.8
// us at 10k nodes, same box, with tiles a quarter longer than now).
// kStreamDA: the dA rows are streamed past the cache (non-temporal stores), for batches up to
// 40 000 nodes: the kernel itself gains 2 us at 10k nodes and the launches after it another 3 us,
// whereas at 200k nodes the backward loses 2% with them and the next forward gains as much.
// kFull: the channel count is a multiple of 64, no lane is ever idle.  The fp32 kernel of the
// 49-row basis sits at the limit for two waves per SIMD: 250 registers without the idle-lane
// handling, 295 (one wave per SIMD, 736 instead of 496 us at 50k nodes / 256 channels) with it.
template <typename T, typename G, int kOcc = 0, bool kStreamDA = false, bool kFull = false, typename TS = T, bool kCM = false>
__global__ __launch_bounds__(kSpecThreads) __attribute__((amdgpu_waves_per_eu(kOcc == 0 ? 1 : kOcc, 8)))
void spec_backward_kernel(const TileDesc* __restrict__ tiles, int n_blocks, int chblocks, const int32_t* __restrict__ perm, int K,
                          const T* __restrict__ wf, const TS* __restrict__ A, const TS* __restrict__ dB, TS* __restrict__ dA,
                          T* __restrict__ partial) {
  extern __shared__ unsigned char lds_raw[];
  T* red = reinterpret_cast<T*>(lds_raw);  // [kSpecWaves][kS][64]
  T* stage = red + kSpecWaves * G::kS * kLanes + wave_of_thread() * kLanes * G::kNlm;  // [64][kNlm] per wave
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int logical = blockIdx.x;   // descriptors are stored largest tile first: dispatch order is the schedule
  if (logical >= n_blocks) return;  // uniform per workgroup
  const int tile = logical / chblocks, cb = logical % chblocks;
  const TileDesc td = tiles[tile];
  if (td.count == 0) return;        // unused descriptor; uniform per workgroup
  const int j0 = td.start + td.count * wave / kSpecWaves;
  const int j1 = td.start + td.count * (wave + 1) / kSpecWaves;
  const int live = kFull ? kLanes : (K - cb * kLanes < kLanes ? K - cb * kLanes : kLanes);   // channels of this block
  const int ch = cb * kLanes + (lane < live ? lane : live - 1);           // dead lanes repeat the last channel
  T dw[G::kS];
#pragma unroll
  for (int s = 0; s < G::kS; ++s) dw[s] = T(0);
  if (j0 < j1) {
    T w[G::kS];
    load_folded<T, G>(wf, td.z, chblocks, cb, lane, w);
    T a0[G::kNlm], a1[G::kNlm], g0[G::kNLM], g1[G::kNLM], da[G::kNlm];
    static_assert(!kCM || std::is_same<T, TS>::value, "component-major rows are stored in the arithmetic type");
    auto load_rows = [&](size_t node, T (&a)[G::kNlm], T (&g)[G::kNLM]) {
      if constexpr (kCM) {
        Cols<TS, G::kNlm>::load(A + node * G::kNlm * K + ch, K, a);
        Cols<TS, G::kNLM>::load(dB + node * G::kNLM * K + ch, K, g);
      } else {
        RowIO<T, TS, G::kNlm>::load(A + (node * K + ch) * G::kNlm, a);
        RowIO<T, TS, G::kNLM>::load(dB + (node * K + ch) * G::kNLM, g);
      }
    };
    auto store_da = [&](size_t node) {
      if constexpr (kCM) {
        if (kFull || lane < live) Cols<TS, G::kNlm>::template store<kStreamDA>(dA + node * G::kNlm * K + ch, K, da);
      } else {
        store_rows_as<T, TS, G::kNlm, kStreamDA>(dA + (node * K + cb * kLanes) * G::kNlm, stage, lane, da, live);
      }
    };
    size_t node0 = perm ? perm[j0] : j0, node1 = 0;   // no permutation: the batch is already grouped
    load_rows(node0, a0, g0);
    for (int j = j0; j < j1; j += 2) {
      if (j + 1 < j1) {
        node1 = perm ? perm[j + 1] : j + 1;
        load_rows(node1, a1, g1);
      }
      G::backward(a0, w, g0, da, dw);
      store_da(node0);
      if (j + 1 < j1) {
        if (j + 2 < j1) {
          node0 = perm ? perm[j + 2] : j + 2;
          load_rows(node0, a0, g0);
        }
        G::backward(a1, w, g1, da, dw);
        store_da(node1);
      }
    }
  }
  // sum the waves' dW' rows in wave order and write the tile's partial rows
#pragma unroll
  for (int s = 0; s < G::kS; ++s) red[(wave * G::kS + s) * kLanes + lane] = dw[s];
  __syncthreads();
  T* out = partial + (static_cast<size_t>(td.id) * chblocks + cb) * G::kS * kLanes;   // rows in (element, position) order
  for (int i = threadIdx.x; i < G::kS * kLanes; i += kSpecThreads) {
    T acc = red[i];
#pragma unroll
    for (int v = 1; v < kSpecWaves; ++v) acc += red[v * G::kS * kLanes + i];
    out[i] = acc;
  }
}

// Second-order pass: the backward skeleton with one more input row (H) and one more output
// row (ddB) per node; its dW2' rows leave through the same per-tile partial rows.
//
// The generated program keeps about 290 values live.  Two kernels:
//  * spec_double_backward_kernel keeps everything in registers (256 VGPRs + AGPRs, one wave
//    per SIMD);
//  * spec_double_backward_lds_kernel keeps the folded weights w' and the dW2' accumulators
//    (2 x kS values per lane) in LDS columns - w' is re-read and the accumulators are updated
//    once per node - which brings it under 256 registers without scratch, so that two waves
//    share a SIMD (measured on MI355X, fp32, 0e+1o: 80 us instead of 106 us at 10k nodes,
//    1.24 ms instead of 1.45 ms at 200k).  It is used where it fits (kUseLdsState): for the
//    larger basis or fp64 it would spill.  Small changes to its text move the register
//    allocation across the spill threshold: check the compiler's resource report
//    (-Rpass-analysis=kernel-resource-usage) after touching it.
// Rows of one node in the second-order kernels, in either layout (see Cols).
template <typename T, typename TS, typename G, bool kCM>
struct NodeRows2 {
  static __device__ __forceinline__ void load(const TS* __restrict__ A, const TS* __restrict__ H, const TS* __restrict__ dB,
                                              size_t node, int K, int ch, T (&a)[G::kNlm], T (&h)[G::kNlm], T (&g)[G::kNLM]) {
    if constexpr (kCM) {
      Cols<TS, G::kNlm>::load(A + node * G::kNlm * K + ch, K, a);
      Cols<TS, G::kNlm>::load(H + node * G::kNlm * K + ch, K, h);
      Cols<TS, G::kNLM>::load(dB + node * G::kNLM * K + ch, K, g);
    } else {
      RowIO<T, TS, G::kNlm>::load(A + (node * K + ch) * G::kNlm, a);
      RowIO<T, TS, G::kNlm>::load(H + (node * K + ch) * G::kNlm, h);
      RowIO<T, TS, G::kNLM>::load(dB + (node * K + ch) * G::kNLM, g);
    }
  }
  template <bool kFull>
  static __device__ __forceinline__ void store(TS* __restrict__ dA2, TS* __restrict__ ddB, size_t node, int K, int cb, int ch,
                                               T* stage, int lane, int live, const T (&da)[G::kNlm], const T (&ddb)[G::kNLM]) {
    if constexpr (kCM) {
      if (kFull || lane < live) {
        Cols<TS, G::kNlm>::template store<true>(dA2 + node * G::kNlm * K + ch, K, da);
        Cols<TS, G::kNLM>::template store<true>(ddB + node * G::kNLM * K + ch, K, ddb);
      }
    } else {
      constexpr bool kStageB = G::kNLM * sizeof(TS) != 16;
      store_rows_as<T, TS, G::kNlm>(dA2 + (node * K + cb * kLanes) * G::kNlm, stage, lane, da, live);
      if constexpr (kStageB) store_rows_as<T, TS, G::kNLM>(ddB + (node * K + cb * kLanes) * G::kNLM, stage, lane, ddb, live);
      else if (kFull || lane < live) RowIO<T, TS, G::kNLM>::store(ddB + (node * K + ch) * G::kNLM, ddb);
    }
  }
};

template <typename T, typename G, bool kFull, typename TS, typename TW, bool kCM>
__global__ __launch_bounds__(kSpecThreads) void spec_double_backward_kernel(
    const TileDesc* __restrict__ tiles, int n_blocks, int chblocks, const int32_t* __restrict__ perm, int K,
    const TW* __restrict__ W, const TS* __restrict__ A, const TS* __restrict__ H, const TS* __restrict__ dB,
    TS* __restrict__ ddB, TS* __restrict__ dA2, T* __restrict__ partial) {
  extern __shared__ unsigned char lds_raw[];
  T* red = reinterpret_cast<T*>(lds_raw);  // [kSpecWaves][kS][64]
  T* stage = red + kSpecWaves * G::kS * kLanes + wave_of_thread() * kLanes * G::kNlm;  // [64][kNlm] per wave
  static_assert(!kCM || std::is_same<T, TS>::value, "component-major rows are stored in the arithmetic type");
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int logical = blockIdx.x;   // descriptors are stored largest tile first: dispatch order is the schedule
  if (logical >= n_blocks) return;  // uniform per workgroup
  const int tile = logical / chblocks, cb = logical % chblocks;
  const TileDesc td = tiles[tile];
  if (td.count == 0) return;        // unused descriptor; uniform per workgroup
  const int j0 = td.start + td.count * wave / kSpecWaves;
  const int j1 = td.start + td.count * (wave + 1) / kSpecWaves;
  const int live = kFull ? kLanes : (K - cb * kLanes < kLanes ? K - cb * kLanes : kLanes);   // channels of this block
  const int ch = cb * kLanes + (lane < live ? lane : live - 1);           // dead lanes repeat the last channel
  T dw[G::kS];
#pragma unroll
  for (int s = 0; s < G::kS; ++s) dw[s] = T(0);
  if (j0 < j1) {
    T w[G::kS];
    G::fold(W + static_cast<size_t>(td.z) * G::kP * K + ch, K, w);
    // one register set of inputs: the next node's rows are requested right after the
    // arithmetic of the current one has consumed them, ahead of its stores
    T a[G::kNlm], h[G::kNlm], g[G::kNLM], da[G::kNlm], ddb[G::kNLM];
    size_t node = perm ? perm[j0] : j0;   // no permutation: the batch is already grouped
    NodeRows2<T, TS, G, kCM>::load(A, H, dB, node, K, ch, a, h, g);
    for (int j = j0; j < j1; ++j) {
      G::double_backward(a, w, g, h, ddb, da, dw);
      const size_t cur = node;
      if (j + 1 < j1) {
        node = perm ? perm[j + 1] : j + 1;
        NodeRows2<T, TS, G, kCM>::load(A, H, dB, node, K, ch, a, h, g);
      }
      NodeRows2<T, TS, G, kCM>::template store<kFull>(dA2, ddB, cur, K, cb, ch, stage, lane, live, da, ddb);
    }
  }
#pragma unroll
  for (int s = 0; s < G::kS; ++s) red[(wave * G::kS + s) * kLanes + lane] = dw[s];
  __syncthreads();
  T* out = partial + (static_cast<size_t>(td.id) * chblocks + cb) * G::kS * kLanes;   // rows in (element, position) order
  for (int i = threadIdx.x; i < G::kS * kLanes; i += kSpecThreads) {
    T acc = red[i];
#pragma unroll
    for (int v = 1; v < kSpecWaves; ++v) acc += red[v * G::kS * kLanes + i];
    out[i] = acc;
  }
}

// See above.  LDS: w' [kSpecWaves][kS][64] | sums [kSpecWaves][kS][64] | stage [kSpecWaves][64][kNlm].
template <typename T, typename G, bool kFull, typename TS, typename TW, bool kCM>
__global__ __launch_bounds__(kSpecThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void spec_double_backward_lds_kernel(
    const TileDesc* __restrict__ tiles, int n_blocks, int chblocks, const int32_t* __restrict__ perm, int K,
    const TW* __restrict__ W, const TS* __restrict__ A, const TS* __restrict__ H, const TS* __restrict__ dB,
    TS* __restrict__ ddB, TS* __restrict__ dA2, T* __restrict__ partial) {
  extern __shared__ unsigned char lds_raw[];
  T* red = reinterpret_cast<T*>(lds_raw);  // [kSpecWaves][kS][64]: every wave's w' columns
  T* acc_all = red + kSpecWaves * G::kS * kLanes;                         // [kSpecWaves][kS][64] dW2' sums
  T* stage = acc_all + kSpecWaves * G::kS * kLanes + wave_of_thread() * kLanes * G::kNlm;  // [64][kNlm] per wave
  static_assert(!kCM || std::is_same<T, TS>::value, "component-major rows are stored in the arithmetic type");
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int logical = blockIdx.x;   // descriptors are stored largest tile first: dispatch order is the schedule
  if (logical >= n_blocks) return;  // uniform per workgroup
  const int tile = logical / chblocks, cb = logical % chblocks;
  const TileDesc td = tiles[tile];
  if (td.count == 0) return;        // unused descriptor; uniform per workgroup
  const int j0 = td.start + td.count * wave / kSpecWaves;
  const int j1 = td.start + td.count * (wave + 1) / kSpecWaves;
  const int live = kFull ? kLanes : (K - cb * kLanes < kLanes ? K - cb * kLanes : kLanes);   // channels of this block
  const int ch = kFull ? cb * kLanes + lane : cb * kLanes + (lane < live ? lane : live - 1);   // dead lanes repeat the last channel
  T* dwl = acc_all + wave * G::kS * kLanes + lane;
#pragma unroll
  for (int s = 0; s < G::kS; ++s) dwl[s * kLanes] = T(0);
  if (j0 < j1) {
    T* wl = red + wave * G::kS * kLanes + lane;   // this wave's slice of red holds w' until the end
    {
      T w0[G::kS];
      G::fold(W + static_cast<size_t>(td.z) * G::kP * K + ch, K, w0);
#pragma unroll
      for (int s = 0; s < G::kS; ++s) wl[s * kLanes] = w0[s];
    }
    // one register set of inputs: the next node's rows are requested right after the
    // arithmetic of the current one has consumed them, ahead of its stores
    T a[G::kNlm], h[G::kNlm], g[G::kNLM], da[G::kNlm], ddb[G::kNLM];
    size_t node = perm ? perm[j0] : j0;   // no permutation: the batch is already grouped
    NodeRows2<T, TS, G, kCM>::load(A, H, dB, node, K, ch, a, h, g);
    for (int j = j0; j < j1; ++j) {
      T w[G::kS];
      asm volatile("" ::: "memory");  // keep the reads of w' inside the loop (registers are short)
#pragma unroll
      for (int s = 0; s < G::kS; ++s) w[s] = wl[s * kLanes];
      T dw[G::kS];
#pragma unroll
      for (int s = 0; s < G::kS; ++s) dw[s] = T(0);
      G::double_backward(a, w, g, h, ddb, da, dw);
#pragma unroll
      for (int s = 0; s < G::kS; ++s) dwl[s * kLanes] += dw[s];
      const size_t cur = node;
      if (j + 1 < j1) {
        node = perm ? perm[j + 1] : j + 1;
        NodeRows2<T, TS, G, kCM>::load(A, H, dB, node, K, ch, a, h, g);
      }
      NodeRows2<T, TS, G, kCM>::template store<kFull>(dA2, ddB, cur, K, cb, ch, stage, lane, live, da, ddb);
    }
  }
  __syncthreads();
  T* out = partial + (static_cast<size_t>(td.id) * chblocks + cb) * G::kS * kLanes;   // rows in (element, position) order
  for (int i = threadIdx.x; i < G::kS * kLanes; i += kSpecThreads) {
    T acc = acc_all[i];
#pragma unroll
    for (int v = 1; v < kSpecWaves; ++v) acc += acc_all[v * G::kS * kLanes + i];
    out[i] = acc;
  }
}

template <typename T, typename G>
constexpr bool kUseLdsState = sizeof(T) == 4 && G::kS <= 32;

// Second stage of the dW reduction and the map to the external paths, one launch.  The fold
// matrix F (dW[p] = sum_s F[s,p] r[s]) falls into small independent blocks of one to three
// internal rows s and the external paths p that depend on them (generated descriptors).  A workgroup takes a group of
// consecutive blocks of one (element, channel block): its waves add the group's rows over an equal share of the element's tiles each, in
// tile order and in fp64, the shares meet in LDS in wave order, and the first wave writes the group's external paths.
// Elements without nodes own no tiles and get zeros.  Every sum has a fixed order: results are bitwise reproducible.
// What bounds it: the instructions of its waves (a launch with a wave per block lasted 1.7 us and 1.1 ns a wave, from 2300 to 9600 waves,
// whatever the waves summed).  So the code of a group is straight-line: its rows, paths and coefficients are constants and not read from a
// descriptor (176 to 520 bytes of scalar loads, a branch per coefficient), absent tiles are skipped and not masked, and a wave has up to four
// rows.  us a launch, a wave per block -> this:
//   128 channels, 0e+1o       3072 nodes 6.6 -> 4.2    10 000 6.8 -> 5.2    200 000 24 -> 16
//   256 channels, 0e+1o+2e    50 000 nodes 20.9 -> 13.7        four outputs, 107 nodes 12.3 -> 6.4        64 channels, 83 nodes 4.2 -> 3.0
// and with four / six / eight rows a group: 3072 nodes 4.2 / 4.3 / 4.1, 10 000 5.2 / 5.4 / 5.2, 200 000 15.9 / 19.0 / 18.0, 83 nodes 3.0 / 3.1 / 3.3.
// Earlier forms (10k / 200k nodes): a sum kernel followed by an unfold kernel
// 11.2 / 15.6 us; one workgroup per (element, channel block) for all rows 13.5 / 31 us (the twelve
// workgroups of the six frequent elements own 60% of the bytes).  A device-scope "last workgroup finishes the job" scheme inside the
// backward kernel was far slower than a launch: its fences flush the per-XCD L2s on this chip.
constexpr int kFinalizeRows = 4;    // rows of a group at most (a block has no more: FinalizeGroups)

// Blocks of F in groups of at most kFinalizeRows rows, in order: group g is the blocks first[g] .. first[g + 1] - 1.
template <typename G>
struct FinalizeGroups {
  static_assert(G::kMaxBlockRows <= kFinalizeRows, "a group holds any block");
  struct Table {
    int n, first[G::kNumBlocks + 1];
  };
  static constexpr Table make() {
    Table t{};
    int rows = 0;
    for (int b = 0; b < G::kNumBlocks; ++b) {
      if (b == 0 || rows + G::kBlocks[b].n_rows > kFinalizeRows) {
        t.first[t.n++] = b;
        rows = 0;
      }
      rows += G::kBlocks[b].n_rows;
    }
    t.first[t.n] = G::kNumBlocks;
    return t;
  }
  static constexpr Table table = make();
  static constexpr int rows_of(int g) {
    int rows = 0;
    for (int b = table.first[g]; b < table.first[g + 1]; ++b) rows += G::kBlocks[b].n_rows;
    return rows;
  }
  static constexpr int row(int g, int i) {   // the i-th row of group g
    for (int b = table.first[g]; b < table.first[g + 1]; ++b) {
      if (i < G::kBlocks[b].n_rows) return G::kBlocks[b].row[i];
      i -= G::kBlocks[b].n_rows;
    }
    return 0;
  }
  static constexpr int first_of(int g, int blk) {   // position of the block's first row in the group
    int i = 0;
    for (int b = table.first[g]; b < blk; ++b) i += G::kBlocks[b].n_rows;
    return i;
  }
};

template <int kBegin, int kEnd, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (kBegin < kEnd) {
    f(std::integral_constant<int, kBegin>{});
    static_for<kBegin + 1, kEnd>(f);
  }
}

// shared: (kWaves - 1) * kFinalizeRows * kLanes values, in which the waves meet.
template <typename T, typename G, typename TW, int kWaves, int g>
__device__ __forceinline__ void finalize_group(int K, int ch, int lane, int wave, const T* __restrict__ src, size_t tstride, int t0, int t1,
                                               TW* __restrict__ out, double* shared) {
  typedef FinalizeGroups<G> F;
  constexpr int R = F::rows_of(g), U = 4;   // U: tiles a trip, the next ones requested ahead
  double sum[R];
#pragma unroll
  for (int r = 0; r < R; ++r) sum[r] = 0.0;
  const int n = t1 - t0, ta = t0 + n * wave / kWaves, tb = t0 + n * (wave + 1) / kWaves;
  if (ta < tb) {
    T v[U][R], next[U][R];
    auto request = [&](int t, T (&x)[U][R]) {   // past the last tile it is read again and dropped
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const T* at = src + static_cast<size_t>(t + u < tb ? t + u : tb - 1) * tstride;
        static_for<0, R>([&](auto r) { x[u][r] = at[F::row(g, r) * kLanes + lane]; });
      }
    };
    request(ta, v);
#pragma unroll 1
    for (int t = ta; t < tb; t += U) {
      request(t + U, next);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (t + u < tb) {
#pragma unroll
          for (int r = 0; r < R; ++r) sum[r] += static_cast<double>(v[u][r]);
        }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int r = 0; r < R; ++r) v[u][r] = next[u][r];
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int r = 0; r < R; ++r) shared[((wave - 1) * R + r) * kLanes + lane] = sum[r];
  }
  __syncthreads();
  if (wave > 0) return;
#pragma unroll
  for (int w = 1; w < kWaves; ++w)
#pragma unroll
    for (int r = 0; r < R; ++r) sum[r] += shared[((w - 1) * R + r) * kLanes + lane];
  if (ch >= K) return;   // lanes past the last channel
  static_for<F::table.first[g], F::table.first[g + 1]>([&](auto blk) {
    static_for<0, G::kBlocks[blk].n_paths>([&](auto i) {
      double v = 0.0;
      static_for<0, G::kBlocks[blk].n_rows>([&](auto r) {
        if constexpr (G::kBlocks[blk].coef[i][r] != 0.0) v += G::kBlocks[blk].coef[i][r] * sum[F::first_of(g, blk) + r];
      });
      out[static_cast<size_t>(G::kBlocks[blk].path[i]) * K + ch] = static_cast<TW>(v);
    });
  });
}

template <typename T, typename G, typename TW, int kWaves>
__global__ __launch_bounds__(kWaves * kLanes) void spec_finalize_kernel(int K, int chblocks, int max_tiles,
                                                                        const T* __restrict__ partial,
                                                                        const int32_t* __restrict__ tile_off,
                                                                        TW* __restrict__ dW) {
  constexpr int S = G::kS, kGroups = FinalizeGroups<G>::table.n;
  __shared__ double shared[(kWaves - 1) * kFinalizeRows * kLanes];
  const int lane = threadIdx.x % kLanes, wave = wave_of_thread();
  const int group = blockIdx.x % kGroups;
  const int cb = blockIdx.x / kGroups;
  const int e = blockIdx.y;
  const int t0 = tile_off[e], t1 = tile_off[e + 1] < max_tiles ? tile_off[e + 1] : max_tiles;
  const size_t tstride = static_cast<size_t>(chblocks) * S * kLanes;
  const T* src = partial + static_cast<size_t>(cb) * S * kLanes;
  TW* out = dW + static_cast<size_t>(e) * G::kP * K;
  static_for<0, kGroups>([&](auto g) {
    if (group == g) finalize_group<T, G, TW, kWaves, g>(K, cb * kLanes + lane, lane, wave, src, tstride, t0, t1, out, shared);
  });
}

SplitGroupArgs group_args(const sc_plan* plan, int64_t n, const int32_t* z, const Workspace& ws,
                          const LaunchShape& shape, bool window_order = false) {
  SplitGroupArgs g{};
  g.z = z;
  g.n = static_cast<int>(n);
  g.Z = plan->cfg.num_elements;
  g.W = shape.split_waves;
  g.nodes_per_wave = shape.split_nodes_per_wave;
  g.tile_nodes = shape.tile_nodes;
  g.max_tiles = shape.max_tiles;
  g.counts = ws.counts;
  g.seg_off = ws.seg_off;
  g.tile_off = ws.tile_off;
  g.ntiles = ws.ntiles;
  g.tiles = ws.tiles;
  g.perm = ws.perm;
  g.wnode = window_order ? ws.wnode : nullptr;
  g.wkey = window_order ? ws.wkey : nullptr;
  return g;
}

template <typename K>
hipError_t raise_lds_limit(K kernel, size_t lds) {
  if (lds <= 64 * 1024) return hipSuccess;  // above the default dynamic LDS limit: raise it for this kernel
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             static_cast<int>(lds));
}

template <typename T, typename G, typename TW>
hipError_t prepare_launch(const sc_plan* plan, int64_t n, const int32_t* z, const void* W, const Workspace& ws,
                          const LaunchShape& shape, bool count, bool fold, bool window_order, hipStream_t stream) {
  const int count_wgs = count ? shape.split_waves / kGroupWavesPerWG : 0;
  const bool window = window_order && ws.wnode && ws.wkey;
  const int window_wgs = window ? static_cast<int>((n + kWindowNodes - 1) / kWindowNodes) : 0;
  const int n_pairs = fold ? plan->cfg.num_elements * shape.chblocks : 0;
  const int grid = window_wgs + count_wgs + n_pairs;
  if (grid == 0) return hipSuccess;
  const size_t lds = window ? split_window_lds_bytes(plan->cfg.num_elements)
                            : count ? split_group_lds_bytes(plan->cfg.num_elements) : 0;
  hipLaunchKernelGGL((spec_prepare_kernel<T, G, TW>), dim3(grid), dim3(kSpecThreads), lds, stream,
                     z, static_cast<int>(n), plan->cfg.num_elements, window_wgs, count_wgs, static_cast<const TW*>(W),
                     static_cast<T*>(ws.wfold), plan->cfg.num_channels, shape.chblocks,
                     group_args(plan, n, z, ws, shape, window));
  return hipGetLastError();
}

// Nodes per workgroup of the natural-order forward.  All workgroups do the same work, so the
// kernel takes (rounds of resident workgroups) x (nodes per wave): the tile is the multiple of
// four nodes in 8..32 (8..64 for the larger bases) that minimises that product for this batch on this chip (10k nodes, 128
// channels, four workgroups per CU: 20 nodes = one round of five nodes per wave instead of two
// rounds of four with 16); among sizes within 2% of the best the largest up to `most` wins, since
// longer shares per wave meet more runs of one element (measured best at 200k nodes before the
// window order: 24..32 nodes with the 29-row basis, 48 with the 49-row basis, whose weights cost
// more to re-read).  From eight rounds on the rounds no longer tell (workgroups are replaced as
// they end) and, with the window order making the runs long whatever the share, the small bases
// do best with five nodes per wave: 200k nodes, 29-row basis, forward 373 us with 20 nodes per
// workgroup against 376 (16), 381 (24), 387 (28), 391 (32); the 49-row basis shows no preference
// between 20 and 48 (268 us at 50k nodes, 256 channels) and keeps the rule above.  Batches that fit one round
// with a node per wave take four: such calls last as long as one wave (fp64, 500 nodes 13.8 -> 11.2 us a call).
inline int forward_tile_nodes(int64_t n, int chblocks, int64_t resident_wgs, int most) {
  auto cost = [&](int t) {
    const int64_t wgs = (n + t - 1) / t * chblocks;
    return static_cast<double>((wgs + resident_wgs - 1) / resident_wgs) * (t / kSpecWaves);
  };
  if ((n + 3) / 4 * chblocks <= resident_wgs) return 4;
  if (most <= 32 && (n + 19) / 20 * chblocks >= 8 * resident_wgs) return 20;
  double best = cost(8);
  for (int t = 12; t <= most; t += 4) best = cost(t) < best ? cost(t) : best;
  int pick = 8;
  for (int t = 8; t <= most; t += 4)
    if (cost(t) <= best * 1.02) pick = t;
  return pick;
}

template <typename T, typename G, typename TS, typename TW, bool kCM, bool kDirect>
hipError_t fwd_launch(const sc_plan* plan, int64_t n, const void* A, const int32_t* z, const void* W, void* B,
                      const Workspace& ws, const LaunchShape& shape, int group, bool window_order, bool fold_table,
                      hipStream_t stream) {
  // group: 0 no grouping roles, 1 scatter + table, 2 table only (the batch is already grouped), 3 no roles and clamped indices
  const bool scatter = group == 1;
  const int table = group == 1 || group == 2;
  const int scatter_wgs = scatter ? shape.split_waves / kGroupWavesPerWG : 0;
  size_t lds = (G::kNLM * sizeof(TS) != 16) ? sizeof(T) * kSpecWaves * G::kNLM * kLanes : 0;
  if (table) {
    const size_t roles = split_group_lds_bytes(plan->cfg.num_elements) + (kDirect ? split_counts_bytes(plan, shape) : 0);
    if (roles > lds) lds = roles;
  }
  constexpr int kPairs = kSpecWaves / direct_fold_waves<G>();   // a workgroup of the fold role
  const bool clamp = kDirect && group == 3;   // given as fold_wgs = -1: no such workgroups then
  const int fold_wgs = kDirect && fold_table && !clamp ? (plan->cfg.num_elements * shape.chblocks + kPairs - 1) / kPairs : 0;
  static const int wgs_per_cu = [] {   // resident workgroups per compute unit of this instance
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, &spec_forward_kernel<T, G, TS, TW, kCM, kDirect>, kSpecThreads, 0) != hipSuccess || nb < 1)
      nb = 1;
    return nb;
  }();
  const int tile = shape.fwd_tile_nodes > 0 ? shape.fwd_tile_nodes
                                            : forward_tile_nodes(n, shape.chblocks, static_cast<int64_t>(wgs_per_cu) * plan->num_cus,
                                                                 G::kS > 32 ? 64 : 32);
  const int tiles = B ? static_cast<int>((n + tile - 1) / tile) : 0;   // (launch_spec_group: the roles alone)
  const int grid = scatter_wgs + table + fold_wgs + tiles * shape.chblocks;
  hipLaunchKernelGGL((spec_forward_kernel<T, G, TS, TW, kCM, kDirect>), dim3(grid), dim3(kSpecThreads), lds, stream,
                     window_order ? ws.wnode : nullptr, window_order ? ws.wkey : z, scatter_wgs, table, shape.chblocks, tile,
                     static_cast<int>(n), plan->cfg.num_elements, plan->cfg.num_channels, clamp ? -1 : fold_wgs,
                     static_cast<const TS*>(A), static_cast<const T*>(ws.wfold), static_cast<const TW*>(W), static_cast<TS*>(B),
                     group_args(plan, n, z, ws, shape, window_order));
  return hipGetLastError();
}

template <typename T, typename G, typename TS, bool kCM>
hipError_t bwd_launch(const sc_plan* plan, int64_t n, const void* A, const void* dB, void* dA,
                      const Workspace& ws, const LaunchShape& shape, hipStream_t stream) {   // ws.perm may be null
  const int n_blocks = shape.max_tiles * shape.chblocks;
  const int grid = (n_blocks + kXcds - 1) / kXcds * kXcds;
  const size_t lds = sizeof(T) * kSpecWaves * (G::kS + G::kNlm) * kLanes;
  const bool full = plan->cfg.num_channels % kLanes == 0;
  auto kernel = full ? &spec_backward_kernel<T, G, 0, false, true, TS, kCM> : &spec_backward_kernel<T, G, 0, false, false, TS, kCM>;
  if constexpr (sizeof(T) == 4) {
    // small batches: dA streamed past the cache (see the kernel)
    if (n <= 40000 && full) kernel = &spec_backward_kernel<T, G, 0, true, true, TS, kCM>;
  }
  const hipError_t e = raise_lds_limit(kernel, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(kSpecThreads), lds, stream, ws.tiles, n_blocks, shape.chblocks, ws.perm,
                     plan->cfg.num_channels, static_cast<const T*>(ws.wfold), static_cast<const TS*>(A),
                     static_cast<const TS*>(dB), static_cast<TS*>(dA), static_cast<T*>(ws.partial));
  return hipGetLastError();
}

template <typename T, typename G, typename TS, typename TW, bool kCM>
hipError_t dbl_launch(const sc_plan* plan, const void* A, const void* W, const void* dB, const void* H, void* ddB,
                      void* dA2, const Workspace& ws, const LaunchShape& shape, hipStream_t stream) {
  const int n_blocks = shape.max_tiles * shape.chblocks;
  const int grid = (n_blocks + kXcds - 1) / kXcds * kXcds;
  constexpr bool kLds = kUseLdsState<T, G>;
  const size_t lds = sizeof(T) * kSpecWaves * ((kLds ? 2 : 1) * G::kS + G::kNlm) * kLanes;
  const bool full = plan->cfg.num_channels % kLanes == 0;   // no idle lanes: an instance without their handling
  auto kernel = full ? &spec_double_backward_kernel<T, G, true, TS, TW, kCM> : &spec_double_backward_kernel<T, G, false, TS, TW, kCM>;
  if constexpr (kLds) kernel = full ? &spec_double_backward_lds_kernel<T, G, true, TS, TW, kCM> : &spec_double_backward_lds_kernel<T, G, false, TS, TW, kCM>;
  const hipError_t e = raise_lds_limit(kernel, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(kSpecThreads), lds, stream, ws.tiles, n_blocks, shape.chblocks, ws.perm,
                     plan->cfg.num_channels, static_cast<const TW*>(W), static_cast<const TS*>(A), static_cast<const TS*>(H),
                     static_cast<const TS*>(dB), static_cast<TS*>(ddB), static_cast<TS*>(dA2), static_cast<T*>(ws.partial));
  return hipGetLastError();
}

template <typename T, typename G, typename TW>
hipError_t finalize_launch(const sc_plan* plan, void* dW, const Workspace& ws, const LaunchShape& shape,
                           hipStream_t stream) {
  const int Z = plan->cfg.num_elements;
  // Waves that share an element's tiles, one / two / four, us a launch: 3072 nodes (three tiles an element on average, nineteen of the frequent
  // ones) 6.5 / 4.2 / 4.2, 10 000 (four) 5.4 / 5.2 / 5.2, 200 000 (20) 39 / 24 / 16; 107 nodes, four outputs, 6.9 / 6.9 / 6.3, 83 nodes 2.8 / 3.0 / 3.3.
  const int waves = shape.max_tiles > 8 * Z ? 4 : 2;
  const auto kernel = waves == 4 ? &spec_finalize_kernel<T, G, TW, 4> : &spec_finalize_kernel<T, G, TW, 2>;
  hipLaunchKernelGGL(kernel, dim3(shape.chblocks * FinalizeGroups<G>::table.n, Z), dim3(waves * kLanes), 0, stream,
                     plan->cfg.num_channels, shape.chblocks, shape.max_tiles, static_cast<const T*>(ws.partial),
                     ws.tile_off, static_cast<TW*>(dW));
  return hipGetLastError();
}


// The types of a kernel family for one plan dtype: T arithmetic, folded weights and per-tile dW rows,
// TS rows of the per-node tensors, TW weights W and dW.
template <typename T_, typename TS_, typename TW_>
struct Types {
  typedef T_ T;
  typedef TS_ TS;
  typedef TW_ TW;
};

// The launches of one generated program G as the functions of its table entry.  kWide: fp32 plans
// compute in fp64 on fp32 rows and weights, with one rounding per result, like the table-driven kernels
// that the same plans run on with SC_PLAN_FORCE_GENERIC; bfloat16 rows and the component-major layout
// are not served.  The table-driven kernels look up every term of the expanded polynomial and keep all
// operands in LDS; measured against them, forward + backward of 2000 nodes x 128 channels, fp32 / fp64
// rows: l_max = 2, nu_max = 3, 0e+1o 672 / 699 -> 24 / 28 us, with 2e 1383 / 1395 -> 36 / 41; l_max = 3,
// nu_max = 2, 0e+1o 170 / 182 -> 22 / 33, with 2e and 3o (fp32) 512 -> 41; l_max = nu_max = 2, 0e+1o 100
// / 106 -> 19 / 22.
template <typename G, bool kWide>
struct Entry {
  template <typename F>
  static hipError_t by_type(const sc_plan* plan, F&& fn) {
    if (plan->cfg.dtype == SC_F64) return fn(Types<double, double, double>());
    if constexpr (kWide) {
      if (plan->cfg.dtype == SC_F32) return fn(Types<double, float, float>());
      return hipErrorInvalidValue;
    } else {
      if (plan->cfg.dtype == SC_BF16) return fn(Types<float, bf16_bits, float>());
      return fn(Types<float, float, float>());
    }
  }
  static hipError_t prepare(const sc_plan* plan, int64_t n, const int32_t* z, const void* W, const Workspace& ws,
                            const LaunchShape& shape, bool count, bool fold, bool window_order, hipStream_t stream) {
    return by_type(plan, [&](auto t) {
      typedef decltype(t) Y;
      return prepare_launch<typename Y::T, G, typename Y::TW>(plan, n, z, W, ws, shape, count, fold, window_order, stream);
    });
  }
  static hipError_t forward(const sc_plan* plan, int64_t n, const void* A, const int32_t* z, const void* W, void* B,
                            const Workspace& ws, const LaunchShape& shape, int group, bool window_order,
                            bool component_major, bool direct, bool fold_table, hipStream_t stream) {
    return by_type(plan, [&](auto t) {
      typedef decltype(t) Y;
      typedef typename Y::T T;
      typedef typename Y::TS TS;
      typedef typename Y::TW TW;
      if (component_major) {
        if constexpr (std::is_same<T, TS>::value && !kWide) {
          if (!direct) return fwd_launch<T, G, TS, TW, true, false>(plan, n, A, z, W, B, ws, shape, group, window_order, false, stream);
        }
        return hipErrorInvalidValue;   // refused by the caller
      }
      if (direct) return fwd_launch<T, G, TS, TW, false, true>(plan, n, A, z, W, B, ws, shape, group, window_order, fold_table, stream);
      return fwd_launch<T, G, TS, TW, false, false>(plan, n, A, z, W, B, ws, shape, group, window_order, false, stream);
    });
  }
  static hipError_t backward(const sc_plan* plan, int64_t n, const void* A, const void* dB, void* dA, const Workspace& ws,
                             const LaunchShape& shape, bool component_major, hipStream_t stream) {
    return by_type(plan, [&](auto t) {
      typedef decltype(t) Y;
      if (component_major) {
        if constexpr (std::is_same<typename Y::T, typename Y::TS>::value && !kWide)
          return bwd_launch<typename Y::T, G, typename Y::TS, true>(plan, n, A, dB, dA, ws, shape, stream);
        return hipErrorInvalidValue;
      }
      return bwd_launch<typename Y::T, G, typename Y::TS, false>(plan, n, A, dB, dA, ws, shape, stream);
    });
  }
  static hipError_t double_backward(const sc_plan* plan, const void* A, const void* W, const void* dB, const void* H,
                                    void* ddB, void* dA2, const Workspace& ws, const LaunchShape& shape,
                                    bool component_major, hipStream_t stream) {
    return by_type(plan, [&](auto t) {
      typedef decltype(t) Y;
      typedef typename Y::T T;
      typedef typename Y::TS TS;
      typedef typename Y::TW TW;
      if (component_major) {
        if constexpr (std::is_same<T, TS>::value && !kWide)
          return dbl_launch<T, G, TS, TW, true>(plan, A, W, dB, H, ddB, dA2, ws, shape, stream);
        return hipErrorInvalidValue;
      }
      return dbl_launch<T, G, TS, TW, false>(plan, A, W, dB, H, ddB, dA2, ws, shape, stream);
    });
  }
  static hipError_t finalize(const sc_plan* plan, void* dW, const Workspace& ws, const LaunchShape& shape,
                             hipStream_t stream) {
    return by_type(plan, [&](auto t) {
      typedef decltype(t) Y;
      return finalize_launch<typename Y::T, G, typename Y::TW>(plan, dW, ws, shape, stream);
    });
  }
  static SpecEntry make() {
    SpecEntry e{};
    e.l_max = G::kLmax;
    e.nu_max = G::kNuMax;
    e.num_out = G::kNumOut;
    for (int o = 0; o < G::kNumOut; ++o) {
      e.out_l[o] = G::kOutL[o];
      e.out_parity[o] = G::kOutParity[o];
    }
    e.n_lm = G::kNlm;
    e.P = G::kP;
    e.S = G::kS;
    e.wide = kWide;
    for (int i = 0; i < 3; ++i) {
      e.ops[i] = G::kOps[i];
      e.flops[i] = G::kFlops[i];
    }
    e.prepare = prepare;
    e.forward = forward;
    e.backward = backward;
    e.double_backward = double_backward;
    e.finalize = finalize;
    return e;
  }
};

}  // namespace
}  // namespace sc
