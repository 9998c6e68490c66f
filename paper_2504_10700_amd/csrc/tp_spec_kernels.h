// Kernel templates of the channelwise tensor product around generated straight-line arithmetic (see
// tp_spec.hip for the mapping): included by the files that instantiate them.
//
// T = type of the arithmetic, TS = type the tensors are stored in.  fp64 rows are computed in fp64.
// fp32 rows are computed in fp32 for the shapes with l_Y = L_max = 3 and l_h <= 1 on full 64-channel
// blocks, and in fp64 everywhere else, like the table-driven kernels: an fp64 instruction issues at
// the rate of an unpacked fp32 one on this chip, and the kernels are bound by the bytes of R.
// kFull: the channel count is a multiple of 64.  Otherwise the lanes past the last channel repeat it:
// their loads are valid, their stores are masked and their share of dY is zero.
#pragma once
#include <type_traits>

#include "tp_internal.h"
#include "tp_spec.h"

namespace tp {
namespace {

using sc::kLanes;

__device__ __forceinline__ float sc_fma(float x, float y, float z) { return __builtin_fmaf(x, y, z); }
__device__ __forceinline__ double sc_fma(double x, double y, double z) { return __builtin_fma(x, y, z); }

// Between two parts of a generated program (one path and the next): the given sums are complete here,
// and nothing moves across.  Left to itself the compiler interleaves the paths until every register is taken
// (second-order pass with l_h = 2 in fp64: 512 registers and 5 KB of scratch per lane).
template <typename T>
__device__ __forceinline__ void is_computed(const T& v) {
  asm volatile("" ::"v"(v));
}
template <typename... V>
__device__ __forceinline__ void end_of_part(const V&... v) {
  (is_computed(v), ...);
  __builtin_amdgcn_sched_barrier(0);
}

// Do the terms of an edge go into the sums over the edges one by one?  Not for fp64 rows, whose results keep the roundings that this costs: an
// edge's terms of equal magnitude, and its share of dh, are formed first there.  (Error of fp64 rows, one by one / so, twenty edges,
// 2-norm, l = 3, l_h = 2: A 5.5e-16 / 4.3e-16, ddA 6.8e-16 / 4.3e-16, dh 3.7e-16 / 2.0e-16.)
template <typename TS>
constexpr bool kDirect = sizeof(TS) == 4;

constexpr int kStageStride = kLanes + 1;  // LDS row stride of the dY transpose (odd: two-way conflicts at most)

// A row of N elements at p: 16-byte accesses and a scalar tail.  p is aligned to 16 B if the row size is
// a multiple of 16 B, else only to the element (16-byte accesses need no more on this chip).
template <typename T, int N>
struct Row {
  static constexpr int V = 16 / sizeof(T);
  typedef T Vec __attribute__((ext_vector_type(V), aligned((N * sizeof(T)) % 16 == 0 ? 16 : sizeof(T))));
};

template <typename T, int N>
__device__ __forceinline__ void load_row(const T* __restrict__ p, T (&v)[N]) {
  constexpr int V = Row<T, N>::V;
#pragma unroll
  for (int i = 0; i + V <= N; i += V) {
    const typename Row<T, N>::Vec x = *reinterpret_cast<const typename Row<T, N>::Vec*>(p + i);
#pragma unroll
    for (int k = 0; k < V; ++k) v[i + k] = x[k];
  }
#pragma unroll
  for (int i = N / V * V; i < N; ++i) v[i] = p[i];
}

template <typename TS, typename T, int N>
__device__ __forceinline__ void store_row(TS* __restrict__ p, const T (&v)[N]) {
  constexpr int V = Row<TS, N>::V;
#pragma unroll
  for (int i = 0; i + V <= N; i += V) {
    typename Row<TS, N>::Vec x;
#pragma unroll
    for (int k = 0; k < V; ++k) x[k] = static_cast<TS>(v[i + k]);
    // A row of one 16-byte piece makes the wave's store one contiguous KB: streamed past the
    // cache (measured faster).  Longer rows are written by several instructions that each touch
    // a part of every line: left to the L2 to merge (streaming them measured slower).
    if constexpr (N * sizeof(TS) == 16) __builtin_nontemporal_store(x, reinterpret_cast<typename Row<TS, N>::Vec*>(p + i));
    else *reinterpret_cast<typename Row<TS, N>::Vec*>(p + i) = x;
  }
#pragma unroll
  for (int i = N / V * V; i < N; ++i) p[i] = static_cast<TS>(v[i]);
}

// Values as stored -> values of the arithmetic (nothing where the types are the same).  The rows that are
// requested ahead stay in the storage type until they are used: without the empty statement the
// compiler moves the conversions, and products of the values with constants, to the request of the row, and
// carries twice the registers from there to the use.
template <typename T, typename TS, int N>
__device__ __forceinline__ void widen(const TS (&v)[N], T (&w)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    TS x = v[i];
    asm volatile("" : "+v"(x));
    w[i] = static_cast<T>(x);
  }
}

// R[e][p][ch] for all paths of edge e.
template <typename T, int P>
__device__ __forceinline__ void load_weights(const T* __restrict__ R, int e, int K, int ch, T (&r)[P]) {
  const T* base = R + static_cast<size_t>(e) * P * K + ch;
#pragma unroll
  for (int p = 0; p < P; ++p) r[p] = base[static_cast<size_t>(p) * K];
}

// r[p] of a row in registers, in the type of the arithmetic.  The conversion happens where the path reads it: done
// for the whole row up front it holds twice the registers of the row through all paths.
template <typename T, typename TS, int P>
struct PathRow {
  const TS (&v)[P];
  __device__ __forceinline__ T operator[](int p) const {
    TS x = v[p];
    if constexpr (!std::is_same<T, TS>::value) asm volatile("" : "+v"(x));
    return static_cast<T>(x);
  }
};

// dR[e][p][ch]: every path's value goes out when it is assigned (every row is written as whole lines: streamed
// past the cache).
template <bool kFull, typename T, typename TS>
struct PathStore {
  TS* out;     // dR + (e * P * K + ch)
  size_t K;
  bool live;
  struct Ref {
    const PathStore& s;
    int p;
    __device__ __forceinline__ void operator=(T v) const {
      if (kFull || s.live) __builtin_nontemporal_store(static_cast<TS>(v), s.out + p * s.K);
    }
  };
  __device__ __forceinline__ Ref operator[](int p) const { return Ref{*this, p}; }
};

// This channel's share of dY[e][a], into the wave's transpose stage (see lane_sum_store) when it is assigned (kAdd: on top of what
// another channel of this lane has put there).
template <bool kFull, bool kAdd, typename T>
struct StageStore {
  T* lane_column;
  bool live;
  struct Ref {
    const StageStore& s;
    int a;
    __device__ __forceinline__ void operator=(T v) const {
      T* const to = s.lane_column + a * kStageStride;
      const T mine = kFull || s.live ? v : T(0);
      *to = kAdd ? *to + mine : mine;
    }
  };
  __device__ __forceinline__ Ref operator[](int a) const { return Ref{*this, a}; }
};

// Empty statements that pin where values are computed.  Before the arithmetic of an edge, on values that do
// not change over the edges of an atom: what follows from them (the row dA times every magnitude of
// the couplings: 130 values for l_h = 2) would otherwise be moved in front of the loop and held in registers.
// After it, on the sums over the edges: their additions would otherwise be moved behind the stores
// of the edge, with all their operands live until there.
template <typename T, int N>
__device__ __forceinline__ void pin_values(T (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[i]));
}

// Y[e][:], identical for all lanes (e is wave-uniform).  Rows in the type of the arithmetic: scalar loads where the edge is
// evaluated.  fp64 arithmetic on fp32 rows: value a in lane a of one register, requested with the other rows of the edge,
// widened by one instruction and read back to scalar registers, which have no room for a second set of them; as
// scalar loads every edge waits for memory there, its other rows long in registers, and every value is widened by itself.
// (Bound by latency at two to four waves per SIMD.  With the forward's requests out of their conditions, below: forward and
// backward, l_h = 2, 3001 atoms, 128 channels, 475 -> 457 us; l_h = 1, fp32 arithmetic, 10 000 atoms, 687 -> 679.)
template <typename T, typename TS, int N>
struct UniformRow {
  static constexpr bool kAhead = !std::is_same<T, TS>::value;
  static_assert(N <= kLanes, "a lane per value");
  TS mine;
  __device__ __forceinline__ void request(const TS* __restrict__ Y, int e, int lane) {
    if constexpr (kAhead) mine = Y[static_cast<size_t>(e) * N + (lane < N ? lane : N - 1)];
  }
  __device__ __forceinline__ void use(const TS* __restrict__ Y, int e, T (&y)[N]) const {
    if constexpr (kAhead) {
      TS x = mine;
      asm volatile("" : "+v"(x));   // widened here and not at the request
      const unsigned long long bits = __builtin_bit_cast(unsigned long long, static_cast<double>(x));
#pragma unroll
      for (int a = 0; a < N; ++a) {
        const unsigned lo = __builtin_amdgcn_readlane(static_cast<unsigned>(bits), a);
        const unsigned hi = __builtin_amdgcn_readlane(static_cast<unsigned>(bits >> 32), a);
        y[a] = __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
      }
    } else {
      const TS* base = Y + static_cast<size_t>(e) * N;
#pragma unroll
      for (int a = 0; a < N; ++a) y[a] = base[a];
    }
  }
};

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// blockIdx -> logical block such that the blocks an XCD receives (round-robin by blockIdx) form
// one contiguous range of atoms: the atoms of one structure, which share their senders' rows of
// h, then meet in one XCD's L2.  gridDim.x is a multiple of kXcds.
constexpr int kXcds = 8;
__device__ __forceinline__ int64_t xcd_contiguous_block() {
  const int64_t per = gridDim.x / kXcds;
  return (blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
}

// Before the first write of an edge's values to the stage: the previous edge's reads of it are done.
__device__ __forceinline__ void stage_is_free() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Sum over the 64 lanes of the N values that every lane has put into the stage (N * kStageStride elements owned by
// this wave, value a of lane i at [a * kStageStride + i]), in a fixed order, written to out[a]: lane 4a+q adds the
// sixteen lanes 16q..16q+15 of component a, then the four quarters are combined with two exchanges.
template <int N, typename T, typename TS>
__device__ __forceinline__ void lane_sum_store(const T* stage, int lane, TS* __restrict__ out) {
  static_assert(N <= 16, "one lane quartet per component");
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int a = lane >> 2, q = lane & 3;
  T s = T(0);
  if (a < N) {
#pragma unroll
    for (int i = 0; i < 16; ++i) s += stage[a * kStageStride + q * 16 + i];
  }
  s += __shfl_xor(s, 1);
  s += __shfl_xor(s, 2);
  if (q == 0 && a < N) out[a] = static_cast<TS>(s);
}

// The sums of a workgroup's waves, added in wave order by wave 0; true for that wave.  scratch: kStride >=
// N * kLanes values per wave, which nobody else reads or writes any more.
template <int kWaves, int kStride, typename T, int N>
__device__ __forceinline__ bool add_waves(int wave, int lane, T (&acc)[N], T* scratch) {
  static_assert(N * kLanes <= kStride, "the sums of a wave fit its scratch");
  stage_is_free();
  if (wave > 0) {
#pragma unroll
    for (int c = 0; c < N; ++c) scratch[wave * kStride + c * kLanes + lane] = acc[c];
  }
  __syncthreads();
  if (wave > 0) return false;
#pragma unroll
  for (int w = 1; w < kWaves; ++w)
#pragma unroll
    for (int c = 0; c < N; ++c) acc[c] += scratch[w * kStride + c * kLanes + lane];
  return true;
}

// Store of a wave's rows (N elements per lane, lane rows N elements apart = one contiguous block
// of 64*N elements) as whole lines: every lane's row goes through an LDS block of the same
// layout and comes back so that store instruction k writes the k-th contiguous KB of the block
// instead of 64 pieces of 16 bytes (partial lines, N*sizeof(T)/16 times the write requests);
// streamed past the cache.  stage: 64*N elements of LDS owned by this wave; block: where lane
// 0's row goes; live: lanes whose rows exist.  Rows that are no whole number of 16-byte pieces (9 values of
// 4 bytes) are aligned to their elements only and go out one element per lane and instruction.
template <typename TS, typename T, int N>
__device__ __forceinline__ void store_rows_coalesced(TS* __restrict__ block, TS* stage, int lane, const T (&v)[N], int live) {
  constexpr int V = (N * sizeof(TS)) % 16 == 0 ? 16 / sizeof(TS) : 1;
  typedef TS Vec __attribute__((ext_vector_type(V)));
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // earlier reads of the stage are done
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int j = 0; j < N / V; ++j) {
    Vec x;
#pragma unroll
    for (int k = 0; k < V; ++k) x[k] = static_cast<TS>(v[j * V + k]);
    *reinterpret_cast<Vec*>(stage + lane * N + j * V) = x;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the other lanes' pieces are visible
  __builtin_amdgcn_wave_barrier();
  const int pieces = live * N / V;
#pragma unroll
  for (int q0 = 0; q0 < kLanes * N / V; q0 += kLanes) {
    const int q = q0 + lane;
    if (live == kLanes || q < pieces) {
      const Vec x = *reinterpret_cast<const Vec*>(stage + q * V);
      __builtin_nontemporal_store(x, reinterpret_cast<Vec*>(block + q * V));
    }
  }
}

// Channels of block cb: the lane's channel (dead lanes repeat the last one) and the number of live lanes.
template <bool kFull>
struct Channels {
  int live, ch, first;   // first: channel of lane 0
  __device__ __forceinline__ Channels(int K, int cb, int lane) : first(cb * kLanes) {
    live = kFull ? kLanes : (K - cb * kLanes < kLanes ? K - cb * kLanes : kLanes);
    ch = cb * kLanes + (kFull || lane < live ? lane : live - 1);
  }
};

// A workgroup = one (atom, 64-channel block); its kWaves waves take every kWaves-th edge and add their sums at the end.
// With twenty edges an atom a wave per (atom, block), four atoms a workgroup, is slower at every size: it walks them in series where
// the chip has waves to spare, waits for the atom with the most edges where it has not, and its waves share no rows.
// Forward / backward / second-order pass, us, 128 channels, l_h = 1, wave -> workgroup per (atom, block): 250 atoms
// 21 -> 9 / 53 -> 24 / 78 -> 37, 2000 40 -> 37 / 100 -> 79 / 230 -> 193, 10 000 243 -> 225 / 500 -> 492 / 859 -> 817; l_h = 2
// (fp64 arithmetic), 3001 atoms 180 -> 165 / 368 -> 361 / 888 -> 817.
// Waves per SIMD that the forward is held to.  fp64 arithmetic on fp32 rows: with 10 to 17 paths it wants 129 registers if left alone, one
// over the limit for four; with 7 paths 91 for 78 (2000 atoms, 20 edges each, 29.5 -> 29.0 us, one edge 6.5 -> 6.1).
template <typename T, typename TS, typename G>
constexpr int kForwardWaves = sizeof(T) == 8 && sizeof(TS) == 4 ? (G::kP >= 10 && G::kP <= 17 ? 4 : G::kP == 7 ? 6 : 1) : 1;

// ... where an atom has few edges, so that a wave of the four has one or two and nothing to overlap: the registers that two edges under way
// take if left alone (fp32, l_h = 1, 105 for 58; fp64, l_max = 2, 116 for 74) are waves missing.  fp32, l_h = 1, us, left alone / held: 2000
// atoms with one edge each 8.2 / 6.5, four 12.9 / 11.8, eight 20.0 / 18.7, twenty 44.4 / 45.5; 10 000 with four 48.9 / 43.4, eight 96.2 / 94.7, ten
// 114 / 116, twenty 213 / 222.  fp64, l_max = 2: 2000 atoms with one 8.1 / 7.1, 10 000 with four 77.4 / 74.8, 2000 with eight 30.3 / 31.0.
template <typename T, typename TS, typename G>
constexpr int kFewEdgesWaves = sizeof(T) == 4 ? 8 : sizeof(TS) == 8 && G::kP == 7 ? 6 : kForwardWaves<T, TS, G>;
template <typename T>
constexpr int kFewEdges = sizeof(T) == 4 ? 9 : 4;     // edges an atom

template <typename T, typename TS, typename G, bool kFull, int kWaves, int kHold>
__global__ __launch_bounds__(kWaves * kLanes) __attribute__((amdgpu_waves_per_eu(kHold))) void forward_kernel(int K, int chblocks, int64_t unit0, int64_t n_units,
                                                           const TS* __restrict__ Y, const TS* __restrict__ h,
                                                           const TS* __restrict__ R,
                                                           const EdgeList el, TS* __restrict__ A) {
  __shared__ __attribute__((aligned(16))) T out_stage[kWaves][kLanes * G::kNout];
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = uniform(threadIdx.x / kLanes);
  const int64_t unit = unit0 + xcd_contiguous_block();
  if (unit >= n_units) return;   // the whole workgroup: its waves meet at the end
  const size_t node = unit / chblocks;
  const int cb = static_cast<int>(unit % chblocks);
  const Channels<kFull> chan(K, cb, lane);
  const int ch = chan.ch;
  const int e0 = uniform(el.first(node)) + wave, e1 = uniform(el.first(node + 1));
  T acc[G::kNout];
#pragma unroll
  for (int c = 0; c < G::kNout; ++c) acc[c] = T(0);
  if (e0 < e1) {
    TS r0[G::kP], r1[G::kP], h0[G::kNh], h1[G::kNh];
    UniformRow<T, TS, G::kNY> y0, y1;
    auto add_edge = [&](int e, const UniformRow<T, TS, G::kNY>& y_row, const TS (&h_row)[G::kNh], const TS (&r_row)[G::kP]) {
      T y[G::kNY], hh[G::kNh];
      y_row.use(Y, e, y);
      widen(h_row, hh);
      G::template forward<kDirect<TS>>(y, hh, PathRow<T, TS, G::kP>{r_row}, acc);
    };
    // No request stands under a condition: behind one the compiler waits for all of them, the one just made included, before
    // the arithmetic that is meant to overlap it.  Past the last edge a request repeats its last one, all lanes the same line.
    auto load_edge = [&](int e, int j, bool next, UniformRow<T, TS, G::kNY>& y_row, TS (&h_row)[G::kNh], TS (&r_row)[G::kP]) {
      const int c = next ? ch : cb * kLanes;
      y_row.request(Y, e, lane);
      load_weights<TS, G::kP>(R, e, K, c, r_row);
      load_row<TS, G::kNh>(h + (el.node(j) * K + c) * G::kNh, h_row);
      __builtin_amdgcn_sched_barrier(0);
    };
    load_edge(e0, el.raw(e0), true, y0, h0, r0);
    int jn = el.raw(e0 + kWaves < e1 ? e0 + kWaves : e0);  // sender of the next edge, read one step ahead
    int e = e0;
    for (; e + kWaves < e1; e += 2 * kWaves) {
      const bool third = e + 2 * kWaves < e1;
      const int eb = e + kWaves, ec = third ? e + 2 * kWaves : eb;
      const int jn2 = el.raw(ec);
      load_edge(eb, jn, true, y1, h1, r1);
      add_edge(e, y0, h0, r0);
      jn = el.raw(e + 3 * kWaves < e1 ? e + 3 * kWaves : ec);
      load_edge(ec, jn2, third, y0, h0, r0);
      add_edge(eb, y1, h1, r1);
    }
    if (e < e1) add_edge(e, y0, h0, r0);
  }
  if (!add_waves<kWaves, kLanes * G::kNout>(wave, lane, acc, out_stage[0])) return;
  store_rows_coalesced<TS, T, G::kNout>(A + (node * K + cb * kLanes) * G::kNout, reinterpret_cast<TS*>(out_stage[wave]),
                                        lane, acc, chan.live);
}

// receiver[e] for every edge, from the receivers' offsets: one thread per receiving atom.
__global__ __launch_bounds__(256) void edge_receiver_kernel(int64_t n_out_nodes, const EdgeList el,
                                                            int32_t* __restrict__ receiver) {
  const int64_t node = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (node >= n_out_nodes) return;
  const int e0 = el.first(node), e1 = el.first(node + 1);
  for (int e = e0; e < e1; ++e) receiver[e] = static_cast<int32_t>(node);
}

// Waves per SIMD that the backward kernels are held to.  With fp64 arithmetic and 10 to 17 paths the compiler takes a
// little over the 256 registers that leave room for two, and a second wave hides more than the registers do: with the
// conversions of r and the stores of dR and dY where their path has them (they waited for the end of the program
// before), l_h = 2 at 3001 atoms and 128 channels, backward 499 -> 361 us, second-order pass 1500 atoms 478 -> 410; 64
// channels, l = 2, l_h = 2, 2500 atoms 556 -> 193.
template <typename T, typename TS, typename G>
constexpr int kMinWaves = sizeof(T) == 8 && G::kP >= 10 && G::kP <= 17 ? 2 : 1;

// Receiving atoms up to which the workgroups of the backward find the receivers of their edges themselves (receivers_by_search): 64 edges of a
// wave at a time, by bisection of the receivers' offsets in LDS.
constexpr int kSearchNodes = 1024;

// The backward walks the edges grouped by SENDER: one workgroup = one (sending atom, kBlocks 64-channel blocks; BackwardBlocks).
// Its waves keep the atom's h rows and their dh sums in registers, walk the edges the atom sends
// (every kWaves-th in send_edge order: with the order of the waves, the order of the sum) and gather
// per edge the dA row of the receiver (rows of
// one structure, met in the XCD's L2) next to the edge's own R rows; dR and the blocks'
// share of dY leave per edge, dh leaves once per atom: no per-edge shares
// of dh go to memory and come back.  Atoms that send nothing get a zero row.  Every index is
// clamped where it is used.
template <typename T, typename TS, typename G, bool kFull, int kWaves, int kBlocks, bool kSearch>
__global__ __launch_bounds__(kWaves * kLanes) __attribute__((amdgpu_waves_per_eu(kMinWaves<T, TS, G>))) void backward_by_sender_kernel(
    int K, int groups, int64_t unit0, int64_t n_units, int64_t n_out_nodes, int n_edges, const TS* __restrict__ Y,
    const TS* __restrict__ h, const TS* __restrict__ R, const int32_t* __restrict__ send_ptr,
    const int32_t* __restrict__ send_edge, const int32_t* __restrict__ receiver, const int32_t* __restrict__ row_ptr,
    const TS* __restrict__ dA, TS* __restrict__ dR, TS* __restrict__ dY_partial, TS* __restrict__ dh) {
  __shared__ T stage_all[kWaves][G::kNY * kStageStride];
  __shared__ int32_t rows[kSearch ? kSearchNodes : 1];   // first edge of every receiving atom
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = uniform(threadIdx.x / kLanes);
  T* stage = stage_all[wave];
  const int64_t unit = unit0 + xcd_contiguous_block();
  if (unit >= n_units) return;   // the whole workgroup: its waves meet at the end
  const size_t node = unit / groups;
  const int group = static_cast<int>(unit % groups);
  const Channels<kFull> chan[2] = {Channels<kFull>(K, group * kBlocks, lane), Channels<kFull>(K, group * kBlocks + kBlocks - 1, lane)};
  auto pos = [&](int v) { return v < 0 ? 0 : (v > n_edges ? n_edges : v); };
  auto edge = [&](int q) {
    const int e = send_edge[q];
    return e < 0 ? 0 : (e >= n_edges ? n_edges - 1 : e);
  };
  auto atom = [&](int r) { return static_cast<size_t>(r < 0 ? 0 : (r >= n_out_nodes ? n_out_nodes - 1 : r)); };
  const int q0 = uniform(pos(send_ptr[node])) + wave, q1 = uniform(pos(send_ptr[node + 1]));
  // The edge at position q of this wave's (q0, q0 + kWaves, ...) and its receiver; past the last one any edge of the list.  kSearch: asked for
  // in order, 64 of them at a time, one a lane, the receiver by bisection of the rows in LDS.
  int my_e = 0, my_r = 0;
  auto next_edge = [&](int q, int& e, int& r) {
    if constexpr (kSearch) {
      const int i = static_cast<int>(static_cast<unsigned>(q - q0) / kWaves), last = (q1 - 1 - q0) / kWaves;
      if ((i & (kLanes - 1)) == 0) {
        my_e = edge(q0 + (i + lane < last ? i + lane : last) * kWaves);
        my_r = 0;
#pragma unroll
        for (int step = kSearchNodes / 2; step > 0; step /= 2) {
          const int at = my_r + step;
          if (at < n_out_nodes && rows[at < kSearchNodes ? at : 0] <= my_e) my_r = at;
        }
      }
      e = __builtin_amdgcn_readlane(my_e, i & (kLanes - 1));
      r = __builtin_amdgcn_readlane(my_r, i & (kLanes - 1));
    } else {
      e = uniform(edge(q < q1 ? q : q0));
      r = uniform(receiver[e]);
    }
  };
  if constexpr (kSearch) {
    for (int v = threadIdx.x; v < n_out_nodes; v += kWaves * kLanes) rows[v] = pos(row_ptr[v]);   // at most kSearchNodes
    __syncthreads();
  }
  T acc[kBlocks][G::kNh];
#pragma unroll
  for (int b = 0; b < kBlocks; ++b)
#pragma unroll
    for (int c = 0; c < G::kNh; ++c) acc[b][c] = T(0);
  if (q0 < q1) {
    TS h_row[kBlocks][G::kNh];
#pragma unroll
    for (int b = 0; b < kBlocks; ++b) load_row<TS, G::kNh>(h + (node * K + chan[b].ch) * G::kNh, h_row[b]);
    // One block: the row widened once.  (As with two, per edge, it takes registers: l = 3, l_h = 1 in fp32 130 for 126, of the 128 that four waves
    // per SIMD have.  us, per edge / once, 64 channels, 8000 atoms 192.3 / 189.7; fp64 rows, l_h = 0, 128 channels, 5000 atoms 327.6 / 319.8.)
    T h_one[G::kNh];
    if constexpr (kBlocks == 1) widen(h_row[0], h_one);
    TS r0[G::kP], g0[G::kNout];
    UniformRow<T, TS, G::kNY> y0;
    auto load_rows = [&](int e, int receiving, int ch, TS (&r_row)[G::kP], TS (&g_row)[G::kNout]) {
      load_weights<TS, G::kP>(R, e, K, ch, r_row);
      load_row<TS, G::kNout>(dA + (atom(receiving) * K + ch) * G::kNout, g_row);
    };
    int ea, ra;
    next_edge(q0, ea, ra);
    y0.request(Y, ea, lane);
    load_rows(ea, ra, chan[0].ch, r0, g0);
    // edge id and receiver of the edge after the current one, read one step ahead of its rows
    int en, rn;
    next_edge(q0 + kWaves, en, rn);

    // One edge and channel block: arithmetic, dR row stores, dh added up; with the last block dY summed over the 64 lanes in a fixed order.
    auto finish_block = [&](auto block, int e, const T (&y)[G::kNY], const TS (&r_row)[G::kP], const TS (&g_row)[G::kNout]) {
      constexpr int b = decltype(block)::value;
      T g[G::kNout], hh[G::kNh];
      const bool live = lane < chan[b].live;
      const PathStore<kFull, T, TS> dr{dR + static_cast<size_t>(e) * G::kP * K + chan[b].ch, static_cast<size_t>(K), live};
      const StageStore<kFull, (b > 0), T> dy{stage + lane, live};
      widen(g_row, g);
      if constexpr (kBlocks == 1) {
#pragma unroll
        for (int c = 0; c < G::kNh; ++c) hh[c] = h_one[c];
      } else {
        widen(h_row[b], hh);
      }
      if (b == 0) stage_is_free();
      // (fp32 rows, one ragged block, 17 paths and more: term by term 1 to 3% slower; 96 channels, l_h = 2, 900 atoms 111.4 / 108.2 us.  Full blocks the
      // other way: 64 channels, l = 2, l_h = 2, 3000 atoms 93 / 105.)
      if constexpr ((!kDirect<TS> || (kBlocks == 1 && !kFull && G::kP >= 17)) && G::kDhByTerms) {
        T share[G::kNh];
#pragma unroll
        for (int c = 0; c < G::kNh; ++c) share[c] = T(0);
        G::backward(y, hh, PathRow<T, TS, G::kP>{r_row}, g, dr, dy, share);
#pragma unroll
        for (int c = 0; c < G::kNh; ++c) acc[b][c] += share[c];
      } else {
        G::backward(y, hh, PathRow<T, TS, G::kP>{r_row}, g, dr, dy, acc[b]);
      }
      pin_values(acc[b]);
      if (b == kBlocks - 1) lane_sum_store<G::kNY>(stage, lane, dY_partial + (static_cast<size_t>(group) * n_edges + e) * G::kNY);
    };
    auto finish_edge = [&](int e, const UniformRow<T, TS, G::kNY>& y_row, const TS (&r_row)[G::kP], const TS (&g_row)[G::kNout]) {
      T y[G::kNY];
      y_row.use(Y, e, y);
      finish_block(std::integral_constant<int, 0>{}, e, y, r_row, g_row);
    };
    constexpr std::integral_constant<int, 0> first{};
    constexpr std::integral_constant<int, kBlocks - 1> last{};

    // one set of rows in registers where two do not fit (see the second-order kernel)
    constexpr bool kOneSet = sizeof(TS) == 8 && G::kP >= 17;
    if constexpr (kBlocks == 2) {
      // The rows of the edge's two blocks in two sets.  No request stands under a condition (see the forward).
      TS r1[G::kP], g1[G::kNout];
      for (int q = q0; q < q1; q += kWaves) {
        load_rows(ea, ra, chan[1].ch, r1, g1);
        __builtin_amdgcn_sched_barrier(0);
        T y[G::kNY];
        y0.use(Y, ea, y);
        int e2, r2;
        if constexpr (!kSearch) e2 = uniform(edge(q + 2 * kWaves < q1 ? q + 2 * kWaves : q0));
        finish_block(first, ea, y, r0, g0);
        y0.request(Y, en, lane);
        load_rows(en, rn, q + kWaves < q1 ? chan[0].ch : chan[0].first, r0, g0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kSearch) next_edge(q + 2 * kWaves, e2, r2);
        else r2 = uniform(receiver[e2]);
        finish_block(last, ea, y, r1, g1);
        ea = en;
        ra = rn;
        en = e2;
        rn = r2;
      }
    } else if constexpr (kOneSet) {
      for (int q = q0; q < q1; q += kWaves) {
        finish_edge(ea, y0, r0, g0);
        if (q + kWaves < q1) {
          ea = en;
          y0.request(Y, ea, lane);
          load_rows(ea, rn, chan[0].ch, r0, g0);
          if (q + 2 * kWaves < q1) next_edge(q + 2 * kWaves, en, rn);
        }
      }
    } else {
      TS r1[G::kP], g1[G::kNout];
      UniformRow<T, TS, G::kNY> y1;
      int eb = 0;
      for (int q = q0; q < q1; q += 2 * kWaves) {
        if (q + kWaves < q1) {
          eb = en;
          y1.request(Y, eb, lane);
          load_rows(eb, rn, chan[0].ch, r1, g1);
          if (q + 2 * kWaves < q1) next_edge(q + 2 * kWaves, en, rn);
        }
        finish_edge(ea, y0, r0, g0);
        if (q + kWaves < q1) {
          if (q + 2 * kWaves < q1) {
            ea = en;
            y0.request(Y, ea, lane);
            load_rows(ea, rn, chan[0].ch, r0, g0);
            if (q + 3 * kWaves < q1) next_edge(q + 3 * kWaves, en, rn);
          }
          finish_edge(eb, y1, r1, g1);
        }
      }
    }
  }
#pragma unroll
  for (int b = 0; b < kBlocks; ++b) {
    if (b > 0) __syncthreads();   // the first block's sums have been read
    if (add_waves<kWaves, G::kNY * kStageStride>(wave, lane, acc[b], stage_all[0]) && (kFull || lane < chan[b].live))
      store_row<TS, T, G::kNh>(dh + (node * K + chan[b].ch) * G::kNh, acc[b]);
  }
}

// Second-order pass: the backward's walk with the cotangents HR (per edge and path), Hh (at the
// sender) and HY (wave-uniform) as additional inputs; ddA of the receiver is summed in registers
// and stored once, d2R / d2Y partial / d2h share leave per edge like dR / dY / dh.
template <typename T, typename TS, typename G, bool kFull, int kWaves>
__global__ __launch_bounds__(kWaves * kLanes) __attribute__((amdgpu_waves_per_eu(kMinWaves<T, TS, G>))) void double_backward_kernel(
    int K, int chblocks, int64_t unit0, int64_t n_units, int64_t n_edges, const TS* __restrict__ Y, const TS* __restrict__ h,
    const TS* __restrict__ R, const EdgeList el,
    const TS* __restrict__ dA, const TS* __restrict__ HY, const TS* __restrict__ Hh, const TS* __restrict__ HR,
    TS* __restrict__ ddA, TS* __restrict__ d2R, TS* __restrict__ d2Y_partial, TS* __restrict__ d2h_edge) {
  __shared__ T stage_all[kWaves][G::kNY * kStageStride];
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = uniform(threadIdx.x / kLanes);
  T* stage = stage_all[wave];
  const int64_t unit = unit0 + xcd_contiguous_block();
  if (unit >= n_units) return;   // the whole workgroup: its waves meet at the end
  const size_t node = unit / chblocks;
  const int cb = static_cast<int>(unit % chblocks);
  const Channels<kFull> chan(K, cb, lane);
  const int ch = chan.ch;
  const int e0 = uniform(el.first(node)) + wave, e1 = uniform(el.first(node + 1));
  T dda[G::kNout];
#pragma unroll
  for (int c = 0; c < G::kNout; ++c) dda[c] = T(0);
  if (e0 < e1) {
    T g[G::kNout];
    {
      TS g_row[G::kNout];
      load_row<TS, G::kNout>(dA + (node * K + ch) * G::kNout, g_row);
      widen(g_row, g);
    }
    // The rows of two edges in registers where they fit; fp64 arithmetic with ten or more paths leaves room for one set,
    // whose next rows are requested when the arithmetic has consumed it (two sets: one wave per SIMD, or scratch).
    constexpr bool kOneSet = sizeof(T) == 8 && G::kP >= 10;
    TS r0[G::kP], q0[G::kP], h0[G::kNh], x0[G::kNh];
    UniformRow<T, TS, G::kNY> y0, hy0;
    auto load_edge = [&](int e, size_t j, TS (&r)[G::kP], TS (&q)[G::kP], TS (&h_row)[G::kNh], TS (&x_row)[G::kNh],
                         UniformRow<T, TS, G::kNY>& y_row, UniformRow<T, TS, G::kNY>& hy_row) {
      y_row.request(Y, e, lane);
      hy_row.request(HY, e, lane);
      load_weights<TS, G::kP>(R, e, K, ch, r);
      load_weights<TS, G::kP>(HR, e, K, ch, q);
      load_row<TS, G::kNh>(h + (j * K + ch) * G::kNh, h_row);
      load_row<TS, G::kNh>(Hh + (j * K + ch) * G::kNh, x_row);
    };
    load_edge(e0, el.snd(e0), r0, q0, h0, x0, y0, hy0);
    int jn = (e0 + kWaves < e1) ? el.raw(e0 + kWaves) : 0;

    auto finish_edge = [&](int e, const TS (&r_row)[G::kP], const TS (&hr_row)[G::kP], const TS (&h_row)[G::kNh],
                           const TS (&hx_row)[G::kNh], const UniformRow<T, TS, G::kNY>& y_row,
                           const UniformRow<T, TS, G::kNY>& hy_row) {
      T y[G::kNY], hy[G::kNY], hh[G::kNh], hx[G::kNh], d2h[G::kNh];
      const PathStore<kFull, T, TS> d2r{d2R + static_cast<size_t>(e) * G::kP * K + ch, static_cast<size_t>(K), lane < chan.live};
      const StageStore<kFull, false, T> d2y{stage + lane, lane < chan.live};
      pin_values(g);
      y_row.use(Y, e, y);
      hy_row.use(HY, e, hy);
      widen(h_row, hh);
      widen(hx_row, hx);
      stage_is_free();
      G::template double_backward<kDirect<TS>>(y, hy, hh, hx, PathRow<T, TS, G::kP>{r_row}, PathRow<T, TS, G::kP>{hr_row}, g, dda, d2r, d2y, d2h);
      pin_values(dda);
      pin_values(d2h);
      if (kFull || lane < chan.live) store_row<TS, T, G::kNh>(d2h_edge + (static_cast<size_t>(e) * K + ch) * G::kNh, d2h);
      lane_sum_store<G::kNY>(stage, lane, d2Y_partial + (static_cast<size_t>(cb) * n_edges + e) * G::kNY);
    };

    if constexpr (kOneSet) {
      for (int e = e0; e < e1; e += kWaves) {
        finish_edge(e, r0, q0, h0, x0, y0, hy0);
        if (e + kWaves < e1) {
          load_edge(e + kWaves, el.node(jn), r0, q0, h0, x0, y0, hy0);
          if (e + 2 * kWaves < e1) jn = el.raw(e + 2 * kWaves);
        }
      }
    } else {
      TS r1[G::kP], q1[G::kP], h1[G::kNh], x1[G::kNh];
      UniformRow<T, TS, G::kNY> y1, hy1;
      for (int e = e0; e < e1; e += 2 * kWaves) {
        int jn2 = 0;
        if (e + kWaves < e1) {
          load_edge(e + kWaves, el.node(jn), r1, q1, h1, x1, y1, hy1);
          if (e + 2 * kWaves < e1) jn2 = el.raw(e + 2 * kWaves);
        }
        finish_edge(e, r0, q0, h0, x0, y0, hy0);
        if (e + kWaves < e1) {
          if (e + 2 * kWaves < e1) {
            load_edge(e + 2 * kWaves, el.node(jn2), r0, q0, h0, x0, y0, hy0);
            if (e + 3 * kWaves < e1) jn = el.raw(e + 3 * kWaves);
          }
          finish_edge(e + kWaves, r1, q1, h1, x1, y1, hy1);
        }
      }
    }
  }
  if (!add_waves<kWaves, G::kNY * kStageStride>(wave, lane, dda, stage_all[0])) return;
  if (kFull || lane < chan.live) store_row<TS, T, G::kNout>(ddA + (node * K + ch) * G::kNout, dda);
}


// Calls launch(first unit, grid) until all units (a workgroup each) are served: a grid holds less than 2^32 threads.
template <typename F>
hipError_t for_all_units(int64_t n_units, F&& launch) {
  constexpr int64_t kMost = int64_t(1) << 23;
  for (int64_t unit0 = 0; unit0 < n_units; unit0 += kMost) {
    const int64_t blocks = n_units - unit0 < kMost ? n_units - unit0 : kMost;
    launch(unit0, dim3(static_cast<unsigned>((blocks + kXcds - 1) / kXcds * kXcds)));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Waves that share the edges of an atom: four, or two where most atoms have fewer edges than four waves and there are
// atoms enough to fill the chip with the waves that have one.  Two / four, 128 channels, l_h = 0 and 1, forward, backward, second-order
// pass: 10 000 atoms with one edge each 0.91, 0.76, 0.78 of the time, with three 0.97, 0.91, 0.87; 30 000 with three 0.96, 0.86, 0.87,
// with four, l_h = 1, 1.03, 0.93, 0.92, with twenty (10 000, 64 channels) 1.05, 1.2, 1.02; 3000 atoms with two 0.92, 1.1, 0.92.
int waves_per_unit(int64_t n_edges, int64_t n_atoms, int64_t n_units) {
  return n_edges <= 3 * n_atoms && n_units >= 8192 ? 2 : 4;
}

// Channel blocks of an atom that a workgroup of the backward walks together.  Two: their shares of dY are added in the lanes, one sum over the
// lanes serves both, and with two blocks in all it is dY (no shares through memory, no launch that adds them).  But half the workgroups, so small
// graphs have eight waves share the edges, and a second row in registers.  Backward with the sum of the shares, us; 128 channels, one / two
// / two and eight waves:
//   l = 3, l_h = 1, fp32      60 atoms 16.8 / 20.6 / 14.0   250 24.4 / 26.9 / 19.5   1000 43.5 / 45.5 / 41.6   2000 78.6 / 80.0 / 76.0
//                             2060 109.1 / 111.6   2700 138.6 / 140.6   4500 221.4 / 221.4   5000 243.3 / 241.8   10 000 466 / 460 / 473
//   l = 3, l_h = 0, fp32      250 16.8 / 15.5 / 10.4   2700 83.1 / 82.3   4000 114.5 / 115.3   9000 240 / 237
//   fp32 rows in fp64 arithmetic (their shares of dY as fp64 are summed once):
//   l = 2, l_h = 1            250 21.5 / 20.2 / 16.6   1000 39.9 / 33.2 / 32.9   4000 140.7 / 127.3 / 134.7
//   l = 2, l_h = 2            250 27.1 / 27.2 / 23.7   1000 63.1 / 56.4 / 64.1   3000 191 / 175
//   96 channels, l_h = 1      250 30.0 / 31.8 / 25.7   2000 124.3 / 102.2 / 130.7
//   17 paths (255 registers)  250 40.2 / 47.5 / 42.9   1000 104.9 / 106.2 / 113.5   3001 315 / 305   23 paths 2100 421 / 390   3001 579 / 546
//   96 channels, 17 paths     900 108 / 113   1300 150 / 147   1755 196 / 186   23 paths 1000 224 / 229   1700 371 / 366
// fp64 rows are bound by what a compute unit takes in (12 KB per edge and block), and 17 paths spill: two only where the second block is half empty
// or the shares of dY are long:
//   l = 3, l_h = 1            330 45.6 / 50.8   1100 132.8 / 137   1800 206.5 / 205   3000 327.9 / 323.1   4500 482 / 466
//   l = 3, l_h = 0            42 15.7 / 19.2   250 25.2 / 26.0   700 47.9 / 48.9   3000 188.5 / 190.3
//   l = 2, l_h = 1, 1500      109.4 / 113.3   2500 172.5 / 174.9   4000 268.8 / 269.7     l = 2, l_h = 2, 2000 210.4 / 214.0   3500 357.2 / 356.8
//   96 channels, l_h = 1      250 26.3 / 25.5   400 34.0 / 29.6   1500 81.4 / 71.6   3000 315 / 272
// With more than two blocks the shares are added up all the same; 256 channels:
//   l_h = 1, fp32             127 22.5 / 22.1   500 46.2 / 47.2   1000 80.6 / 84.4   3000 286.7 / 286.2
//   l = 2, l_h = 1            330 31.2 / 33.1   1500 98.3 / 89.6   3000 212.5 / 200.9      17 paths 1100 236 / 232   1500 316 / 306   23 paths 1100 416 / 402
//   fp64 rows, l_h = 1        330 76.4 / 82.6   1500 316.7 / 316.3
template <typename T, typename TS, typename G, bool kFull>
struct BackwardBlocks {
  static constexpr bool kSingle = sizeof(T) == 4, kRows64 = sizeof(TS) == 8, kManyPaths = G::kP >= 17;
  // Are there workgroups of two blocks, some whose edges find their receivers themselves (receivers_by_search: small graphs), and some of eight
  // waves, up to how many workgroups?
  static constexpr bool kTwo = !kRows64 || (!kManyPaths && (!kFull || (G::kNY == 16 && G::kNh > 1)));
  static constexpr bool kTwoSearch = kTwo && (kRows64 ? !kFull : !kManyPaths);
  static constexpr int64_t kEightWaves = kRows64 || kManyPaths ? 0 : kSingle ? 2048 : 512;
  static bool two(int chblocks, int64_t n_in) {
    if (!kTwo || chblocks % 2 != 0) return false;
    if (kRows64) return chblocks == 2 && n_in >= (kFull ? 1792 : 384);
    if (chblocks > 2) return !kSingle && n_in * (chblocks / 2) > 2048;
    if (kSingle) return G::kNh == 1 || n_in <= kEightWaves || n_in > 4608;
    return !kManyPaths || n_in >= (kFull ? 2048 : 1280);
  }
};

// Do the workgroups of the backward search for the receivers of their edges?  It saves the launch that writes every edge's receiver and costs
// each workgroup the rows in LDS and about ten reads there per 64 edges of a wave: it pays up to some number of workgroups (six per compute
// unit), and the rows are kSearchNodes at most.  Receivers and backward, us, with the launch / searched, by workgroups:
//   128 channels, fp32      l_h = 0    42 9.6 / 8.3     330 19.2 / 14.9    1000 27.5 / 25.1
//                           l_h = 1    127 19.9 / 15.6  330 28.5 / 23.4    1000 46.0 / 42.4
//   l = 2, l_h = 2          250 28.8 / 24.5
//   256 channels, l_h = 1   1320 39.0 / 36.2    2800 60.5 / 60.1    l = 2 1400 52.2 / 53.7
//   17 paths                500 41.3 / 37.0     2000 106.1 / 107.3
//   fp64 rows, l_h = 1      660 46.3 / 44.6     2000 89.8 / 89.7
inline bool receivers_by_search(int64_t n_out_nodes, int64_t n_units) { return n_out_nodes <= kSearchNodes && n_units <= 1536; }

EdgeList edge_list(const FwdArgs& a) {
  return EdgeList{a.sender, a.row_ptr, static_cast<int>(a.n_in), static_cast<int>(a.n_edges)};
}
EdgeList edge_list(const BwdArgs& a) {
  return EdgeList{a.sender, a.row_ptr, static_cast<int>(a.n_in), static_cast<int>(a.n_edges)};
}

// Launches of one instance; chblocks = 64-channel blocks, the last one may be ragged (kFull = false).
template <typename T, typename TS, typename G, bool kFull>
struct Launch {
  static hipError_t forward(const tp_plan* plan, const FwdArgs& a, hipStream_t stream) {
    const int K = plan->cfg.num_channels, chblocks = (K + kLanes - 1) / kLanes;
    const int64_t n_units = a.n_out_nodes * chblocks;
    const int waves = waves_per_unit(a.n_edges, a.n_out_nodes, n_units);
    constexpr int kUsual = kForwardWaves<T, TS, G>, kFew = kFewEdgesWaves<T, TS, G>;
    const auto kernel = waves == 2                                         ? &forward_kernel<T, TS, G, kFull, 2, kUsual>
                        : a.n_edges <= kFewEdges<T> * a.n_out_nodes ? &forward_kernel<T, TS, G, kFull, 4, kFew>
                                                                    : &forward_kernel<T, TS, G, kFull, 4, kUsual>;
    return for_all_units(n_units, [&](int64_t unit0, dim3 grid) {
      hipLaunchKernelGGL(kernel, grid, dim3(waves * kLanes), 0, stream, K, chblocks, unit0, n_units,
                         static_cast<const TS*>(a.Y), static_cast<const TS*>(a.h), static_cast<const TS*>(a.R),
                         edge_list(a), static_cast<TS*>(a.A));
    });
  }

  typedef BackwardBlocks<T, TS, G, kFull> Blocks;
  static hipError_t backward(const tp_plan* plan, const BwdArgs& a, hipStream_t stream) {
    const int K = plan->cfg.num_channels, chblocks = (K + kLanes - 1) / kLanes;
    const int groups = a.dY_parts, blocks = chblocks / groups;
    const int64_t n_units = a.n_in * groups;
    const bool search = receivers_by_search(a.n_out_nodes, n_units) && (blocks == 1 || Blocks::kTwoSearch);
    int32_t* receiver = static_cast<int32_t*>(a.dh_edge);   // the shares' part of the workspace is free on this path
    if (a.n_edges > 0 && a.n_out_nodes > 0 && !search) {
      hipLaunchKernelGGL(edge_receiver_kernel, dim3(static_cast<unsigned>((a.n_out_nodes + 255) / 256)), dim3(256), 0,
                         stream, a.n_out_nodes, edge_list(a), receiver);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    int waves = search ? 4 : waves_per_unit(a.n_edges, a.n_in, a.n_in * chblocks);
    auto kernel = search ? &backward_by_sender_kernel<T, TS, G, kFull, 4, 1, true>
                : waves == 4 ? &backward_by_sender_kernel<T, TS, G, kFull, 4, 1, false> : &backward_by_sender_kernel<T, TS, G, kFull, 2, 1, false>;
    if constexpr (Blocks::kTwo) {
      if (blocks == 2) {
        kernel = waves == 4 ? &backward_by_sender_kernel<T, TS, G, kFull, 4, 2, false> : &backward_by_sender_kernel<T, TS, G, kFull, 2, 2, false>;
        if constexpr (Blocks::kTwoSearch) {
          if (search) kernel = &backward_by_sender_kernel<T, TS, G, kFull, 4, 2, true>;
        }
        if constexpr (Blocks::kEightWaves > 0) {
          if (n_units <= Blocks::kEightWaves && a.n_edges > 4 * a.n_in) {
            waves = 8;
            kernel = search ? &backward_by_sender_kernel<T, TS, G, kFull, 8, 2, true> : &backward_by_sender_kernel<T, TS, G, kFull, 8, 2, false>;
          }
        }
      }
    }
    // without receivers or edges no list is walked: every atom gets its zero row
    const int n_edges = a.n_out_nodes > 0 ? static_cast<int>(a.n_edges) : 0;
    return for_all_units(n_units, [&](int64_t unit0, dim3 grid) {
      hipLaunchKernelGGL(kernel, grid, dim3(waves * kLanes), 0, stream, K, groups, unit0,
                         n_units, a.n_out_nodes, n_edges, static_cast<const TS*>(a.Y), static_cast<const TS*>(a.h),
                         static_cast<const TS*>(a.R), a.send_ptr, a.send_edge, receiver, a.row_ptr,
                         static_cast<const TS*>(a.dA), static_cast<TS*>(a.dR), static_cast<TS*>(a.dY_partial), static_cast<TS*>(a.dh));
    });
  }

  static int dY_parts(int chblocks, int64_t n_in) { return Blocks::two(chblocks, n_in) ? chblocks / 2 : chblocks; }

  static hipError_t double_backward(const tp_plan* plan, const DblArgs& d, hipStream_t stream) {
    const BwdArgs& a = d.b;
    const int K = plan->cfg.num_channels, chblocks = (K + kLanes - 1) / kLanes;
    const int64_t n_units = a.n_out_nodes * chblocks;
    const int waves = waves_per_unit(a.n_edges, a.n_out_nodes, n_units);
    const auto kernel = waves == 4 ? &double_backward_kernel<T, TS, G, kFull, 4> : &double_backward_kernel<T, TS, G, kFull, 2>;
    return for_all_units(n_units, [&](int64_t unit0, dim3 grid) {
      hipLaunchKernelGGL(kernel, grid, dim3(waves * kLanes), 0, stream, K, chblocks, unit0,
                         n_units, a.n_edges, static_cast<const TS*>(a.Y), static_cast<const TS*>(a.h),
                         static_cast<const TS*>(a.R), edge_list(a), static_cast<const TS*>(a.dA),
                         static_cast<const TS*>(d.HY), static_cast<const TS*>(d.Hh), static_cast<const TS*>(d.HR),
                         static_cast<TS*>(d.ddA), static_cast<TS*>(a.dR), static_cast<TS*>(a.dY_partial),
                         static_cast<TS*>(a.dh_edge));
    });
  }
};

// Calls fn.template operator()<Launch<...>>() for the instance that serves the plan.
template <typename G, typename F>
auto with_instance(const tp_plan* plan, F&& fn) {
  constexpr bool kSingle = G::kLY == 3 && G::kLout == 3 && G::kLh <= 1;   // fp32 arithmetic on full blocks (see the top)
  typedef typename std::conditional<kSingle, float, double>::type F32Full;
  const bool full = plan->cfg.num_channels % kLanes == 0;
  if (plan->cfg.dtype == SC_F64)
    return full ? fn.template operator()<Launch<double, double, G, true>>() : fn.template operator()<Launch<double, double, G, false>>();
  return full ? fn.template operator()<Launch<F32Full, float, G, true>>() : fn.template operator()<Launch<double, float, G, false>>();
}

struct ForwardFn {
  const tp_plan* plan; const FwdArgs& a; hipStream_t stream;
  template <typename L> hipError_t operator()() const { return L::forward(plan, a, stream); }
};
struct BackwardFn {
  const tp_plan* plan; const BwdArgs& a; hipStream_t stream;
  template <typename L> hipError_t operator()() const { return L::backward(plan, a, stream); }
};
struct PartsFn {
  int chblocks; int64_t n_in;
  template <typename L> int operator()() const { return L::dY_parts(chblocks, n_in); }
};
struct DoubleBackwardFn {
  const tp_plan* plan; const DblArgs& a; hipStream_t stream;
  template <typename L> hipError_t operator()() const { return L::double_backward(plan, a, stream); }
};

// What tp_spec.hip needs to know of one generated shape.
template <typename G>
struct GeneratedShape {
  static hipError_t forward(const tp_plan* p, const FwdArgs& a, hipStream_t s) { return with_instance<G>(p, ForwardFn{p, a, s}); }
  static hipError_t backward(const tp_plan* p, const BwdArgs& a, hipStream_t s) { return with_instance<G>(p, BackwardFn{p, a, s}); }
  static hipError_t double_backward(const tp_plan* p, const DblArgs& a, hipStream_t s) {
    return with_instance<G>(p, DoubleBackwardFn{p, a, s});
  }
  static int dY_parts(const tp_plan* p, int64_t n_in) {
    return with_instance<G>(p, PartsFn{(p->cfg.num_channels + kLanes - 1) / kLanes, n_in});
  }
  static SpecEntry entry() {
    return SpecEntry{G::kLY, G::kLh, G::kLout, G::kP, G::kOps, G::kFlops, &forward, &backward, &double_backward, &dY_parts};
  }
};

}  // namespace
}  // namespace tp
