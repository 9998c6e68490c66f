// Pieces of the channel-mixing linear's MFMA kernels that the fused linear + contraction kernel
// shares: operand layouts of the 16x16x4 instruction, 64-byte row access, and the LDS-staged
// product of one 16-atom row tile.
#pragma once
#include "sc_internal.h"

namespace el {

using sc::kLanes;

constexpr int kWaves = 4;
constexpr int kThreads = kWaves * kLanes;

template <typename T>
struct Mma;
template <>
struct Mma<float> {
  typedef float acc_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc_t mma(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane / 16) + r; }
};
template <>
struct Mma<double> {
  typedef double acc_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * r + lane / 16; }
};

__host__ __device__ constexpr int order_of(int c) { return c >= 9 ? 3 : c >= 4 ? 2 : c >= 1 ? 1 : 0; }

// N consecutive elements (16-byte accesses when the row is a multiple of 16 bytes).
template <typename T, int N>
__device__ __forceinline__ void load_row(const T* __restrict__ p, T (&v)[N]) {
  constexpr int V = 16 / sizeof(T);
  if constexpr ((N * sizeof(T)) % 16 == 0) {
    typedef T Vec __attribute__((ext_vector_type(V)));
#pragma unroll
    for (int i = 0; i < N; i += V) {
      const Vec x = *reinterpret_cast<const Vec*>(p + i);
#pragma unroll
      for (int k = 0; k < V; ++k) v[i + k] = x[k];
    }
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = p[i];
  }
}

// The same from an address that is aligned to its elements only (16-byte accesses need no more on this chip).
template <typename T, int N>
__device__ __forceinline__ void load_unaligned(const T* __restrict__ p, T (&v)[N]) {
  constexpr int V = 16 / sizeof(T);
  typedef T Vec __attribute__((ext_vector_type(V), aligned(sizeof(T))));
#pragma unroll
  for (int i = 0; i + V <= N; i += V) {
    const Vec x = *reinterpret_cast<const Vec*>(p + i);
#pragma unroll
    for (int k = 0; k < V; ++k) v[i + k] = x[k];
  }
#pragma unroll
  for (int i = N / V * V; i < N; ++i) v[i] = p[i];
}

template <typename T, int N>
__device__ __forceinline__ void store_row(T* __restrict__ p, const T (&v)[N]) {
  constexpr int V = 16 / sizeof(T);
  if constexpr ((N * sizeof(T)) % 16 == 0) {
    typedef T Vec __attribute__((ext_vector_type(V)));
#pragma unroll
    for (int i = 0; i < N; i += V) {
      Vec x;
#pragma unroll
      for (int k = 0; k < V; ++k) x[k] = v[i + k];
      *reinterpret_cast<Vec*>(p + i) = x;
    }
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = v[i];
  }
}

// The same product for fp32 and l_max = 3 (64-byte rows) with the A operands shared through
// LDS.  In the kernel above each of the four waves reads the whole X tile itself; those
// 16-byte accesses to 32 cache lines per instruction keep the vector memory path as busy as the
// matrix cores (measured: 30 us per row tile against 15 us of matrix time).  Here the
// workgroup stages X in chunks of 16 reduction channels (16 atoms x 16 channels x 64 B = 16 KB,
// two buffers): every thread loads 64 contiguous bytes once, all waves read their A operands
// from LDS (rows padded by 16 B against bank conflicts).  B operands (this wave's columns of
// W) are read from global memory one MFMA step ahead.  k_red % 16 == 0, k_cols % 128 == 0.
constexpr int kChunk = 16;                       // reduction channels per LDS chunk
constexpr int kRowPad = kChunk * 16 + 4;         // floats per atom row in LDS
constexpr int kBuffers = 2;                      // LDS buffers of 16 * kRowPad floats per workgroup

// lds_tile_product: the accumulators of rows n0..n0+15 and of this wave's CT column tiles of column
// group g (columns jc[t] per lane); xs = the workgroup's two staging buffers.
template <int CT>
__device__ __forceinline__ void lds_tile_product(int64_t n_nodes, int64_t n0, int g, int k_red, int k_cols,
                                                 const float* __restrict__ X, const float* __restrict__ W,
                                                 float* xs /* kBuffers * 16 * kRowPad floats */, typename Mma<float>::acc_t (&acc)[16][CT],
                                                 int (&jc)[CT]) {
  constexpr int NC = 16, L = 4, SPC = kChunk / 4;   // SPC: MFMA steps per chunk
  static_assert(SPC == 4, "the B operand sets rotate with period 4");
  typedef Mma<float>::acc_t acc_t;
  typedef float V4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int kq = lane / 16;
  const int chunks = k_red / kChunk;
  // staging role of this thread: atom tid/16 of the tile, reduction channel tid%16 of the chunk
  const int sn = threadIdx.x / 16, sk = threadIdx.x % 16;
  float* const swr = xs + sn * kRowPad + sk * 16;
  const float* const ard = xs + (lane & 15) * kRowPad + kq * 16;   // A operands of MFMA step 0 of a chunk
  int64_t ns = n0 + sn;
  if (ns >= n_nodes) ns = n_nodes - 1;       // rows past the end stage a valid atom and are not stored
  const float* xsrc = X + (static_cast<size_t>(ns) * k_red + sk) * NC;
#pragma unroll
  for (int t = 0; t < CT; ++t) jc[t] = ((g + t) * kWaves + wave) * 16 + (lane & 15);
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int t = 0; t < CT; ++t) acc[c][t] = acc_t{0, 0, 0, 0};

  auto gload = [&](int chunk, V4 (&x)[4]) {
    const V4* p = reinterpret_cast<const V4*>(xsrc + static_cast<size_t>(chunk) * kChunk * NC);
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = p[i];
  };
  auto stage = [&](int buf, const V4 (&x)[4]) {
    V4* p = reinterpret_cast<V4*>(swr + buf * 16 * kRowPad);
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = x[i];
  };
  // B operands through a buffer descriptor of W: per load one 32-bit per-lane byte offset (it
  // advances by one MFMA step = 4 rows of W) and a scalar offset for the order, no 64-bit address
  // arithmetic in the loop; a read past the end of W would return zero instead of faulting.
  unsigned boff[CT];
#pragma unroll
  for (int t = 0; t < CT; ++t) boff[t] = static_cast<unsigned>(kq * k_cols + jc[t]) * 4u;
  const unsigned bstep = static_cast<unsigned>(k_cols) * 16u;                    // bytes per MFMA step
  const unsigned lstride = static_cast<unsigned>(k_red) * k_cols * 4u;           // bytes per order
  const __amdgpu_buffer_rsrc_t wrs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(W), 0, static_cast<int>(L * lstride), 0x00020000);
  const int steps = chunks * SPC;
  auto bload = [&](int step, float (&b)[L][CT]) {   // B operands of one MFMA step
    const unsigned so = static_cast<unsigned>(step < steps ? step : steps - 1) * bstep;   // past the end: the last step again
#pragma unroll
    for (int l = 0; l < L; ++l)
#pragma unroll
      for (int t = 0; t < CT; ++t)
        b[l][t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wrs, static_cast<int>(boff[t] + so),
                                                                                 static_cast<int>(l * lstride), 0));
  };

  // Two LDS buffers, one barrier per chunk; B operands are requested kBDist MFMA steps before
  // their use (four register sets, of which kBDist + 1 are live at a time).
  constexpr int kBDist = 2;
  V4 xr[4];
  float b[4][L][CT];
  __syncthreads();                           // the previous unit's reads of both buffers are done
  gload(0, xr);
#pragma unroll
  for (int d = 0; d < kBDist; ++d) bload(d, b[d]);
  stage(0, xr);
  if (chunks > 1) gload(1, xr);
  __syncthreads();
  for (int c = 0; c < chunks; ++c) {
    const float* abuf = ard + (c & 1) * 16 * kRowPad;
#pragma unroll
    for (int st = 0; st < SPC; ++st) {       // SPC == 4: the roles of the four B sets repeat per chunk
      bload(c * SPC + st + kBDist, b[(st + kBDist) & 3]);
      const V4* p = reinterpret_cast<const V4*>(abuf + st * 4 * 16);
      V4 a4[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a4[i] = p[i];
#pragma unroll
      for (int cc = 0; cc < NC; ++cc)
#pragma unroll
        for (int t = 0; t < CT; ++t)
          acc[cc][t] = Mma<float>::mma(a4[cc / 4][cc % 4], b[st & 3][order_of(cc)][t], acc[cc][t]);
    }
    if (c + 1 < chunks) {
      stage((c + 1) & 1, xr);
      if (c + 2 < chunks) gload(c + 2, xr);
    }
    __syncthreads();
  }
}

// ---- the same product on the bfloat16 matrix cores
//
// An fp32 value of magnitude 2^-110 or more is the exact sum of three bfloat16 values (rounded to nearest: h, then what
// is left: m, then l; 8 + 8 + 8 bits), |m| <= 2^-8 |x|, |l| <= 2^-17 |x|.  Below, its last bits may be under 2^-133, the last
// bit that a bfloat16 has, and the sum is another value: split_pair notes it.  (The matrix core takes subnormal parts as they are.)
// Of the nine products of the parts, l l (at most 2^-34 of |x w|) is left out.  An instruction sums its products and the accumulator
// in fp32 and cuts smaller products off at the last bit of the largest; the seven products with an m or an l are therefore
// summed by themselves, which costs 2^-8 of that error, and join the sum of the h h once per 32 channels.
typedef __bf16 Bf8 __attribute__((ext_vector_type(8)));
typedef unsigned U4 __attribute__((ext_vector_type(4)));

struct SplitPair {   // two values, a 16-bit half each
  unsigned h, m, l;
};
__device__ __forceinline__ unsigned pack_bf16(float x, float y) {
  typedef float F2 __attribute__((ext_vector_type(2)));
  typedef __bf16 B2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(unsigned, __builtin_convertvector(F2{x, y}, B2));
}
__device__ __forceinline__ float low_half(unsigned u) { return __builtin_bit_cast(float, u << 16); }
__device__ __forceinline__ float high_half(unsigned u) { return __builtin_bit_cast(float, u & 0xffff0000u); }
// left: collects what l stands for; its low 16 bits stay zero as long as every value is the sum of its parts.
__device__ __forceinline__ SplitPair split_pair(float x, float y, unsigned& left) {
  SplitPair s;
  s.h = pack_bf16(x, y);
  const float rx = x - low_half(s.h), ry = y - high_half(s.h);
  s.m = pack_bf16(rx, ry);
  const float tx = rx - low_half(s.m), ty = ry - high_half(s.m);
  s.l = pack_bf16(tx, ty);
  left |= __builtin_bit_cast(unsigned, tx) | __builtin_bit_cast(unsigned, ty);
  asm volatile("" : "+v"(left));             // collected here: put off, the compiler holds two registers of every pair
  return s;
}

// A pass: R row tiles of 16 atoms (R = 1, 2) times the 128 columns from j0 on, by a workgroup of eight waves.  Wave w owns the 32
// columns of w % 4 and, of the sixteen components, the eight of two orders: 0 and 3, or 1 and 2 (w / 4).  So every value
// of X that is read from LDS serves two column tiles, every part of W that a wave holds all row tiles, and nothing is split
// twice within a pass.  k_red % 32 == 0.
//
// Steps (chunk of 32 reduction channels, row tile).  The rows of a step are split into three planes of [component][eight
// channels][atom] bfloat16, the A operands as the instruction reads them; the planes have two slots, and while the matrix cores work on
// one step the next one is split into the other slot, a pair of values per thread between the products of two components
// (one barrier a step).  A wave splits its own columns of W, an order right after that order's last products of the chunk,
// requested an order ahead.
constexpr int kSplitWaves = 8;
constexpr int kSplitThreads = kSplitWaves * kLanes;
constexpr int kSplitChunk = 32;
constexpr int kSplitRows = 2;                               // row tiles of a pass
constexpr int kSplitEight = 16 * 4 + 4;                     // 32-bit words (two channels each) of eight channels of the 16 atoms
constexpr int kSplitComp = 4 * kSplitEight + 4;             // ... of a component
constexpr int kSplitPlane = 16 * kSplitComp;                // ... of a part of a row tile
constexpr int kSplitSlot = 3 * kSplitPlane;                 // ... of a row tile

// Results leave through LDS, four atoms x 128 columns at a time (rows of 16 components padded to 80 bytes), two stages in turn.
constexpr int kSplitStage = 4 * 128 * 20;
static_assert(2 * kSplitStage <= 2 * kSplitSlot, "the stages reuse the planes");

template <int G>
struct SplitOrders {   // the two orders of wave group G, the shorter one first
  static constexpr int lo = G == 0 ? 0 : 1, hi = 3 - lo, n_lo = 2 * lo + 1;
  static constexpr int component(int i) { return i < n_lo ? lo * lo + i : hi * hi + i - n_lo; }
};

struct SplitArgs {
  int64_t n_nodes;
  int k_red, k_cols;
  const float* X;
  const float* W;
  float* Y;
};

// kTrans: W is [order][column][reduction channel], a lane's eight channels are contiguous.
template <int R, bool kTrans, int G>
struct SplitPass {
  typedef SplitOrders<G> O;
  typedef Mma<float>::acc_t acc_t;
  typedef float V4 __attribute__((ext_vector_type(4)));
  typedef float V2 __attribute__((ext_vector_type(2)));
  static constexpr int NC = 16;

  // The fp32 products of the same results, operands straight from memory: what the parts do not serve, a row tile (X) or a wave's
  // columns (W) at a time.  Forward, us, with no such value / one weight / one value of X / one in a tenth of the tiles / one in each atom:
  // 128 -> 128 channels, 4096 atoms 23 / 43 / 53 / 54 / 56, 10 000 56 / 109 / 72 / 89 / 146 (mfma_forward_lds_kernel 61), 256 -> 256, 4096
  // 64 / 133 / 131 / 129 / 187.  With both tiles of a pass computed again for a value in one: 10 000 atoms 99 for one value of X, 117 in a tenth.
  static __device__ __forceinline__ void plain(const SplitArgs& p, int64_t n0, int jc, int q, int i16, acc_t (&acc)[8][2]) {
    const int64_t na = n0 + i16 < p.n_nodes ? n0 + i16 : p.n_nodes - 1;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int t = 0; t < 2; ++t) acc[i][t] = acc_t{0, 0, 0, 0};
    for (int k = q; k < p.k_red; k += 4) {
      float a[NC], b[2][2];
      load_row<float, NC>(p.X + (static_cast<size_t>(na) * p.k_red + k) * NC, a);
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int l = o == 0 ? O::lo : O::hi;
          b[o][t] = p.W[kTrans ? (static_cast<size_t>(l) * p.k_cols + jc + t) * p.k_red + k
                               : (static_cast<size_t>(l) * p.k_red + k) * p.k_cols + jc + t];
        }
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[i][t] = Mma<float>::mma(a[O::component(i)], b[i < O::n_lo ? 0 : 1][t], acc[i][t]);
    }
  }

  // lds: two slots; x_bad: a word of LDS per row tile.  Called by all waves of the workgroup, those of both groups with the same n0 and j0.
  static __device__ __forceinline__ void run(const SplitArgs& p, int64_t n0, int j0, unsigned* lds, int* x_bad) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));              // what is derived from it here is not held in registers from pass to pass
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kLanes);
    const int q = tid / 16 % 4, i16 = tid % 16;
    const int chunks = p.k_red / kSplitChunk;
    const int jc = j0 + wave % 4 * 32 + 2 * i16;   // this lane's two columns: jc + t in column tile t
    acc_t acc[R][8][2];
#pragma unroll
    for (int t = 0; t < R; ++t)
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int u = 0; u < 2; ++u) acc[t][i][u] = acc_t{0, 0, 0, 0};
    if (tid < R) x_bad[tid] = 0;               // (read last before the barriers of the previous pass's stores)

    // rows of X.  This thread: quarter xp of the rows of reduction channels 2 xk, 2 xk + 1 of atoms wave and wave + 8 of
    // the tile: four lanes read a row, and an instruction whole lines between them.
    const int xk = tid % 64 / 4, xp = tid % 4;
    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(p.X + static_cast<size_t>(n0) * p.k_red * NC), 0, R * 16 * p.k_red * NC * 4, 0x00020000);
    const int left_rows = static_cast<int>(p.n_nodes - n0 < R * 16 ? p.n_nodes - n0 : R * 16);
    const int xlane = (2 * xk * NC + xp * 4) * 4;
    V4 xr[2][2];
    auto gload = [&](int step) {               // (past the end: the last step of that row tile again)
      const int t = step % R, ch = step / R < chunks ? step / R : chunks - 1;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        int row = t * 16 + wave + 8 * e;
        if (row >= left_rows) row = left_rows - 1;   // rows past the end split a valid atom and are not stored
        const int so = (row * p.k_red + ch * kSplitChunk) * NC * 4;
#pragma unroll
        for (int j = 0; j < 2; ++j)
          xr[e][j] = __builtin_bit_cast(V4, __builtin_amdgcn_raw_buffer_load_b128(xrs, xlane + j * NC * 4, so, 0));
      }
    };
    unsigned long long w_inexact = 0, x_inexact[R] = {};   // lanes that have split a value into parts of another sum
    auto split_x = [&](int slot, int i, unsigned& left) {   // the i-th of this thread's eight pairs of the step
      unsigned* const dst = lds + slot * kSplitSlot + (4 * xp + i % 4) * kSplitComp + xk / 4 * kSplitEight + (wave + i / 4 * 8) * 4 + xk % 4;
      const SplitPair s = split_pair(xr[i / 4][0][i % 4], xr[i / 4][1][i % 4], left);
      dst[0] = s.h;
      dst[kSplitPlane] = s.m;
      dst[2 * kSplitPlane] = s.l;
    };

    // this lane's columns of W: the eight channels 8 q .. 8 q + 7 of a chunk
    const int row_bytes = kTrans ? 4 : p.k_cols * 4;   // from a reduction channel to the next
    const int wlane = (kTrans ? jc * p.k_red + 8 * q : 8 * q * p.k_cols + jc) * 4;
    const int lstride = p.k_red * p.k_cols * 4;
    const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.W), 0, 4 * lstride, 0x00020000);
    float wr[2][8];
    U4 b[2][2][3];
    auto wload = [&](int o, int ch) {          // order o of the wave's two
      const int so = (o == 0 ? O::lo : O::hi) * lstride + (ch < chunks ? ch : chunks - 1) * kSplitChunk * row_bytes;
      if constexpr (kTrans) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int i = 0; i < 8; i += 4) {
            const V4 v = __builtin_bit_cast(V4, __builtin_amdgcn_raw_buffer_load_b128(wrs, wlane + u * p.k_red * 4, so + i * 4, 0));
#pragma unroll
            for (int k = 0; k < 4; ++k) wr[u][i + k] = v[k];
          }
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const V2 v = __builtin_bit_cast(V2, __builtin_amdgcn_raw_buffer_load_b64(wrs, wlane, so + i * row_bytes, 0));
          wr[0][i] = v[0];
          wr[1][i] = v[1];
        }
      }
    };
    auto split_w = [&](int o) {
      unsigned left = 0;
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const SplitPair s = split_pair(wr[u][2 * i], wr[u][2 * i + 1], left);
          b[o][u][0][i] = s.h;
          b[o][u][1][i] = s.m;
          b[o][u][2][i] = s.l;
        }
      w_inexact |= __builtin_amdgcn_ballot_w64((left & 0xffffu) != 0);
    };

    // The products of a step, and the split of the next one (inexact: of its tile).  The parts of X in turn, l
    // first; where one has been used for the last time, the next component's is requested.  last: the chunk's last step, after which the next chunk's W takes the registers.
    auto multiply = [&](int slot, acc_t (&sum)[8][2], unsigned long long& inexact, bool last, int ch, int ahead) {
      const unsigned* const src = lds + slot * kSplitSlot + q * kSplitEight + i16 * 4;
      unsigned left = 0;
      U4 a[3];
#pragma unroll
      for (int part = 0; part < 3; ++part) a[part] = *reinterpret_cast<const U4*>(src + part * kSplitPlane + O::component(0) * kSplitComp);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (i >= 4) {                          // (late: their requests have had half a step)
          split_x(slot ^ 1, 2 * i - 8, left);
          split_x(slot ^ 1, 2 * i - 7, left);
        }
        const int o = i < O::n_lo ? 0 : 1;
        acc_t small[2] = {acc_t{0, 0, 0, 0}, acc_t{0, 0, 0, 0}};
#pragma unroll
        for (int part = 2; part >= 0; --part) {
#pragma unroll
          for (int w = 2; w >= 0; --w) {
            if (part + w == 4) continue;       // l l
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              acc_t& to = part + w == 0 ? sum[i][u] : small[u];
              to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(Bf8, a[part]), __builtin_bit_cast(Bf8, b[o][u][w]), to, 0, 0, 0);
            }
          }
          if (i < 7) a[part] = *reinterpret_cast<const U4*>(src + part * kSplitPlane + O::component(i < 7 ? i + 1 : 7) * kSplitComp);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int r = 0; r < 4; ++r) sum[i][u][r] += small[u][r];
        __builtin_amdgcn_sched_barrier(0);
        if (last && i == O::n_lo - 1) {
          split_w(0);
          __builtin_amdgcn_sched_barrier(0);
          wload(1, ch + 1);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      inexact |= __builtin_amdgcn_ballot_w64((left & 0xffffu) != 0);
      __builtin_amdgcn_sched_barrier(0);       // (what is split is out of the registers before the next rows come in)
      gload(ahead);
      if (last) {
        split_w(1);
        __builtin_amdgcn_sched_barrier(0);
        wload(0, ch + 2);
        __builtin_amdgcn_sched_barrier(0);
      }
    };

    gload(0);
    wload(0, 0);
    split_w(0);
    wload(1, 0);
    __builtin_amdgcn_sched_barrier(0);
    unsigned first = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) split_x(0, i, first);
    x_inexact[0] = __builtin_amdgcn_ballot_w64((first & 0xffffu) != 0);
    gload(1);
    split_w(1);
    wload(0, 1);
    for (int ch = 0; ch < chunks; ++ch) {
#pragma unroll
      for (int t = 0; t < R; ++t) {
        const int slot = R == 2 ? t : ch & 1;
        __syncthreads();                       // this step's planes are written, those of the other slot have been read
        multiply(slot, acc[t], x_inexact[(t + 1) % R], t == R - 1, ch, ch * R + t + 2);
      }
    }
#pragma unroll
    for (int t = 0; t < R; ++t)
      if (x_inexact[t] != 0) x_bad[t] = 1;
    __syncthreads();                           // also: the planes have been read, the stages may take their place
    float* const stages = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int t = 0; t < R; ++t) {
      // An infinity, or a value that h rounds to one (from 0x7f7f8000 on), leaves an infinity or a NaN in every result it
      // enters, where the product in fp32 may have another value.
      float bad = 0;
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int r = 0; r < 4; ++r) bad = __builtin_fmaf(acc[t][i][u][r], 0.0f, bad);
      if (x_bad[t] != 0 || w_inexact != 0 || __builtin_amdgcn_ballot_w64(bad != 0.0f) != 0) plain(p, n0 + t * 16, jc, q, i16, acc[t]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float* const stage = stages + (r & 1) * kSplitStage;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          float* const d = stage + (q * 128 + jc - j0 + u) * 20;
          const acc_t(&s)[8][2] = acc[t];
          if constexpr (G == 0) {
            d[0] = s[0][u][r];
            d[9] = s[1][u][r];
            *reinterpret_cast<V2*>(d + 10) = V2{s[2][u][r], s[3][u][r]};
            *reinterpret_cast<V4*>(d + 12) = V4{s[4][u][r], s[5][u][r], s[6][u][r], s[7][u][r]};
          } else {
            d[1] = s[0][u][r];
            *reinterpret_cast<V2*>(d + 2) = V2{s[1][u][r], s[2][u][r]};
            *reinterpret_cast<V4*>(d + 4) = V4{s[3][u][r], s[4][u][r], s[5][u][r], s[6][u][r]};
            d[8] = s[7][u][r];
          }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {          // atom 4 i + r of the tile: 8 KB, a 16-byte piece per thread
          const V4 x = *reinterpret_cast<const V4*>(stage + (i * 128 + tid / 4) * 20 + tid % 4 * 4);
          const int64_t n = n0 + t * 16 + 4 * i + r;
          if (n < p.n_nodes)
            __builtin_nontemporal_store(x, reinterpret_cast<V4*>(p.Y + (static_cast<size_t>(n) * p.k_cols + j0) * NC + tid * 4));
        }
      }
    }
    __syncthreads();                           // the stages have been read, the next pass's planes may take their place
  }
};

// The accumulators of rows n0..n0+15 and of the wave's 16 of the 128 columns from j0 on, in half the registers of a pass: a workgroup with
// one tile each for two workgroups on a CU (mfma_forward_bf16_pair_kernel).  The workgroup (eight waves) splits X in chunks of 32 reduction
// channels into LDS (three planes of [component][atom][32]; the next chunk's rows are requested a chunk ahead); a wave splits its own
// columns of W order by order, requested an order ahead.  x_served: the values of X that the wave has split are the sums of their parts (for other
// waves' columns as well).  redo[G]: not so for the wave's values of W, or results that are not finite, in the orders of wave group G of a pass.
constexpr int kPairPlane = 16 * 16 * kSplitChunk / 2;     // 32-bit words of a plane: two channels each

__device__ __forceinline__ void split_tile_product(int64_t n_nodes, int64_t n0, int j0, int k_red, int k_cols,
                                                   const float* __restrict__ X, const float* __restrict__ W,
                                                   unsigned* planes /* 3 * kPairPlane words */,
                                                   typename Mma<float>::acc_t (&acc)[16][1], bool& x_served, bool (&redo)[2]) {
  constexpr int NC = 16, L = 4;
  typedef Mma<float>::acc_t acc_t;
  typedef float V4 __attribute__((ext_vector_type(4)));
  // The thread's number as a value of its own: what is derived from it here ends with the loop, and what the
  // caller derives from it is not held in registers through the loop.
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int q = tid / 16 % 4, i16 = tid % 16, jc = j0 + tid / kLanes * 16 + i16;
  const int chunks = k_red / kSplitChunk;
  // splitting role of this thread: half of the components of one atom of the tile and two reduction channels
  const int half = tid / 256, sa = tid / 16 % 16, sk = tid % 16;
  int64_t ns = n0 + sa;
  if (ns >= n_nodes) ns = n_nodes - 1;       // rows past the end split a valid atom and are not stored
  // (through a descriptor of the tile's rows, like W: the lane's part is one 32-bit offset)
  const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(X + static_cast<size_t>(n0) * k_red * NC), 0, 16 * k_red * NC * 4, 0x00020000);
  const unsigned xoff = ((static_cast<unsigned>(ns - n0) * k_red + 2 * sk) * NC + half * 8) * 4u;
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c][0] = acc_t{0, 0, 0, 0};

  unsigned long long x_inexact = 0, w_inexact[2] = {};   // lanes that have split a value into parts of another sum
  V4 xr[2][2];
  auto gload = [&](int chunk) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      xr[i / 2][i % 2] = __builtin_bit_cast(V4, __builtin_amdgcn_raw_buffer_load_b128(
          xrs, static_cast<int>(xoff), (chunk * kSplitChunk * NC + i / 2 * NC + i % 2 * 4) * 4, 0));
  };
  auto split_x = [&]() {
    unsigned left = 0;
    unsigned* dst = planes + half * 8 * 256 + sa * 16 + sk;
#pragma unroll
    for (int c = 0; c < NC / 2; ++c) {
      const float x = xr[0][c / 4][c % 4], y = xr[1][c / 4][c % 4];
      const SplitPair s = split_pair(x, y, left);
      dst[c * 256] = s.h;
      dst[c * 256 + kPairPlane] = s.m;
      dst[c * 256 + 2 * kPairPlane] = s.l;
    }
    x_inexact |= __builtin_amdgcn_ballot_w64((left & 0xffffu) != 0);
  };
  // this lane's column of W: eight channels 8 q .. 8 q + 7 of a chunk, as in lds_tile_product through a descriptor
  const unsigned boff = static_cast<unsigned>(8 * q * k_cols + jc) * 4u;
  const unsigned row_bytes = static_cast<unsigned>(k_cols) * 4u;   // from a reduction channel to the next
  const unsigned lstride = static_cast<unsigned>(k_red) * static_cast<unsigned>(k_cols) * 4u;
  const __amdgpu_buffer_rsrc_t wrs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(W), 0, static_cast<int>(L * lstride), 0x00020000);
  float wr[8];
  auto bload = [&](int chunk, int l) {
    const unsigned so = static_cast<unsigned>(l) * lstride + static_cast<unsigned>(chunk * kSplitChunk) * row_bytes;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      wr[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wrs, static_cast<int>(boff),
                                                                             static_cast<int>(so + i * row_bytes), 0));
  };
  auto read_a = [&](int part, int c) {
    return *reinterpret_cast<const U4*>(planes + part * kPairPlane + c * 256 + i16 * 16 + q * 4);
  };
  gload(0);
  bload(0, L - 1);
  // The waves that multiply go first: the two workgroups of a CU drift apart, and one's products cover the other's
  // requests and splitting (20 000 atoms: 112 -> 102 us, with six products).
  for (int ch = 0; ch < chunks; ++ch) {
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();                         // the reads of the previous chunk are done
    split_x();
    __builtin_amdgcn_sched_barrier(0);       // (what is split is out of the registers before the next rows come in)
    // (no condition on the request: at its join the compiler would wait for every outstanding load)
    gload(ch + 1 < chunks ? ch + 1 : ch);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    U4 a[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) a[p] = read_a(p, (L - 1) * (L - 1));
#pragma unroll
    for (int l = L - 1; l >= 0; --l) {
      U4 b[3];
      unsigned left = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const SplitPair s = split_pair(wr[2 * i], wr[2 * i + 1], left);
        b[0][i] = s.h;
        b[1][i] = s.m;
        b[2][i] = s.l;
      }
      w_inexact[l % 3 == 0 ? 0 : 1] |= __builtin_amdgcn_ballot_w64((left & 0xffffu) != 0);
      __builtin_amdgcn_sched_barrier(0);
      const int next = l > 0 ? ch : (ch + 1 < chunks ? ch + 1 : ch);   // past the end: a valid chunk again
      bload(next, l > 0 ? l - 1 : L - 1);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int c = l * l; c < (l + 1) * (l + 1); ++c) {
        // The parts of X in turn, l first; where one has been used for the last time, the next component's is requested
        // (4000 atoms, 256 -> 256 channels: 76 -> 71 us).
        const int next_c = c + 1 < (l + 1) * (l + 1) ? c + 1 : (l > 0 ? (l - 1) * (l - 1) : -1);
        acc_t small{0, 0, 0, 0};
#pragma unroll
        for (int p = 2; p >= 0; --p) {
#pragma unroll
          for (int w = 2; w >= 0; --w) {
            if (p + w == 4) continue;        // l l
            acc_t& sum = p + w == 0 ? acc[c][0] : small;
            sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(Bf8, a[p]), __builtin_bit_cast(Bf8, b[w]), sum, 0, 0, 0);
          }
          if (next_c >= 0) a[p] = read_a(p, next_c);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[c][0][r] += small[r];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  __builtin_amdgcn_s_setprio(0);
  bool finite[2] = {true, true};
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) finite[order_of(c) % 3 == 0 ? 0 : 1] &= __builtin_isfinite(acc[c][0][r]);
  x_served = x_inexact == 0;
#pragma unroll
  for (int g = 0; g < 2; ++g) redo[g] = w_inexact[g] != 0 || __builtin_amdgcn_ballot_w64(!finite[g]) != 0;
}

// The accumulators of wave group G's orders on the fp32 matrix cores, operands straight from memory: what the parts do not serve.
template <int G>
__device__ __forceinline__ void plain_tile_product(int64_t n_nodes, int64_t n0, int jc, int k_red, int k_cols,
                                                   const float* __restrict__ X, const float* __restrict__ W,
                                                   typename Mma<float>::acc_t (&acc)[16][1]) {
  typedef SplitOrders<G> O;
  constexpr int NC = 16;
  const int lane = threadIdx.x & (kLanes - 1), q = lane / 16, i16 = lane & 15;
  const int64_t na = n0 + i16 < n_nodes ? n0 + i16 : n_nodes - 1;
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[O::component(i)][0] = Mma<float>::acc_t{0, 0, 0, 0};
  for (int k = q; k < k_red; k += 4) {
    float a[NC], b[2];
    load_row<float, NC>(X + (static_cast<size_t>(na) * k_red + k) * NC, a);
#pragma unroll
    for (int o = 0; o < 2; ++o) b[o] = W[(static_cast<size_t>(o == 0 ? O::lo : O::hi) * k_red + k) * k_cols + jc];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      acc[O::component(i)][0] = Mma<float>::mma(a[O::component(i)], b[i < O::n_lo ? 0 : 1], acc[O::component(i)][0]);
  }
}

// Store of a wave's result tile Y[n0 + 4*(lane/16) + r][jc[t]][0..15].  A lane holds whole 64-byte
// rows; stored directly, every instruction would write a quarter of each row (16-byte pieces 64
// bytes apart: partial lines, four times the write requests).  Per (t, r) the 16 rows of a
// 16-lane group are one contiguous KB of Y: they go through LDS (rows padded to 80 bytes) and
// come back so that instruction i writes the i-th contiguous 256 bytes of each KB, streamed past
// the cache.  stage: kStoreStageFloats floats of LDS owned by this wave; the caller puts a
// workgroup barrier between the last LDS read of the product and this call when the stage
// overlaps the product's buffers.  Measured on the forward kernel (10k atoms): 87 -> 73.5 us.
constexpr int kStoreRow = 20;                          // floats per staged row
constexpr int kStoreStageFloats = 4 * 16 * kStoreRow;  // per wave

template <int CT>
__device__ __forceinline__ void store_tile_coalesced(float* __restrict__ Y, int64_t n_nodes, int64_t n0, int k_cols,
                                                     const int (&jc)[CT],
                                                     const typename Mma<float>::acc_t (&acc)[16][CT], float* stage) {
  typedef float V4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x & (kLanes - 1);
  const int q = lane / 16, j16 = lane & 15;
  float* const mine = stage + (q * 16 + j16) * kStoreRow;
#pragma unroll
  for (int t = 0; t < CT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the previous round's reads of the stage are done
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<V4*>(mine + 4 * i) = V4{acc[4 * i][t][r], acc[4 * i + 1][t][r], acc[4 * i + 2][t][r], acc[4 * i + 3][t][r]};
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the other lanes' rows are visible
      __builtin_amdgcn_wave_barrier();
      const int64_t n = n0 + Mma<float>::row(lane, r);
      if (n < n_nodes) {
        float* yblock = Y + (static_cast<size_t>(n) * k_cols + (jc[t] - j16)) * 16;   // the group's KB
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int p = i * 16 + j16;                  // 16-byte piece of the KB: row p / 4, quarter p % 4
          const V4 x = *reinterpret_cast<const V4*>(stage + (q * 16 + p / 4) * kStoreRow + (p % 4) * 4);
          __builtin_nontemporal_store(x, reinterpret_cast<V4*>(yblock + p * 4));
        }
      }
    }
}

// Work of a persistent grid of S workgroups over U full units (row tile x 128 columns), two
// workgroups per CU (workgroups b and b + S/2 share a CU: read from the hardware id registers).
// Two workgroups that start together tend to stay in step: both run their matrix phase, then
// both their epilogue (stores, or the contraction).  So the second half of the grid starts with
// HALF a unit (64 columns) and is from then on half a phase away from its neighbour, whose matrix
// work then covers its epilogue and vice versa (measured: -4% on the fused kernel, about neutral
// on the plain linear).  The last n_split = min(U, S/4) full units are cut into the 2 n_split
// halves; the other units go round the workgroups as usual.  stagger = false: no halves.
struct UnitSchedule {
  bool has_half;
  int64_t half_unit;   // full unit that the half belongs to
  int half;            // which half of it (0 or 1)
  int64_t n_full;      // full units 0 .. n_full-1 are dealt blockIdx.x, blockIdx.x + gridDim.x, ...
};

__device__ __forceinline__ UnitSchedule unit_schedule(int64_t full_units, bool stagger) {
  const int S = gridDim.x, b = blockIdx.x;
  UnitSchedule u{false, 0, 0, full_units};
  if (!stagger || S % 4 != 0) return u;
  const int64_t n_split = full_units < S / 4 ? full_units : S / 4;
  u.n_full = full_units - n_split;
  const int rank = b - S / 2;
  if (rank >= 0 && rank < 2 * n_split) {
    u.has_half = true;
    u.half_unit = full_units - 1 - rank / 2;
    u.half = rank & 1;
  }
  return u;
}

}  // namespace el
