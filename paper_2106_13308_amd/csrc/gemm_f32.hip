// FP32 products of the masked MADE on operands read straight into registers (gfx950).
//
// The four products (Sec. 5.1 layers; Sec. 2.1 score gradient) as in the other engines:
//   A[b][k] = b1[k] + sum_{d : c[d] <= k} S[b][d] P[d][k],  R = relu(A)      (first layer)
//   Z[b][d] = b2[d] + sum_{k < c[d]} R[b][k] P[d][k]                         (second layer)
//   D[b][k] = [A[b][k] > 0] sum_{d : c[d] > k} G[b][d] P[d][k]                (dF/dA)
//   dP[d][k] = sum_b G[b][d] R[b][k] (k < c[d]),  sum_b S[b][d] D[b][k] (else)
//
// Engine: v_mfma_f32_32x32x2_f32 (64 cycles) takes one float per lane and operand, lane l the value of
// row l % 32 at one of two ks.  Every operand is read from the one of its two layouts in which the rows
// are adjacent in memory (X[k][row]): a load instruction is then two full 128-byte lines, and the
// caches deliver the 256 bytes per operand and 64 matrix cycles without LDS staging and without a
// barrier in the loop.  (So the gradient's batch products read G, relu(A) and D by sample and the
// spins as they are, and no transposed copies of the spins and of D are written.)  The first layer's
// spins have the sites adjacent: two lanes read 32 bytes of a row and hand them out by ds_bpermute,
// a byte per k.  The waves of a workgroup share a tile of 32 WM x 32 WN and split its K range WK ways;
// their partial tiles are added in a fixed order through LDS once, at the end.  Short K ranges with few
// tiles (the small models, where the products are latency chains) thus spread over eight waves per
// tile, large ones over 64 x 64 tiles that halve the cache traffic.
//
// What bounds it: at small sizes the launch, the fetch of the kernel's code and two or three dependent loads
// (hence 4 - 6 KB of code, buffer descriptors that end with the matrix instead of clamped addresses,
// 64-way searches of c, and the epilogue's inputs loaded before the products); at the larger ones
// the matrix cores, at about half their rate: a run's conversions and masks wait for its loads.
// Measured (us; before: 64 x 64 tiles staged through LDS, one wave set per tile, both weight halves
// and both bias sums in launches of their own):
//                                 n = 20, h = 45,   n = 500, h = 193,   n = h = 500,
//                                 B = 1024          B = 1024            B = 4096
//   first layer                                                         22 (41)
//   second layer, log p / adjoint                                       20 / 25 (36 / 40)
//   hidden adjoint                5.4 (6.2)         9.0 (25)            23 (36)
//   weight and bias gradients     8.6 (84)          9.4 (90)            42 (307)
#include "common.hpp"
#include "kernels.hpp"

namespace vqmc {

typedef __attribute__((ext_vector_type(16))) float floatx16_t;

template <int WM_, int WN_, int WK_>
struct F32 {
  static constexpr int WM = WM_, WN = WN_, WK = WK_;
  static constexpr int NT = 64 * WM * WN * WK, BM = 32 * WM, BN = 32 * WN;
  static constexpr int NI = BM * BN / NT;  // tile elements per thread
  float red[WK][BM][BN + 1];
  int bound[BN];  // limits of the tile's columns (unit_limits)

  __device__ static int wave() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
  // first row and column of this wave's part of the tile
  __device__ static int row0() { return 32 * (wave() / (WK * WN)); }
  __device__ static int col0() { return 32 * ((wave() / WK) % WN); }

  // acc = A x B^T over ks [kbeg, kend), then the sum over the WK waves of a tile: on return red[0] holds
  // the BM x BN tile.  A run is LA::KC ks (run q of the range to wave q mod WK); both operands take its
  // ks in the order LA::k gives: step s, lane half g.  The code is kept short because every launch
  // fetches it anew.
  template <class LA, class LB>
  __device__ void run(const LA& la, const LB& lb, int kbeg, int kend) {
    constexpr int KC = LA::KC, NS = KC / 2, PD = 2;  // PD runs in flight per wave
    const int t = threadIdx.x, lane = t & 63;
    const int wk = wave() % WK;
    const int nrun = kend > kbeg ? (kend - kbeg + KC - 1) / KC : 0;
    floatx16_t acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    if (wk < nrun) {
      typename LA::Raw ra[PD];
      float rb[PD][NS];
      auto load = [&](int p, int q) {  // past the end: the last run's loads again, never used
        const int k = kbeg + KC * min(q, nrun - 1);
        la.load(ra[p], k);
        lb.load(rb[p], k);
      };
#pragma unroll
      for (int p = 0; p < PD; ++p) load(p, wk + WK * p);
#pragma unroll 1
      for (int q0 = wk; q0 < nrun; q0 += PD * WK) {
#pragma unroll
        for (int p = 0; p < PD; ++p) {
          const int q = q0 + WK * p;
          if (q < nrun) {
            float a[NS], b[NS];
            la.values(ra[p], a);
            if (lb.inside(kbeg + KC * q)) lb.values(rb[p], b);
            else lb.masked(rb[p], kbeg + KC * q, b);
            load(p, q + PD * WK);
#pragma unroll
            for (int s = 0; s < NS; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], b[s], acc, 0, 0, 0);
          }
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) red[wk][row0() + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)][col0() + (lane & 31)] = acc[e];
    __syncthreads();
    if constexpr (WK > 1) {
      for (int x = t; x < BM * BN; x += NT) {
        const int m = x / BN, n = x % BN;
        float v = red[0][m][n];
#pragma unroll
        for (int q = 1; q < WK; ++q) v += red[q][m][n];
        red[0][m][n] = v;
      }
      __syncthreads();
    }
  }
};

// The step order of a run whose operands both have their rows adjacent.  A lane's offsets within a run have 32 bits: from
// 2^31 / (4 * 15) columns of a matrix on (35.8 million samples), runs of two ks.
template <int KC_>
struct FPairsOf {
  static constexpr int KC = KC_;
  __device__ static int k(int s, int g) { return 2 * s + g; }
};
using FPairs = FPairsOf<16>;
using FFar = FPairsOf<2>;
static bool f32_far(int64_t ld) { return (FPairs::KC - 1) * ld * (int64_t)sizeof(float) > 0x7FFFFFFF; }

enum FMask { F_ALL, F_BELOW, F_FROM };  // ks of a row that count: all, those below its limit, those from it on

// Operand X[k][row] (T = float, or int8_t spins), rows adjacent, row0 < ld, kmax ks (those past the end read as zero: the
// buffer descriptor of a run ends with the matrix), the ks of a run in the order of ORDER
template <typename T, class ORDER, FMask MASK = F_ALL>
struct FCols {
  static constexpr int KC = ORDER::KC, NS = KC / 2;
  __device__ static int k(int s, int g) { return ORDER::k(s, g); }
  const T* X;
  int64_t ld, row0;
  int kmax, limit, full;  // full: a bound of the limits of all lanes
  uint32_t off[NS];  // this lane's byte of step s, from the run's first k
  __device__ FCols(const T* x, int64_t ld_, int64_t row0_, int kmax_, int limit_ = 0, int full_ = 0)
      : X(x), ld(ld_), row0(row0_), kmax(kmax_), limit(limit_), full(full_) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int s = 0; s < NS; ++s) off[s] = (uint32_t)((k(s, lane >> 5) * (int)ld + (lane & 31)) * (int)sizeof(T));
  }
  using Raw = T[NS];
  __device__ void load(T (&v)[NS], int k0) const {
    const int64_t left = ((int64_t)(kmax - k0) * ld - row0) * (int64_t)sizeof(T);
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc((void*)(X + (int64_t)k0 * ld + row0), 0, (int)min(left, (int64_t)0x7FFFFFFF), 0x00020000);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if constexpr (sizeof(T) == 4) v[s] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off[s], 0, 0));
      else v[s] = (T)__builtin_amdgcn_raw_buffer_load_b8(r, (int)off[s], 0, 0);
    }
  }
  __device__ void values(const T (&x)[NS], float (&v)[NS]) const {
#pragma unroll
    for (int s = 0; s < NS; ++s) v[s] = (float)x[s];
  }
  // whether every k of the run at k0 counts for every lane
  __device__ bool inside(int k0) const { return MASK == F_ALL || (MASK == F_BELOW ? k0 + KC <= full : k0 >= full); }
  __device__ void masked(const T (&x)[NS], int k0, float (&v)[NS]) const {
    const int l = limit - k0 - k(0, (threadIdx.x >> 5) & 1);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int ks = k(s, 0);
      v[s] = (MASK == F_ALL || (MASK == F_BELOW ? ks < l : ks >= l)) ? (float)x[s] : 0.f;
    }
  }
};

// Spins by sample as the first operand with the sites as ks: S[row][k], columns past n meet masked
// weights.  Lanes 2 r and 2 r + 1 read 32 bytes of row r; lane (r, g) takes the even (g = 0) or odd ones.
struct FSpinRows {
  static constexpr int KC = 32;
  __device__ static int k(int s, int g) { return 2 * s + g; }
  using Raw = uint4;
  const int8_t* p;
  __device__ FSpinRows(const int8_t* S, int64_t lds, int64_t row0, int64_t rows) {
    const int lane = threadIdx.x & 63;
    p = S + min(row0 + (lane >> 1), rows - 1) * lds + 16 * (lane & 1);
  }
  struct __attribute__((aligned(8))) Bytes16 {  // spin rows may start on any 8-byte boundary
    uint32_t x[4];
  };
  __device__ void load(Raw& v, int k0) const {
    const Bytes16 b = *(const Bytes16*)(p + k0);
    v = make_uint4(b.x[0], b.x[1], b.x[2], b.x[3]);
  }
  __device__ void values(const Raw& x, float (&v)[KC / 2]) const {
    const int lane = threadIdx.x & 63, g = lane >> 5;
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint32_t u = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (2 * (lane & 31) + (q >> 2)), (int)w[q & 3]) >> (8 * g);
      v[2 * q] = (float)(int8_t)u;
      v[2 * q + 1] = (float)(int8_t)(u >> 16);
    }
  }
};

// Column tile of a workgroup.  The K ranges grow or shrink along the columns; workgroups are dealt
// round-robin to the 8 XCDs and, in grids of one or two workgroups per CU, the second half lands on the
// CUs of the first.  So each row of tiles starts one column further on, and the second half of the rows
// runs through the columns backwards: every XCD and every CU gets long and short ranges.
__device__ inline int f_column() {
  const int x = (int)((blockIdx.x + blockIdx.y) % gridDim.x);
  return 2 * blockIdx.y < gridDim.y ? x : (int)gridDim.x - 1 - x;
}

// ---------------------------------------------------------------- first layer
// relu(S P_upper + b1) by unit (Rt: h x ldB, zero past B) and, if R, by sample (B x ldh)
template <class E>
__global__ __launch_bounds__(E::NT) void f32_hidden_kernel(const int8_t* __restrict__ S, int64_t lds,
                                                           const float* __restrict__ P, int64_t ldh,
                                                           const float* __restrict__ b1, const int32_t* __restrict__ c,
                                                           int n, int h, int64_t B, float* __restrict__ R,
                                                           float* __restrict__ Rt, int64_t ldB) {
  __shared__ E e;
  const int64_t m0 = (int64_t)blockIdx.y * E::BM;  // samples
  const int n0 = f_column() * E::BN;               // units
  int first, last;
  unit_limits<E::BN, E::NT>(e.bound, c, n, h, n0, first, last);
  const int kb = n0 + threadIdx.x % E::BN;  // the thread's unit in the epilogue
  const float bias = kb < h ? b1[kb] : 0.f;
  e.run(FSpinRows(S, lds, m0 + E::row0(), B),
        FCols<float, FSpinRows, F_BELOW>(P, ldh, n0 + E::col0(), n,
                                           e.bound[E::col0() + (threadIdx.x & 31)], first),
        0, last);
  for (int x = threadIdx.x; x < E::BM * E::BN; x += E::NT) {
    const int m = x / E::BN, nn = x % E::BN, k = n0 + nn;
    const float v = (k < h && m0 + m < B) ? fmaxf(e.red[0][m][nn] + bias, 0.f) : 0.f;
    if (R && m0 + m < B && k < ldh) R[(m0 + m) * ldh + k] = v;
    e.red[0][m][nn] = v;
  }
  __syncthreads();
  for (int x = threadIdx.x; x < E::BM * E::BN; x += E::NT) {
    const int nn = x / E::BM, m = x % E::BM, k = n0 + nn;
    if (k < h && m0 + m < ldB) Rt[(int64_t)k * ldB + m0 + m] = e.red[0][m][nn];
  }
}

// ---------------------------------------------------------------- second layer
// GRAD = false: log sigma partials (one row of B per site tile) and optionally Z (B x ldn).
// GRAD = true: G = coef s sigma(-s z) by sample (B x ldn) and by site (Gt, n x ldB, zero past B), the
// spins by site (St, the same, nullable), and db2 partials (one row of ldn per sample tile).
template <class E, bool GRAD, class ORDER = FPairs>
__global__ __launch_bounds__(E::NT) void f32_out_kernel(const float* __restrict__ Rt, int64_t ldB,
                                                        const float* __restrict__ Pt, int64_t ldn,
                                                        const float* __restrict__ b2, const int32_t* __restrict__ c,
                                                        int n, int h, int64_t B, const int8_t* __restrict__ S,
                                                        float* __restrict__ lp_part, float* __restrict__ Z,
                                                        const float* __restrict__ coef, float* __restrict__ G,
                                                        float* __restrict__ Gt, float* __restrict__ St,
                                                        float* __restrict__ db2_part) {
  static_assert(E::WK > 1, "the spins use the second partial tile");
  __shared__ E e;
  const int64_t m0 = (int64_t)blockIdx.y * E::BM;  // samples
  const int tile = f_column();                     // sites
  const int d0 = tile * E::BN;
  // what the epilogue needs, loaded before the products: the thread's site and its elements' samples
  const int t = threadIdx.x, nn = t % E::BN, d = d0 + nn;
  const float bias = d < n ? b2[d] : 0.f;
  float cb[E::NI];
  int8_t sb[E::NI];
#pragma unroll
  for (int i = 0; i < E::NI; ++i) {
    const int64_t b = m0 + t / E::BN + i * (E::NT / E::BN);
    const bool ok = d < n && b < B;
    sb[i] = ok ? S[b * ldn + d] : (int8_t)0;
    cb[i] = (GRAD && ok) ? coef[b] : 0.f;
  }
  const int dl = d0 + E::col0() + (t & 31);
  // (the tile's second rows may start past an unpadded batch: their results are not stored, but the rows must lie in the
  // matrix for its descriptor to end with it)
  e.run(FCols<float, ORDER>(Rt, ldB, min(m0 + E::row0(), ldB - 1), h),
        FCols<float, ORDER, F_BELOW>(Pt, ldn, d0 + E::col0(), h, dl < n ? c[dl] : 0, c[d0]),  // unit k feeds site d iff k < c[d]
        0, c[min(d0 + E::BN, n) - 1]);
#pragma unroll
  for (int i = 0; i < E::NI; ++i) {
    const int m = t / E::BN + i * (E::NT / E::BN);
    const int64_t b = m0 + m;
    const bool ok = d < n && b < B;
    const float z = e.red[0][m][nn] + bias, s = (float)sb[i];
    if constexpr (GRAD) {
      const float g = ok ? cb[i] * s * sigmoid(-s * z) : 0.f;
      if (b < B && d < ldn) G[b * ldn + d] = g;
      e.red[0][m][nn] = g;
      e.red[1][m][nn] = s;
    } else {
      if (Z && ok) Z[b * ldn + d] = z;
      float v = ok ? log_sigmoid(s * z) : 0.f;  // summed over the tile's sites, which are BN adjacent lanes
#pragma unroll
      for (int o = 1; o < E::BN; o <<= 1) v += __shfl_xor(v, o);
      if (nn == 0 && b < B) lp_part[(int64_t)tile * B + b] = v;
    }
  }
  if constexpr (GRAD) {
    __syncthreads();
    for (int x = threadIdx.x; x < E::BM * E::BN; x += E::NT) {
      const int nn = x / E::BM, m = x % E::BM, d = d0 + nn;
      const float g = e.red[0][m][nn];
      if (d < n && m0 + m < ldB) {
        Gt[(int64_t)d * ldB + m0 + m] = g;
        if (St) St[(int64_t)d * ldB + m0 + m] = e.red[1][m][nn];
      }
      float v = g;  // over the tile's samples, BM adjacent lanes
#pragma unroll
      for (int o = 1; o < E::BM; o <<= 1) v += __shfl_xor(v, o);
      if (m == 0 && d < ldn) db2_part[(int64_t)blockIdx.y * ldn + d] = v;
    }
  }
}

// ---------------------------------------------------------------- hidden adjoint
// [Rt > 0] (G P_lower) by sample (D, B x ldh) or by unit (Dt, h x ldB, zero past B), whichever is given, db1
// partials (one row of ldh per sample tile) and, if R, relu(A) by sample from Rt.
template <class E, class ORDER = FPairs>
__global__ __launch_bounds__(E::NT) void f32_adjoint_kernel(const float* __restrict__ Gt, int64_t ldB,
                                                            const float* __restrict__ P, int64_t ldh,
                                                            const int32_t* __restrict__ c, int n, int h, int64_t B,
                                                            const float* __restrict__ Rt, float* __restrict__ D,
                                                            float* __restrict__ Dt, float* __restrict__ R,
                                                            float* __restrict__ db1_part) {
  static_assert(E::WK > 1, "relu(A) uses the second partial tile");
  __shared__ E e;
  const int64_t m0 = (int64_t)blockIdx.y * E::BM;  // samples
  const int n0 = f_column() * E::BN;               // units
  int first, last;
  unit_limits<E::BN, E::NT>(e.bound, c, n, h, n0, first, last);
  // relu(A) of the thread's elements, loaded before the products
  const int t = threadIdx.x, m = t % E::BM;
  float rv[E::NI];
#pragma unroll
  for (int i = 0; i < E::NI; ++i) {
    const int k = n0 + t / E::BM + i * (E::NT / E::BM);
    rv[i] = (k < h && m0 + m < ldB) ? Rt[(int64_t)k * ldB + m0 + m] : 0.f;
  }
  e.run(FCols<float, ORDER>(Gt, ldB, m0 + E::row0(), n),
        FCols<float, ORDER, F_FROM>(P, ldh, n0 + E::col0(), n, e.bound[E::col0() + (t & 31)], last), first, n);
#pragma unroll
  for (int i = 0; i < E::NI; ++i) {
    const int nn = t / E::BM + i * (E::NT / E::BM), k = n0 + nn;
    float v = (m0 + m < B && rv[i] > 0.f) ? e.red[0][m][nn] : 0.f;
    if (Dt && k < h && m0 + m < ldB) Dt[(int64_t)k * ldB + m0 + m] = v;
    e.red[0][m][nn] = v;
    e.red[1][m][nn] = rv[i];
#pragma unroll
    for (int o = 1; o < E::BM; o <<= 1) v += __shfl_xor(v, o);
    if (m == 0 && k < ldh) db1_part[(int64_t)blockIdx.y * ldh + k] = v;
  }
  if (!D) return;
  __syncthreads();
  for (int x = t; x < E::BM * E::BN; x += E::NT) {
    const int mm = x / E::BN, nn = x % E::BN, k = n0 + nn;
    if (m0 + mm < B && k < ldh) {
      D[(m0 + mm) * ldh + k] = e.red[0][mm][nn];
      if (R) R[(m0 + mm) * ldh + k] = e.red[1][mm][nn];
    }
  }
}

// ---------------------------------------------------------------- weight gradient
// Tiles of dP (sites x units): the lower product (G x R) where k < c[d], the upper one (S x D) elsewhere.  A
// tile across the staircase needs both: in one workgroup, or (SPLIT, for grids that leave CUs idle)
// in two, the second ntile workgroups taking the upper products.  The workgroups past the tiles sum the
// partials of the bias gradients, 64 entries each: db2 (np2 rows of ldn), then db1 (np1 rows of ldh).
template <class E, bool SPLIT>
__global__ __launch_bounds__(E::NT) void f32_weight_kernel(const float* __restrict__ G, int64_t ldn,
                                                           const float* __restrict__ R, int64_t ldh,
                                                           const int8_t* __restrict__ S, const float* __restrict__ D,
                                                           int64_t B, const int32_t* __restrict__ c, int n, int h,
                                                           float* __restrict__ dP, int ntile,
                                                           const float* __restrict__ db2_part, int np2,
                                                           const float* __restrict__ db1_part, int np1,
                                                           float* __restrict__ db2, float* __restrict__ db1) {
  __shared__ E e;
  constexpr int NH = SPLIT ? 2 : 1;
  if ((int)blockIdx.x >= NH * ntile) {
    constexpr int NQ = E::NT / 64;
    const int t = threadIdx.x, q = t >> 6, nb2 = (n + 63) / 64;
    const int x = (int)blockIdx.x - NH * ntile;
    const bool two = x < nb2;
    const int i = 64 * (two ? x : x - nb2) + (t & 63), len = two ? n : h, np = two ? np2 : np1;
    const int64_t stride = two ? ldn : ldh;
    const float* part = two ? db2_part : db1_part;
    float s = 0.f;
    if (i < len)
      for (int p = q; p < np; p += NQ) s += part[(int64_t)p * stride + i];
    float* sum = &e.red[0][0][0];
    sum[q * 64 + (t & 63)] = s;
    __syncthreads();
    if (q == 0 && i < len) {
      for (int p = 1; p < NQ; ++p) s += sum[p * 64 + t];
      (two ? db2 : db1)[i] = s;
    }
    return;
  }
  const int nkt = (h + E::BN - 1) / E::BN;
  const int half = SPLIT && (int)blockIdx.x >= ntile, tile = (int)blockIdx.x - half * ntile;
  const int d0 = tile / nkt * E::BM, k0 = tile % nkt * E::BN;
  const bool lower = half == 0 && k0 < c[min(d0 + E::BM, n) - 1];
  const bool upper = (!SPLIT || half == 1) && min(k0 + E::BN, h) - 1 >= c[d0];
  auto store = [&](bool low) {
    for (int x = threadIdx.x; x < E::BM * E::BN; x += E::NT) {
      const int m = x / E::BN, nn = x % E::BN, d = d0 + m, k = k0 + nn;
      if (d < n && k < h && (k < c[d]) == low) dP[(int64_t)d * h + k] = e.red[0][m][nn];
    }
  };
  if (lower) {
    e.run(FCols<float, FPairs>(G, ldn, d0 + E::row0(), (int)B), FCols<float, FPairs>(R, ldh, k0 + E::col0(), (int)B), 0, (int)B);
    store(true);
  }
  if (upper) {
    if (lower) __syncthreads();  // red is written again
    e.run(FCols<int8_t, FPairs>(S, ldn, d0 + E::row0(), (int)B), FCols<float, FPairs>(D, ldh, k0 + E::col0(), (int)B), 0, (int)B);
    store(false);
  }
}

// ---------------------------------------------------------------- launches
using FSmall = F32<1, 1, 8>;
using FLarge = F32<2, 2, 2>;

static inline unsigned tiles(int64_t x, int t) { return (unsigned)((x + t - 1) / t); }

// The rule between the two shapes, for an M x N output.
static bool f32_large(int64_t M, int64_t N) { return (int64_t)tiles(M, 64) * tiles(N, 64) >= 512; }

// ordered: no split of K.  A product is then a chain of multiply-adds in the order of the sites, whatever the tile,
// and the pre-activations are those of the staged engine to the last bit: the gradient's mask [A > 0] must
// not depend on the path.  log p does not see the last bit's sign and splits K.
hipError_t launch_f32_hidden(const vqmc_made& m, const int8_t* S, int64_t B, float* R, float* Rt, int64_t ldr,
                             bool ordered, hipStream_t st) {
  const int64_t ldn = round_up(m.n, kPad), ldh = round_up(m.h, kPad), ldB = round_up(B, kPad);
  auto go = [&](auto kern, int bm, int bn, int nt) {
    kern<<<dim3(tiles(m.h, bn), tiles(ldB, bm)), nt, 0, st>>>(S, ldn, (const float*)m.P, ldh, m.b1, m.c, m.n, m.h, B, R, Rt,
                                                              ldr);
    return hipGetLastError();
  };
  using FOne = F32<1, 1, 1>;
  using FFour = F32<2, 2, 1>;
  if (ordered)
    return f32_large(ldB, ldh) ? go(f32_hidden_kernel<FFour>, FFour::BM, FFour::BN, FFour::NT)
                               : go(f32_hidden_kernel<FOne>, FOne::BM, FOne::BN, FOne::NT);
  return f32_large(ldB, ldh) ? go(f32_hidden_kernel<FLarge>, FLarge::BM, FLarge::BN, FLarge::NT)
                             : go(f32_hidden_kernel<FSmall>, FSmall::BM, FSmall::BN, FSmall::NT);
}

// (32 x 64 tiles where the other products take 32 x 32 ones: half the partial sums, so that the scratch of
// vqmc_logprob_noalloc goes as far as with 64 x 64 tiles)
hipError_t launch_f32_logp(const vqmc_made& m, const int8_t* S, int64_t B, const float* Rt, int64_t ldr, float* lp_part,
                           float* Z, int* nparts, hipStream_t st) {
  const int64_t ldn = round_up(m.n, kPad), ldB = round_up(B, kPad);
  auto go = [&](auto kern, int bm, int bn, int nt) {
    *nparts = (int)tiles(m.n, bn);
    kern<<<dim3(tiles(m.n, bn), tiles(B, bm)), nt, 0, st>>>(Rt, ldr, (const float*)m.Pt, ldn, m.b2, m.c, m.n, m.h, B, S,
                                                            lp_part, Z, nullptr, nullptr, nullptr, nullptr, nullptr);
    return hipGetLastError();
  };
  using FWide = F32<1, 2, 4>;
  return f32_large(ldB, ldn) ? go(f32_out_kernel<FLarge, false>, FLarge::BM, FLarge::BN, FLarge::NT)
                             : go(f32_out_kernel<FWide, false>, FWide::BM, FWide::BN, FWide::NT);
}

hipError_t launch_f32_out_grad(const vqmc_made& m, const int8_t* S, int64_t B, const float* Rt, const float* coef,
                               float* G, float* Gt, float* St, float* db2_part, int* np2, hipStream_t st) {
  const int64_t ldn = round_up(m.n, kPad), ldB = round_up(B, kPad);
  auto go = [&](auto kern, int bm, int bn, int nt) {
    *np2 = (int)tiles(ldB, bm);
    kern<<<dim3(tiles(m.n, bn), tiles(ldB, bm)), nt, 0, st>>>(Rt, ldB, (const float*)m.Pt, ldn, m.b2, m.c, m.n, m.h, B, S,
                                                              nullptr, nullptr, coef, G, Gt, St, db2_part);
    return hipGetLastError();
  };
  if (f32_far(ldB)) return go(f32_out_kernel<FLarge, true, FFar>, FLarge::BM, FLarge::BN, FLarge::NT);
  return f32_large(ldB, ldn) ? go(f32_out_kernel<FLarge, true>, FLarge::BM, FLarge::BN, FLarge::NT)
                             : go(f32_out_kernel<FSmall, true>, FSmall::BM, FSmall::BN, FSmall::NT);
}

hipError_t launch_f32_adjoint(const vqmc_made& m, int64_t B, const float* Gt, const float* Rt, float* D, float* Dt,
                              float* R, float* db1_part, int* np1, hipStream_t st) {
  const int64_t ldh = round_up(m.h, kPad), ldB = round_up(B, kPad);
  auto go = [&](auto kern, int bm, int bn, int nt) {
    *np1 = (int)tiles(ldB, bm);
    kern<<<dim3(tiles(m.h, bn), tiles(ldB, bm)), nt, 0, st>>>(Gt, ldB, (const float*)m.P, ldh, m.c, m.n, m.h, B, Rt, D, Dt,
                                                              R, db1_part);
    return hipGetLastError();
  };
  if (f32_far(ldB)) return go(f32_adjoint_kernel<FLarge, FFar>, FLarge::BM, FLarge::BN, FLarge::NT);
  return f32_large(ldB, ldh) ? go(f32_adjoint_kernel<FLarge>, FLarge::BM, FLarge::BN, FLarge::NT)
                             : go(f32_adjoint_kernel<FSmall>, FSmall::BM, FSmall::BN, FSmall::NT);
}

hipError_t launch_f32_weight(const vqmc_made& m, const int8_t* S, int64_t B, const float* G, const float* R,
                             const float* D, float* dP, const float* db2_part, int np2, const float* db1_part, int np1,
                             float* db2, float* db1, hipStream_t st) {
  const int64_t ldn = round_up(m.n, kPad), ldh = round_up(m.h, kPad);
  auto go = [&](auto kern, int bm, int bn, int nt, int halves) {
    const int64_t ntile = (int64_t)tiles(m.n, bm) * tiles(m.h, bn);
    kern<<<(unsigned)(halves * ntile + tiles(m.n, 64) + tiles(m.h, 64)), nt, 0, st>>>(
        G, ldn, R, ldh, S, D, B, m.c, m.n, m.h, dP, (int)ntile, db2_part, np2, db1_part, np1, db2, db1);
    return hipGetLastError();
  };
  return f32_large(m.n, m.h) ? go(f32_weight_kernel<FLarge, false>, FLarge::BM, FLarge::BN, FLarge::NT, 1)
                             : go(f32_weight_kernel<FSmall, true>, FSmall::BM, FSmall::BN, FSmall::NT, 2);
}

}  // namespace vqmc
