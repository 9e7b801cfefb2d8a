// BF16 products of the masked MADE fed by direct-to-LDS loads (gfx950).
//
//   A[b][k] = b1[k] + sum_{d : c[d] <= k} S[b][d] P[d][k],  R = relu(A)      (first layer)
//   Z[b][d] = b2[d] + sum_{k < c[d]} R[b][k] P[d][k]                         (second layer)
//   D[b][k] = [A[b][k] > 0] sum_{d : c[d] > k} G[b][d] P[d][k]                (dF/dA)
//   dP[d][k] = sum_b G[b][d] R[b][k] (k < c[d]),  sum_b S[b][d] D[b][k] (else)
//
// Engine: a BM x BN tile per workgroup of WGM x WGN waves, each a grid of v_mfma_f32_16x16x32_bf16
// blocks (FP32 accumulation, ks in rising order).  K advances 64 elements per stage; NS stages rotate
// through LDS arrays of their own, NS - 1 of them in flight while one is multiplied.  A stage is
// brought in by global_load_lds_dwordx4 (16 bytes per lane straight into LDS, no registers): a wave
// instruction fills 1 KB of rows, from a per-lane byte offset fixed for the whole run.  The 16-byte chunk
// c of row r is stored at position c ^ (r % 8), so the 16 rows an MFMA operand read touches spread
// over the LDS banks.  A wave waits for its own loads of a stage (vmcnt) before the stage's
// barrier; after the barrier every wave's loads of that stage have landed, and the next stage to fetch
// goes into the buffer every wave has finished reading.
//
// Spins stay int8 up to the matrix operand: a row of a stage is 64 bytes, and the sign and lowest bit
// of a byte are an FP8 number (+-2^-9 or 0) that one conversion with scale 2^9 makes a pair of BF16.
// The staircase masks touch only the stages between the first and the last limit of the tile's rows:
// there the weight operand is masked in registers, elsewhere it is used as loaded (and everywhere where the adjoint
// has the masked copy of the sampler's tables).
//
// What bounds it: the chain of stages of one tile.  The longest column of tiles launched alone takes 43 of the first
// layer's 48 us and 50 of the adjoint's 54 (157 stages of 0.3 us: barrier, operand reads, products, the
// issue of the next loads, which move 40 - 50 of the 128 GB/s that a CU's loads into LDS can);
// deeper rings, two stages per barrier, twice the waves and operands read a stage ahead change nothing.
// For short runs it is a tile's start and epilogue.  So long runs take small tiles (more of
// them at once, long and short ranges paired on a CU) until the tiles fill the chip several times; there
// and in the weight gradient, whose runs are all alike, large tiles halve the operand reads per product.
// Both halves of a stage read as one set of operands cost the large adjoint 96 us instead of 70 below.
// Measured (us; before: operands staged through registers, conversions and masks in the loop; adjoint and
// weights of a step: 64 x 128 and 128 x 128 tiles on a masked copy of P^T):
//                               n = 10000, h = 1000,   n = 3001, h = 611,   n = h = 2000,
//                               B = 2048               B = 1500             B = 8192
//   first layer                 48 (282)               21 (94)              82
//   second layer, log p         53 (157)               17 (35)              78
//   second layer, gradient                             21 (48)
//   hidden adjoint              54 (70)                18 (66)              70 (75)
//   ... with the masked copy    53                                          60
//   weight and bias gradients   66 (78)                16 (72 + 9)          113 (123)
#include "common.hpp"
#include "kernels.hpp"

namespace vqmc {

typedef __attribute__((address_space(3))) void b_lds_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;

// The barrier between two stages: the wave's loads but the last N have landed in LDS and its operand reads
// have returned (so the buffer read last may be filled again); no memory access moves across it.
template <int N>
__device__ inline void b_stage_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));  // vmcnt(N) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
__device__ inline const uint8_t* b_uniform(const uint8_t* p) {
  const uint64_t v = (uint64_t)p;
  return (const uint8_t*)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
                          (uint32_t)__builtin_amdgcn_readfirstlane((int)v));
}

enum BMask { B_ALL, B_BELOW, B_FROM };  // ks of a weight row that count: all, those below its limit, those from it on

template <int BM_, int BN_, int WGM_, int WGN_, int NS_, bool SPIN_, BMask MASK_>
struct BE {
  static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, NS = NS_;
  static constexpr bool SPIN = SPIN_;
  static constexpr BMask MASK = MASK_;
  static constexpr int NW = WGM * WGN, NT = 64 * NW;
  static constexpr int FM = BM / (16 * WGM), FN = BN / (16 * WGN);  // 16x16 blocks per wave
  static constexpr int AROW = SPIN ? 64 : 128;                      // bytes of an A row per stage
  static constexpr int ABYTES = BM * AROW, STAGE = ABYTES + BN * 128;
  static constexpr int AI = ABYTES / (1024 * NW), BI = BN * 128 / (1024 * NW);  // load instructions per wave
  static constexpr int NLD = AI + BI;
  static_assert(AI * 1024 * NW == ABYTES && BI * 1024 * NW == BN * 128, "a stage must split evenly over the waves");
  static_assert(NS >= 2 && NS <= 6, "stages");

  // K columns of a row-major matrix (bf16, or int8 for spins) from row0 on; rows past rows - 1 are
  // loaded as the last one (their results are never stored)
  struct Op {
    const void* X;
    int64_t ld;  // elements; a multiple of 64, zero padding
    int64_t row0, rows;
  };
  // K range [kbeg, kend) in steps of 32 of the stages from kbeg / 64 on; the ks [mbeg, mend) need the mask
  struct Range {
    int kbeg, kend, mbeg, mend;
  };
  // per-lane offsets, fixed for a run: of the loads from column 0 of the operands, of the operand reads
  // of the two K halves from the start of a stage
  struct Lanes {
    uint32_t a[AI], b[BI], fa[2], fb[2];
    int wv;
  };
  __device__ static int wave() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
  __device__ static int wm() { return (wave() / WGN) * (BM / WGM); }
  __device__ static int wn() { return (wave() % WGN) * (BN / WGN); }

  __device__ static Lanes lanes(const Op& a, const Op& b) {
    Lanes L;
    const int lane = threadIdx.x & 63, g = lane >> 4;
    L.wv = wave();
#pragma unroll
    for (int j = 0; j < AI; ++j) {
      const int r = SPIN ? 16 * (NW * j + L.wv) + (lane >> 2) : 8 * (NW * j + L.wv) + (lane >> 3);
      const int p = SPIN ? ((lane & 3) ^ ((r >> 2) & 3)) : ((lane & 7) ^ (r & 7));
      const int64_t row = min((int64_t)r, a.rows - 1 - a.row0);
      L.a[j] = (uint32_t)(row * a.ld * (SPIN ? 1 : 2) + 16 * p);
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
      const int r = 8 * (NW * j + L.wv) + (lane >> 3);
      const int64_t row = min((int64_t)r, b.rows - 1 - b.row0);
      L.b[j] = (uint32_t)(row * b.ld * 2 + 16 * ((lane & 7) ^ (r & 7)));
    }
    const int ra = wm() + (lane & 15), rb = wn() + (lane & 15);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      L.fa[ks] = SPIN ? ra * 64 + 16 * ((2 * ks + (g >> 1)) ^ ((ra >> 2) & 3)) + 8 * (g & 1)
                      : ra * 128 + 16 * ((4 * ks + g) ^ (ra & 7));
      L.fb[ks] = ABYTES + rb * 128 + 16 * ((4 * ks + g) ^ (rb & 7));
    }
    return L;
  }
  // K columns [k, k + 64) into a stage.  Past the end of the range (!live) every lane fetches the same 16
  // bytes, never used, so that the count of loads in flight is the same on every path.
  __device__ static void issue(const uint8_t* ab, const uint8_t* bb, const Lanes& L, int k, bool live, uint4* st) {
    const uint32_t keep = live ? ~0u : 0u;
    ab = b_uniform(ab + (int64_t)k * (SPIN ? 1 : 2));
    bb = b_uniform(bb + (int64_t)k * 2);
    uint8_t* s = (uint8_t*)st + 1024 * L.wv;
#pragma unroll
    for (int j = 0; j < AI; ++j)
      __builtin_amdgcn_global_load_lds((const void*)(ab + (L.a[j] & keep)), (b_lds_t*)(s + 1024 * NW * j), 16, 0, 0);
#pragma unroll
    for (int j = 0; j < BI; ++j)
      __builtin_amdgcn_global_load_lds((const void*)(bb + (L.b[j] & keep)), (b_lds_t*)(s + ABYTES + 1024 * NW * j), 16,
                                       0, 0);
  }

  __device__ static bf16x8_t keep_if(bf16x8_t x, uint32_t m) {
    uint4 v = __builtin_bit_cast(uint4, x);
    v.x &= m; v.y &= m; v.z &= m; v.w &= m;
    return __builtin_bit_cast(bf16x8_t, v);
  }
  // the lane's 8 ks from k on, those the limit excludes cleared
  __device__ static bf16x8_t masked(bf16x8_t x, int k, int limit) {
    uint4 v = __builtin_bit_cast(uint4, x);
    uint32_t* w = (uint32_t*)&v;
    const int nv = limit - k;  // ks below the limit
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t below = nv >= 2 * q + 2 ? ~0u : (nv == 2 * q + 1 ? 0xFFFFu : 0u);
      w[q] &= MASK == B_BELOW ? below : ~below;
    }
    return __builtin_bit_cast(bf16x8_t, v);
  }

  // eight spins (bytes +-1 or 0) as BF16
  __device__ static bf16x8_t spins(uint2 s) {
    const uint32_t x = s.x & 0x81818181u, y = s.y & 0x81818181u;
    const bf16x2_t a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x, 512.f, false);
    const bf16x2_t b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x, 512.f, true);
    const bf16x2_t c = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(y, 512.f, false);
    const bf16x2_t d = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(y, 512.f, true);
    return (bf16x8_t){a[0], a[1], b[0], b[1], c[0], c[1], d[0], d[1]};
  }

  // the operands of half ks of a stage (32 ks)
  struct Frags {
    bf16x8_t a[FM], b[FN];
    uint2 raw[FM];
  };
  __device__ static void read(const uint4* st, const Lanes& L, int ks, Frags& f) {
    const uint8_t* s = (const uint8_t*)st;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      if constexpr (SPIN) f.raw[i] = *(const uint2*)(s + L.fa[ks] + i * 16 * 64);
      else f.a[i] = *(const bf16x8_t*)(s + L.fa[ks] + i * 16 * 128);
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) f.b[j] = *(const bf16x8_t*)(s + L.fb[ks] + j * 16 * 128);
  }
  // masks the weights of the half whose first K column is k0 and clears it if it lies outside the range (both
  // operands: an infinity there must not become a NaN), without branches, so the sums stay in place
  __device__ static void mask(Frags& f, int k0, const Range& q, const int (&limit)[FN]) {
    const uint32_t in = k0 >= q.kbeg && k0 < q.kend ? ~0u : 0u;
    if constexpr (!SPIN) {
#pragma unroll
      for (int i = 0; i < FM; ++i) f.a[i] = keep_if(f.a[i], in);
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      f.b[j] = keep_if(f.b[j], in);
      if constexpr (MASK != B_ALL) f.b[j] = masked(f.b[j], k0 + 8 * (int)((threadIdx.x & 63) >> 4), limit[j]);
    }
  }
  __device__ static void multiply(Frags& f, floatx4_t (&acc)[FM][FN]) {
    if constexpr (SPIN) {
#pragma unroll
      for (int i = 0; i < FM; ++i) f.a[i] = spins(f.raw[i]);
    }
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
  }

  // Starts the run: fetches its first NS - 1 stages, from column k on (ld columns in all, so before the end
  // of the range need be known).
  __device__ static Lanes start(const Op& a, const Op& b, int k, int64_t ld, uint4* const (&st)[NS]) {
    const Lanes L = lanes(a, b);
    const int nst = (int)(ld / 64) - k / 64;
#pragma unroll
    for (int p = 0; p < NS - 1; ++p) issue(base(a, SPIN ? 1 : 2, k), base(b, 2, k), L, 64 * min(p, nst - 1), p < nst, st[p]);
    return L;
  }
  __device__ static const uint8_t* base(const Op& o, int es, int k) {
    return (const uint8_t*)o.X + (o.row0 * o.ld + k / 64 * 64) * es;
  }

  // acc = A x B^T over the range, after start from its first column; limit: those of the lane's weight rows
  // (wn() + 16 j + lane % 16)
  __device__ static void run(const Op& a, const Op& b, const Lanes& L, const Range& q, const int (&limit)[FN],
                             uint4* const (&st)[NS], floatx4_t (&acc)[FM][FN]) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = (floatx4_t){0.f, 0.f, 0.f, 0.f};
    const int s0 = q.kbeg / 64, nst = q.kend > q.kbeg ? (q.kend + 63) / 64 - s0 : 0;
    const uint8_t* ab = base(a, SPIN ? 1 : 2, q.kbeg);
    const uint8_t* bb = base(b, 2, q.kbeg);
    // groups of NS stages: first those that need a mask (B_FROM), then the plain ones, then masks and
    // the end (the last group may run past it: its surplus stages only wait)
    const int m0 = q.kbeg % 64 ? max(q.mend, q.kbeg / 64 * 64 + 1) : q.mend;
    const int lead = MASK == B_FROM ? min((m0 + 63) / 64 - s0, nst) : 0;  // stages masked at the start
    const int plain = MASK == B_BELOW ? min(q.mbeg / 64 - s0, nst) : nst;   // first one masked after that
    int i = 0;
    auto step = [&](int p, bool live, bool edge) {
      b_stage_barrier<(NS - 2) * NLD>();
      issue(ab, bb, L, live ? 64 * (i + p + NS - 1) : 64 * min(i + p + NS - 1, nst - 1), live || i + p + NS - 1 < nst,
            st[(p + NS - 1) % NS]);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        Frags f;
        read(st[p], L, ks, f);
        if (edge) mask(f, 64 * (s0 + i + p) + 32 * ks, q, limit);
        multiply(f, acc);
      }
    };
    auto edge = [&](int end) {
      for (; i < end; i += NS) {
#pragma unroll
        for (int p = 0; p < NS; ++p) step(p, false, true);
      }
    };
    if constexpr (MASK == B_FROM) edge(lead);
    for (; i + NS <= plain && i + 2 * NS - 1 <= nst; i += NS) {
#pragma unroll
      for (int p = 0; p < NS; ++p) step(p, true, false);
    }
    edge(nst);
    // drain the loads still in flight before the buffers are reused
    b_stage_barrier<0>();
  }
};

// LDS of an engine: one array per stage (a stage being read must not alias one being filled)
#define B_STAGES(E, st)                                                                                   \
  __shared__ __attribute__((aligned(16))) uint4 st##0[E::STAGE / 16], st##1[E::STAGE / 16],               \
      st##2[E::NS > 2 ? E::STAGE / 16 : 1], st##3[E::NS > 3 ? E::STAGE / 16 : 1],                         \
      st##4[E::NS > 4 ? E::STAGE / 16 : 1], st##5[E::NS > 5 ? E::STAGE / 16 : 1];                         \
  uint4* const st##_all[6] = {st##0, st##1, st##2, st##3, st##4, st##5};                                  \
  uint4* st[E::NS];                                                                                       \
  _Pragma("unroll") for (int p_ = 0; p_ < E::NS; ++p_) st[p_] = st##_all[p_]

// Tiles of a grid whose K ranges differ by column: workgroup w -> (row, column).  Workgroups are dealt
// round-robin to the 8 XCDs, each with its own L2: XCD x takes the rows x, x + 8, ... with all their columns,
// so a row's operand is fetched into one L2.  It runs through the columns from the longest range to
// the shortest; where its tiles fill its 32 CUs once but not twice, those past the first 32 come in
// the opposite order, so that the CU with the longest range gets the shortest second one.
// Launch b_grid(nrow, ncol); row >= nrow marks a surplus workgroup.
__device__ inline void b_tile(int w, int nrow, int ncol, int& row, int& rank) {
  const int x = w & 7, nr = (nrow + 7) / 8, T = nr * ncol;
  int i = w >> 3;
  if (T > 32 && T <= 64 && i >= 32) i = T + 31 - i;
  rank = __builtin_amdgcn_readfirstlane(i / nr);  // 0: the longest range
  row = __builtin_amdgcn_readfirstlane(x + 8 * (i - nr * rank));
}
__host__ inline unsigned b_grid(int64_t nrow, int64_t ncol) { return (unsigned)(8 * ((nrow + 7) / 8) * ncol); }

// ---------------------------------------------------------------- first layer
// R = relu(S P_upper + b1) by sample (B x ldh, units past h zero), if Rt by unit (h x ldB, zero past B), if A also
// the FP32 pre-activations (B x ldh)
template <class E>
__global__ __launch_bounds__(E::NT, 2) void b_hidden_kernel(const int8_t* __restrict__ S, int64_t ldn,
                                                           const bf16_t* __restrict__ Pt, const float* __restrict__ b1,
                                                           const int32_t* __restrict__ c, int n, int h, int64_t B,
                                                           bf16_t* __restrict__ R, int64_t ldh, bf16_t* __restrict__ Rt,
                                                           int64_t ldB, float* __restrict__ A) {
  B_STAGES(E, st);
  __shared__ int bound[E::BN];
  const int t = threadIdx.x, lane = t & 63;
  const int ncol = (h + E::BN - 1) / E::BN, nrow = (int)((B + E::BM - 1) / E::BM);
  int row, rank;
  b_tile(blockIdx.x, nrow, ncol, row, rank);
  if (row >= nrow) return;
  const int64_t m0 = (int64_t)row * E::BM;  // samples
  const int n0 = (ncol - 1 - rank) * E::BN;  // units: later ones see more sites
  const typename E::Op oa{S, ldn, m0, B}, ob{Pt, ldn, n0, h};
  const typename E::Lanes L = E::start(oa, ob, 0, ldn, st);
  int first, last;
  unit_limits<E::BN, E::NT>(bound, c, n, h, n0, first, last);
  int limit[E::FN];
  float bias[E::FN];
#pragma unroll
  for (int j = 0; j < E::FN; ++j) {
    const int u = E::wn() + 16 * j + (lane & 15);
    limit[j] = bound[u];
    bias[j] = n0 + u < h ? b1[n0 + u] : 0.f;
  }
  floatx4_t acc[E::FM][E::FN];
  E::run(oa, ob, L, {0, last, first, n}, limit, st, acc);
  constexpr int TS = E::BN + 8;
  bf16_t* T = (bf16_t*)st[0];  // the tile by sample
  static_assert(E::BM * TS * 2 <= E::STAGE, "tile staging");
#pragma unroll
  for (int j = 0; j < E::FN; ++j) {
    const int u = E::wn() + 16 * j + (lane & 15), k = n0 + u;
#pragma unroll
    for (int i = 0; i < E::FM; ++i) {
      const int mr = E::wm() + 16 * i + 4 * (lane >> 4);
      bf16_t v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool ok = k < h && m0 + mr + e < B;
        const float a = acc[i][j][e] + bias[j];
        v[e] = f32_to_bf16(ok ? fmaxf(a, 0.f) : 0.f);
        T[(mr + e) * TS + u] = v[e];
        if (A && m0 + mr + e < B && k < ldh) A[(m0 + mr + e) * ldh + k] = k < h ? a : 0.f;
      }
      if (Rt && k < h && m0 + mr < ldB) *(uint2*)(Rt + (int64_t)k * ldB + m0 + mr) = *(const uint2*)v;
    }
  }
  __syncthreads();
  for (int x = t; x < E::BM * E::BN / 8; x += E::NT) {
    const int m = x / (E::BN / 8), q = x % (E::BN / 8);
    if (m0 + m < B && n0 + 8 * q < ldh) *(uint4*)(R + (m0 + m) * ldh + n0 + 8 * q) = *(const uint4*)(T + m * TS + 8 * q);
  }
}

// ---------------------------------------------------------------- second layer
// GRAD = false: log sigma partials (one row of B per site tile) and, if Z, the logits (B x ldn).
// GRAD = true: G = coef s sigma(-s z) by sample (B x ldn) and by site (Gt, n x ldB, zero past B), the
// spins by site (St, the same) and db2 partials (one row of ldn per sample tile).
template <class E, bool GRAD, int OCC = 2>
__global__ __launch_bounds__(E::NT, OCC) void b_out_kernel(const bf16_t* __restrict__ R, int64_t ldh,
                                                        const bf16_t* __restrict__ P, const float* __restrict__ b2,
                                                        const int32_t* __restrict__ c, int n, int h, int64_t B,
                                                        const int8_t* __restrict__ S, int64_t ldn,
                                                        float* __restrict__ lp_part, float* __restrict__ Z,
                                                        const float* __restrict__ coef, bf16_t* __restrict__ G,
                                                        bf16_t* __restrict__ Gt, bf16_t* __restrict__ St, int64_t ldB,
                                                        float* __restrict__ db2_part) {
  B_STAGES(E, st);
  __shared__ float rowacc[E::WGN][E::BM];
  __shared__ float colacc[E::WGM][E::BN];
  const int t = threadIdx.x, lane = t & 63;
  // eight site tiles at a time go round the XCDs (the weights are the larger operand), those left over run through
  // their batch tiles in order; later sites see more units and come first
  const int nsite = (n + E::BN - 1) / E::BN, nbat = (int)((B + E::BM - 1) / E::BM), dealt = (nsite & ~7) * nbat;
  const int w = blockIdx.x, v = w < dealt ? w >> 3 : w - dealt;
  const int q = __builtin_amdgcn_readfirstlane(v / nbat), mt = v - nbat * q;
  const int tile = nsite - 1 - (w < dealt ? (w & 7) + 8 * q : (nsite & ~7) + q);
  const int64_t m0 = (int64_t)mt * E::BM;
  const int d0 = tile * E::BN;
  const typename E::Op oa{R, ldh, m0, B}, ob{P, ldh, d0, n};
  const typename E::Lanes L = E::start(oa, ob, 0, ldh, st);
  // the epilogue's inputs are loaded before the products
  constexpr int NSV = E::BM * E::BN / 16 / E::NT;
  uint4 sv16[NSV];
#pragma unroll
  for (int v = 0; v < NSV; ++v) {
    const int x = t + v * E::NT, m = x / (E::BN / 16), q = x % (E::BN / 16);
    sv16[v] = make_uint4(0, 0, 0, 0);
    if (m0 + m < B && d0 + 16 * q < ldn) sv16[v] = *(const uint4*)(S + (m0 + m) * ldn + d0 + 16 * q);
  }
  int limit[E::FN];
  float bias[E::FN];
#pragma unroll
  for (int j = 0; j < E::FN; ++j) {
    const int d = d0 + E::wn() + 16 * j + (lane & 15);
    limit[j] = d < n ? c[d] : 0;
    bias[j] = d < n ? b2[d] : 0.f;
  }
  float cf[E::FM][4];
  if constexpr (GRAD) {
#pragma unroll
    for (int i = 0; i < E::FM; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t b = m0 + E::wm() + 16 * i + 4 * (lane >> 4) + e;
        cf[i][e] = b < B ? coef[b] : 0.f;
      }
  }
  floatx4_t acc[E::FM][E::FN];
  const int first = __builtin_amdgcn_readfirstlane(c[d0]), last = __builtin_amdgcn_readfirstlane(c[min(d0 + E::BN, n) - 1]);
  E::run(oa, ob, L, {0, last, first, h}, limit, st, acc);
  constexpr int TS = E::BN + 8;
  constexpr int SS = E::BN + 16;  // stride of the spin tile
  bf16_t* T = (bf16_t*)st[0];
  int8_t* sp = (int8_t*)st[1];
  static_assert(E::BM * TS * 2 <= E::STAGE && E::BM * SS <= E::STAGE, "tile staging");
#pragma unroll
  for (int v = 0; v < NSV; ++v) {
    const int x = t + v * E::NT;
    *(uint4*)(sp + (x / (E::BN / 16)) * SS + 16 * (x % (E::BN / 16))) = sv16[v];
  }
  __syncthreads();
  float rs[E::FM][4] = {};
  float cs[E::FN] = {};
#pragma unroll
  for (int j = 0; j < E::FN; ++j) {
    const int u = E::wn() + 16 * j + (lane & 15), d = d0 + u;
#pragma unroll
    for (int i = 0; i < E::FM; ++i) {
      const int mr = E::wm() + 16 * i + 4 * (lane >> 4);
      bf16_t gv[4], sv[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool ok = d < n && m0 + mr + e < B;
        const int8_t si = sp[(mr + e) * SS + u];
        const float z = acc[i][j][e] + bias[j], s = (float)si, tt = s * z;
        if constexpr (GRAD) {
          const float g = ok ? cf[i][e] * s * sigmoid(-tt) : 0.f;
          cs[j] += g;
          gv[e] = f32_to_bf16(g);
          sv[e] = (!ok || si == 0) ? (bf16_t)0 : (si > 0 ? (bf16_t)0x3F80 : (bf16_t)0xBF80);
          T[(mr + e) * TS + u] = gv[e];
        } else {
          if (ok) rs[i][e] += log_sigmoid(tt);
          if (Z && ok) Z[(m0 + mr + e) * ldn + d] = z;
        }
      }
      if (GRAD && d < n && m0 + mr < ldB) {
        *(uint2*)(Gt + (int64_t)d * ldB + m0 + mr) = *(const uint2*)gv;
        *(uint2*)(St + (int64_t)d * ldB + m0 + mr) = *(const uint2*)sv;
      }
    }
  }
  if constexpr (GRAD) {
#pragma unroll
    for (int j = 0; j < E::FN; ++j) {
      float v = cs[j];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (lane < 16) colacc[E::wave() / E::WGN][E::wn() + 16 * j + lane] = v;
    }
  } else {
#pragma unroll
    for (int i = 0; i < E::FM; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v = rs[i][e];
        v += VQMC_DPP(v, 0xB1);
        v += VQMC_DPP(v, 0x4E);
        v += VQMC_DPP(v, 0x141);
        v += VQMC_DPP(v, 0x140);
        if ((lane & 15) == 0) rowacc[E::wave() % E::WGN][E::wm() + 16 * i + 4 * (lane >> 4) + e] = v;
      }
  }
  __syncthreads();
  if constexpr (GRAD) {
    for (int x = t; x < E::BM * E::BN / 8; x += E::NT) {
      const int m = x / (E::BN / 8), q = x % (E::BN / 8);
      if (m0 + m < B && d0 + 8 * q < ldn) *(uint4*)(G + (m0 + m) * ldn + d0 + 8 * q) = *(const uint4*)(T + m * TS + 8 * q);
    }
    for (int x = t; x < E::BN; x += E::NT) {
      float v = colacc[0][x];
#pragma unroll
      for (int q = 1; q < E::WGM; ++q) v += colacc[q][x];
      if (d0 + x < ldn) db2_part[(int64_t)mt * ldn + d0 + x] = v;
    }
  } else {
    for (int x = t; x < E::BM; x += E::NT) {
      float v = rowacc[0][x];
#pragma unroll
      for (int q = 1; q < E::WGN; ++q) v += rowacc[q][x];
      if (m0 + x < B) lp_part[(int64_t)tile * B + m0 + x] = v;
    }
  }
}

// ---------------------------------------------------------------- hidden adjoint
// Dt = [Rt > 0] (G P_lower) by unit (h x ldB, zero past B) and db1 partials (one row of ldh per sample tile).  E::MASK =
// B_ALL: Pt is the masked copy of P^T.
template <class E>
__global__ __launch_bounds__(E::NT, 2) void b_adjoint_kernel(const bf16_t* __restrict__ G, int64_t ldn,
                                                            const bf16_t* __restrict__ Pt, const int32_t* __restrict__ c,
                                                            int n, int h, int64_t B, const bf16_t* __restrict__ Rt,
                                                            bf16_t* __restrict__ Dt, int64_t ldB,
                                                            float* __restrict__ db1_part, int64_t ldh) {
  B_STAGES(E, st);
  __shared__ int bound[E::BN];
  __shared__ float colacc[E::WGM][E::BN];
  const int t = threadIdx.x, lane = t & 63;
  const int ncol = (h + E::BN - 1) / E::BN, nrow = (int)((B + E::BM - 1) / E::BM);
  int row, rank;
  b_tile(blockIdx.x, nrow, ncol, row, rank);
  if (row >= nrow) return;
  const int64_t m0 = (int64_t)row * E::BM;
  const int n0 = rank * E::BN;  // units: earlier ones feed more sites
  uint2 rv[E::FM][E::FN];
#pragma unroll
  for (int j = 0; j < E::FN; ++j)
#pragma unroll
    for (int i = 0; i < E::FM; ++i) {
      const int k = n0 + E::wn() + 16 * j + (lane & 15);
      const int64_t bb = m0 + E::wm() + 16 * i + 4 * (lane >> 4);
      rv[i][j] = k < h && bb < ldB ? *(const uint2*)(Rt + (int64_t)k * ldB + bb) : make_uint2(0, 0);
    }
  int first, last;
  unit_limits<E::BN, E::NT>(bound, c, n, h, n0, first, last);
  int limit[E::FN];
#pragma unroll
  for (int j = 0; j < E::FN; ++j) limit[j] = bound[E::wn() + 16 * j + (lane & 15)];
  const typename E::Op oa{G, ldn, m0, B}, ob{Pt, ldn, n0, h};
  const int kbeg = E::MASK == B_ALL ? first / 64 * 64 : first / 32 * 32;
  const typename E::Lanes L = E::start(oa, ob, kbeg, ldn, st);
  floatx4_t acc[E::FM][E::FN];
  E::run(oa, ob, L, {kbeg, n, first, last}, limit, st, acc);
#pragma unroll
  for (int j = 0; j < E::FN; ++j) {
    const int u = E::wn() + 16 * j + (lane & 15), k = n0 + u;
    float cs = 0.f;
#pragma unroll
    for (int i = 0; i < E::FM; ++i) {
      const int64_t bb = m0 + E::wm() + 16 * i + 4 * (lane >> 4);
      bf16_t r[4], v[4];
      *(uint2*)r = rv[i][j];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float d = (bf16_to_f32(r[e]) > 0.f && bb + e < B) ? acc[i][j][e] : 0.f;
        cs += d;
        v[e] = f32_to_bf16(d);
      }
      if (k < h && bb < ldB) *(uint2*)(Dt + (int64_t)k * ldB + bb) = *(const uint2*)v;
    }
    cs += __shfl_xor(cs, 16);
    cs += __shfl_xor(cs, 32);
    if (lane < 16) colacc[E::wave() / E::WGN][u] = cs;
  }
  __syncthreads();
  for (int x = t; x < E::BN; x += E::NT) {
    float v = colacc[0][x];
#pragma unroll
    for (int q = 1; q < E::WGM; ++q) v += colacc[q][x];
    if (n0 + x < ldh) db1_part[(int64_t)row * ldh + n0 + x] = v;
  }
}

// ---------------------------------------------------------------- weight and bias gradients
// One half of the tile at site d0, unit k0
template <class E>
__device__ inline void b_weight_tile(const bf16_t* Gt, const bf16_t* Rt, const bf16_t* St, const bf16_t* Dt, int64_t ldB,
                                     const int32_t* __restrict__ c, int n, int h, float* __restrict__ dP, int d0, int k0,
                                     bool upper, uint4* const (&st)[E::NS]) {
  const int lane = threadIdx.x & 63;
  const typename E::Op oa{upper ? St : Gt, ldB, d0, n}, ob{upper ? Dt : Rt, ldB, k0, h};
  const typename E::Lanes L = E::start(oa, ob, 0, ldB, st);
  int limit[E::FN];  // unused
  floatx4_t acc[E::FM][E::FN];
  E::run(oa, ob, L, {0, (int)ldB, 0, 0}, limit, st, acc);
#pragma unroll
  for (int i = 0; i < E::FM; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int d = d0 + E::wm() + 16 * i + 4 * (lane >> 4) + e;
      if (d < n) {
        const int cd = c[d];
        float* p = dP + (int64_t)d * h;
#pragma unroll
        for (int j = 0; j < E::FN; ++j) {
          const int k = k0 + E::wn() + 16 * j + (lane & 15);
          if (k < h && (k >= cd) == upper) p[k] = acc[i][j][e];
        }
      }
    }
}

// dP[d][k] = sum_b Gt[d][b] Rt[k][b] (k < c[d]), sum_b St[d][b] Dt[k][b] (else): a workgroup per tile, for the lower
// half if it has an element of it, else for the upper one.  The upper halves of the tiles that the staircase crosses have
// workgroups of their own: one per row of tiles, beside the row's, for the first such tile, and one per column for the
// row that comes into the column further on.  (So any staircase has one workgroup a half: all degrees equal, n = h = 2000,
// B = 2048: 36 us; with the later tiles of a row in one workgroup 230.)  lead: of the columns, rounded up to eight.  The first nbias
// workgroups sum the partials of the bias gradients instead.
template <class E>
__global__ __launch_bounds__(E::NT, 2) void b_weight_kernel(const bf16_t* __restrict__ Gt, const bf16_t* __restrict__ Rt,
                                                           const bf16_t* __restrict__ St, const bf16_t* __restrict__ Dt,
                                                           int64_t ldB, const int32_t* __restrict__ c, int n, int h,
                                                           float* __restrict__ dP, int nbias, int lead,
                                                           const float* __restrict__ db1_part, int np1, int64_t ldh,
                                                           const float* __restrict__ db2_part, int np2, int64_t ldn,
                                                           float* __restrict__ db1, float* __restrict__ db2) {
  B_STAGES(E, st);
  const int t = threadIdx.x, lane = t & 63;
  if ((int)blockIdx.x < nbias) {
    // 64 sums per workgroup, the parts dealt to its waves
    float* red = (float*)st[0];
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    const int wv = E::wave();
    float v = 0.f;
    if (i < n) v = sum_parts(db2_part + wv * ldn, (np2 - wv + E::NW - 1) / E::NW, E::NW * ldn, i);
    else if (i < n + h) v = sum_parts(db1_part + wv * ldh, (np1 - wv + E::NW - 1) / E::NW, E::NW * ldh, i - n);
    red[t] = v;
    __syncthreads();
    if (t < 64) {
#pragma unroll
      for (int q = 1; q < E::NW; ++q) v += red[64 * q + t];
      if (i < n) db2[i] = v;
      else if (i < n + h) db1[i - n] = v;
    }
    return;
  }
  const int nrow = (n + E::BM - 1) / E::BM, ncol = (h + E::BN - 1) / E::BN;
  int row, col;
  bool upper;
  const int w = (int)blockIdx.x - nbias, v = max(w - lead, 0);
  const int g = __builtin_amdgcn_readfirstlane(v / (8 * (ncol + 1))), i = v - 8 * (ncol + 1) * g;
  if (w < lead) {
    // the row in which the staircase comes into column w: the first whose lower elements reach it
    col = w;
    row = 0;
    for (int r0 = 0;; r0 += 64) {
      const int r = r0 + lane;
      const int k = __popcll(__ballot(r < nrow && c[min((r + 1) * E::BM, n) - 1] <= col * E::BN));
      row += k;
      if (k < 64) break;
    }
    row = __builtin_amdgcn_readfirstlane(row);
    // (the row's own workgroup has its first column)
    if (col >= ncol || row >= nrow || c[row * E::BM] / E::BN >= col) return;
    upper = true;
  } else if (i < 8) {
    row = i + 8 * g;
    if (row >= nrow) return;
    const int cfirst = __builtin_amdgcn_readfirstlane(c[row * E::BM]);
    col = cfirst / E::BN;
    if (cfirst >= h || col * E::BN >= __builtin_amdgcn_readfirstlane(c[min((row + 1) * E::BM, n) - 1])) return;
    upper = true;
  } else {
    row = (i & 7) + 8 * g;
    if (row >= nrow) return;
    col = (i >> 3) - 1;
    upper = col * E::BN >= __builtin_amdgcn_readfirstlane(c[min((row + 1) * E::BM, n) - 1]);
  }
  b_weight_tile<E>(Gt, Rt, St, Dt, ldB, c, n, h, dP, row * E::BM, col * E::BN, upper, st);
}

// ---------------------------------------------------------------- launches
using BHidden = BE<64, 64, 2, 2, 4, true, B_BELOW>;
using BOut = BE<64, 128, 2, 4, 2, false, B_BELOW>;
using BAdjoint = BE<64, 64, 2, 2, 4, false, B_FROM>;
using BAdjointLarge = BE<128, 128, 2, 4, 2, false, B_FROM>;
using BAdjointPm = BE<64, 64, 2, 2, 4, false, B_ALL>;
using BAdjointLargePm = BE<128, 128, 2, 4, 2, false, B_ALL>;
using BWeight = BE<128, 128, 4, 4, 4, false, B_ALL>;
using BWeightSmall = BE<64, 64, 2, 2, 4, false, B_ALL>;

static int64_t b_tiles(int64_t x, int t) { return (x + t - 1) / t; }

template <class E>
static hipError_t b_adjoint_t(const vqmc_made& m, const bf16_t* Pt, int64_t B, const bf16_t* G, const bf16_t* Rt, bf16_t* Dt,
                              float* db1_part, int* np1, hipStream_t st) {
  const int64_t ldn = round_up(m.n, kPad), ldh = round_up(m.h, kPad), ldB = round_up(B, kPad);
  *np1 = (int)b_tiles(B, E::BM);
  b_adjoint_kernel<E><<<b_grid(*np1, b_tiles(m.h, E::BN)), E::NT, 0, st>>>(G, ldn, Pt, m.c, m.n, m.h, B, Rt, Dt, ldB, db1_part,
                                                                           ldh);
  return hipGetLastError();
}

hipError_t launch_b_adjoint(const vqmc_made& m, bool tables, int64_t B, const bf16_t* G, const bf16_t* Rt, bf16_t* Dt,
                            float* db1_part, int* np1, hipStream_t st) {
  // 128 x 128 tiles once there are two per CU (the ranges of a column of tiles differ up to its whole
  // length; fewer large tiles leave CUs with one short run): 53 against 63 us at 512 of them (n = h = 2000,
  // B = 4096), 33.5 against 31.6 at 256 (h = 1000), 150 against 56 at n = 10000, h = 1000, B = 2048
  const bool large = b_tiles(B, 128) * b_tiles(m.h, 128) >= 512;
  // The masked copy of P^T among the sampler's tables spares the masks, which are most of a stage where a tile's units lie
  // far apart (n = 10000, h = 100, B = 2048: 42 against 77 us; h = 1000 alike, n = h = 2000: 25 against 31)
  if (tables && m.band && ((uintptr_t)m.band & 15) == 0) {
    int64_t z, u, pm;
    int nz, nu;
    sample_tables_layout(m.n, m.h, m.wdtype, &z, &u, &pm, &nz, &nu);
    const bf16_t* Pm = (const bf16_t*)((const uint8_t*)m.band + pm);
    return large ? b_adjoint_t<BAdjointLargePm>(m, Pm, B, G, Rt, Dt, db1_part, np1, st)
                 : b_adjoint_t<BAdjointPm>(m, Pm, B, G, Rt, Dt, db1_part, np1, st);
  }
  return large ? b_adjoint_t<BAdjointLarge>(m, (const bf16_t*)m.Pt, B, G, Rt, Dt, db1_part, np1, st)
               : b_adjoint_t<BAdjoint>(m, (const bf16_t*)m.Pt, B, G, Rt, Dt, db1_part, np1, st);
}

template <class E>
static hipError_t b_weight_t(const vqmc_made& m, int64_t B, const bf16_t* Gt, const bf16_t* St, const bf16_t* Rt,
                             const bf16_t* Dt, float* dP, const float* db2_part, int np2, const float* db1_part, int np1,
                             float* db2, float* db1, hipStream_t st) {
  const int64_t ldn = round_up(m.n, kPad), ldh = round_up(m.h, kPad), ldB = round_up(B, kPad);
  const int nbias = (int)(round_up((int64_t)m.n + m.h, 512) / 64);  // a multiple of 8: the tiles keep their XCDs
  const int64_t nrow = b_tiles(m.n, E::BM), ncol = b_tiles(m.h, E::BN);
  const int lead = (int)round_up(ncol, 8);
  b_weight_kernel<E><<<nbias + lead + b_grid(nrow, ncol + 1), E::NT, 0, st>>>(
      Gt, Rt, St, Dt, ldB, m.c, m.n, m.h, dP, nbias, lead, db1_part, np1, ldh, db2_part, np2, ldn, db1, db2);
  return hipGetLastError();
}

hipError_t launch_b_weight(const vqmc_made& m, int64_t B, const bf16_t* Gt, const bf16_t* St, const bf16_t* Rt,
                           const bf16_t* Dt, float* dP, const float* db2_part, int np2, const float* db1_part, int np1,
                           float* db2, float* db1, hipStream_t st) {
  // 64 x 64 tiles while 128 x 128 ones would leave most CUs idle: 5.7 against 8.9 us at 16 of them (n = 1000,
  // h = 239, B = 512), 13.6 against 15.3 at 64 (n = 2000, h = 500, B = 1500), 41 against 32 at 128
  const bool small = b_tiles(m.n, 128) * b_tiles(m.h, 128) <= 64;
  return small ? b_weight_t<BWeightSmall>(m, B, Gt, St, Rt, Dt, dP, db2_part, np2, db1_part, np1, db2, db1, st)
               : b_weight_t<BWeight>(m, B, Gt, St, Rt, Dt, dP, db2_part, np2, db1_part, np1, db2, db1, st);
}

hipError_t launch_b_hidden(const vqmc_made& m, const int8_t* S, int64_t B, bf16_t* R, bf16_t* Rt, float* A, hipStream_t st) {
  const int64_t ldn = round_up(m.n, kPad), ldh = round_up(m.h, kPad), ldB = round_up(B, kPad);
  b_hidden_kernel<BHidden><<<b_grid((B + BHidden::BM - 1) / BHidden::BM, (m.h + BHidden::BN - 1) / BHidden::BN), BHidden::NT, 0, st>>>(
      S, ldn, (const bf16_t*)m.Pt, m.b1, m.c, m.n, m.h, B, R, ldh, Rt, ldB, A);
  return hipGetLastError();
}

// (64 x 128 tiles of two stages: three workgroups of eight waves per CU hide the start and the epilogue of a
// tile, about 35 of the 54 us at n = 10000, h = 1000, B = 2048; three stages, two workgroups: 67; 64 x 64: 60 - 71)
hipError_t launch_b_logp(const vqmc_made& m, const int8_t* S, int64_t B, const bf16_t* R, float* lp_part, float* Z,
                         int* nparts, hipStream_t st) {
  using E = BOut;
  const int64_t ldn = round_up(m.n, kPad), ldh = round_up(m.h, kPad), ldB = round_up(B, kPad);
  *nparts = (m.n + E::BN - 1) / E::BN;
  b_out_kernel<E, false><<<(unsigned)(*nparts * b_tiles(B, E::BM)), E::NT, 0, st>>>(
      R, ldh, (const bf16_t*)m.P, m.b2, m.c, m.n, m.h, B, S, ldn, lp_part, Z, nullptr, nullptr, nullptr, nullptr, ldB,
      nullptr);
  return hipGetLastError();
}

hipError_t launch_b_out_grad(const vqmc_made& m, const int8_t* S, int64_t B, const bf16_t* R, const float* coef, bf16_t* G,
                             bf16_t* Gt, bf16_t* St, float* db2_part, int* np2, hipStream_t st) {
  using E = BOut;
  const int64_t ldn = round_up(m.n, kPad), ldh = round_up(m.h, kPad), ldB = round_up(B, kPad);
  *np2 = (int)((B + E::BM - 1) / E::BM);
  b_out_kernel<E, true><<<(unsigned)(b_tiles(m.n, E::BN) * *np2), E::NT, 0, st>>>(
      R, ldh, (const bf16_t*)m.P, m.b2, m.c, m.n, m.h, B, S, ldn, nullptr, nullptr, coef, G, Gt, St, ldB, db2_part);
  return hipGetLastError();
}

}  // namespace vqmc
