// HIP kernels (gfx950) for the RK stages of the modal ESDG shallow-water scheme.
//
// One workgroup processes a tile of consecutive elements of one instance:
//   0. every global array the tile needs (its entropy-projected values, the values its
//      face neighbours pushed into its slots, metric factors, state, RK register, the
//      static block of mass data, weights, bathymetry and push targets) is fetched into
//      LDS with asynchronous copies, so the global-memory latency is exposed once per tile;
//   1. node records at the Nh hybridized nodes are built in LDS;
//   2. flux differencing in skew form (Section 5.2, Step 4): every row m of every
//      nonzero block of Q_skew = Q_h - Q_h^T (volume-volume and volume-surface; the zero
//      surface-surface block is skipped), with the element's physical operator built on
//      the fly from averaged geometric factors (Section 2.7) and the EC flux of
//      Section 2.8; each task takes R rows of one element so a column's node record is
//      read once for R rows.  The bathymetry source is folded in as
//      1/2 g h_m (H_n - Href) Q_mn (exact because Q_h 1 = 0);
//   3. interface flux f_S(u~+, u~), boundary half of the source and optional local
//      Lax-Friedrichs penalty (Section 2.8) on the face rows;
//   4. lift rhs = -(M_h^k)^{-1} V_h^T r_h, with the stored inverses (Section 2.8) or the
//      weight-adjusted inverse named after eq. (dgform);
//   5. LSRK update (Section 4), then, fused, the entropy projection of the updated state
//      (Section 2.6), written to the other stage buffer and pushed into the face slots of
//      the neighbours (or, on a reflective wall, Section 2.9, the mirror state into the
//      node's own slot).
// Between stages the face exchange needs every neighbour's projection: either the launch
// boundary (one launch per stage) or, in a multi-stage launch, per-tile progress counts
// that a tile waits on before it reads its neighbours' values.
//
// The products with the constant operators (lift, projection) run on the matrix cores, with the
// columns (field, element) of the tile side by side; the pair loop is a Hadamard product and
// stays on the vector ALUs.  What bounds a stage is the chain of these short phases.
//
// Depth is carried as the free-surface anomaly eta = h + b - Href (Href a per-instance
// constant), so the projection works on v1 - g Href and no quantity of size g H is
// rounded to the bulk precision; the conversions to h are done in double.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cmath>
#include <map>
#include <type_traits>

#include "device_types.hpp"

namespace esdg {

__device__ inline bool bad_value(double h, double a, double b) {
  return !(h > 0.0) || !isfinite(h) || !isfinite(a) || !isfinite(b);
}

// The wave's index in the workgroup, as a wave-uniform (scalar) value: loops over
// wave-sized chunks then keep their counters, bounds and LDS bases in scalar registers.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6); }

// The thread index, read through an empty asm so that the compiler cannot hoist index
// arithmetic derived from it out of the stage loop of a multi-stage launch (hoisted, every
// phase's per-thread indices would stay live across all phases and spill).
__device__ __forceinline__ int phase_tid() {
  int t = int(threadIdx.x);
  asm volatile("" : "+v"(t));
  return t;
}

// Threads of the workgroup: a constant in the kernels built for one kind (LT::NT).
template <int T> struct Threads { static constexpr int NT = T; };
template <class LT>
__device__ __forceinline__ int threads() { return LT::NT != 0 ? LT::NT : int(blockDim.x); }

// Task i of a phase over (field c, element e, mode or node j) in [3][ne][M] order: c, the
// offset r = e M + j within field c's block, e and j.  The products take 24-bit multiplies
// and the division is unsigned by the constant M: 32-bit multiplies issue at a quarter of
// the vector-ALU rate, and these phases run their index arithmetic once per task.
template <int M>
struct FieldTask {
  int c, r, e, j;
  __device__ __forceinline__ FieldTask(int i, int nem) {     // nem = ne * M
    c = (i >= nem) + (i >= 2 * nem);
    r = i - __umul24(unsigned(c), unsigned(nem));
    e = int(unsigned(r) / unsigned(M));
    j = r - __umul24(unsigned(e), unsigned(M));
  }
};

// ---------------------------------------------------------------- matrix-core contractions
// C[M x NC] = A[M x KD] B[KD x NC], A and B read from LDS, on the matrix cores.  One wave
// per 16x16 output block; blocks are dealt to the workgroup's waves.  Lane layout of the
// 16x16xK instructions used: lane l holds A[row l%16][k in k-quad l/16], B[k in k-quad
// l/16][col l%16]; it receives D[row 4(l/16) + r][col l%16], r = 0..3, from the f32 and
// bf16 instructions, but D[row l/16 + 4r][col l%16] from v_mfma_f64_16x16x4_f64.
// Out-of-range rows, columns and k are zero.  Modes:
//   kMfmaNative: v_mfma_f32_16x16x4_f32 or v_mfma_f64_16x16x4_f64 (products and sums in the
//                bulk precision);
//   kMfmaBf16x3: each operand split x = hi + lo (hi = bf16(x), lo = bf16(x - hi)), product
//                hi_a hi_b + hi_a lo_b + lo_a hi_b by v_mfma_f32_16x16x16_bf16 with float
//                accumulation (relative error ~2^-16 per product).
enum ContractionMode : int { kMfmaNative = 1, kMfmaBf16x3 = 2 };

typedef short bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef double f64x4_t __attribute__((ext_vector_type(4)));
template <typename real> struct Acc { typedef f32x4_t type; };
template <> struct Acc<double> { typedef f64x4_t type; };
__device__ __forceinline__ f32x4_t mfma(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f64x4_t mfma(double a, double b, f64x4_t c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// output row of item r of the lanes of k-quad `quad`
template <typename real>
__device__ __forceinline__ int acc_row(int quad, int r) { return sizeof(real) == 4 ? 4 * quad + r : quad + 4 * r; }


__device__ inline unsigned short bf16_rne(float x) {
  unsigned u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);            // round to nearest even (finite inputs)
  return (unsigned short)(u >> 16);
}
__device__ inline float bf16_value(unsigned short h) { return __uint_as_float(unsigned(h) << 16); }

// C[M x ncol] = A[M x KD] B[KD x ncol] in the bulk precision (kMfmaNative): a(row) is a
// pointer to row `row` of A (elements lda reals apart), b(col) a functor giving B[k][col].
// Row and column indices beyond the matrices are clamped (the loads stay inside them, the
// results are dropped), and so is the last k-quad, whose B values beyond KD are zeroed, so
// the loop has no bounds checks: a step is one LDS word of A and of B per 16x16x4 product.
// The steps go to two accumulators in turn, added at the end: half as long a chain of roundings
// and of dependent products.  RMS error of an FP32 right-hand side against 64 bits with one
// accumulator and with two, relative to two partial sums on the vector ALUs (geometric means over
// meshes, options and seeds): N = 1..5 1.008, 1.036, 1.024, 1.074, 1.033 and 0.993, 0.998, 0.964,
// 0.979, 0.912; N+2 points 1.098 and 1.003.  Time: N = 2, K = 65522 39.7 -> 40.0 us a stage, the
// other degrees within 0.4 %.
template <int M, int KD, typename real, class FA, class FB, class FC>
__device__ __forceinline__ void gemm_native(int ncol, int nwaves, FA a, int lda, FB b, FC c_store) {
  typedef typename Acc<real>::type acc_t;
  constexpr int MB = (M + 15) / 16, KS = (KD + 3) / 4, CH = KS > 1 ? 2 : 1;
  const int t = phase_tid(), lane = t & 63, lrow = lane & 15, quad = lane >> 4;
  const int nblk = MB * ((ncol + 15) >> 4);
#pragma unroll 1
  for (int blk = wave_id(); blk < nblk; blk += nwaves) {
    const int bj = int(unsigned(blk) / unsigned(MB)), bi = blk - bj * MB;
    const int row = bi * 16 + lrow, col = bj * 16 + lrow;
    const real *ap = a(M % 16 == 0 || row < M ? row : M - 1);
    const auto bp = b(col < ncol ? col : ncol - 1);
    acc_t acc[CH] = {};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int k = 4 * s + quad;
      const bool in = KD % 4 == 0 || s + 1 < KS || k < KD;
      const int kc = in ? k : KD - 1;
      const real av = ap[kc * lda], bv = bp(kc, s);
      acc[s % CH] = mfma(av, in ? bv : real(0), acc[s % CH]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = bi * 16 + acc_row<real>(quad, r);
      if (i < M && col < ncol) c_store(i, col, CH == 1 ? acc[0][r] : acc[0][r] + acc[CH - 1][r]);
    }
  }
}

// The same with split-bf16 products (kMfmaBf16x3): a(row, k) and b(k, col) return the values.
template <class FA, class FB, class FC>
__device__ __forceinline__ void gemm_bf16x3(int M, int KD, int NC, FA a_at, FB b_at, FC c_store) {
  const int lane = threadIdx.x & 63, wave = wave_id(), nwaves = blockDim.x >> 6;
  const int mb = (M + 15) / 16, nb = (NC + 15) / 16;
  const int lrow = lane & 15, quad = lane >> 4;
#pragma unroll 1
  for (int blk = wave; blk < mb * nb; blk += nwaves) {
    const int bi = blk % mb, bj = blk / mb;
    const int row = bi * 16 + lrow, col = bj * 16 + lrow;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int k0 = 0; k0 < KD; k0 += 16) {
      bf16x4_t ahi, alo, bhi, blo;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = k0 + 4 * quad + r;
        const float av = (row < M && k < KD) ? float(a_at(row, k)) : 0.f;
        const float bv = (col < NC && k < KD) ? float(b_at(k, col)) : 0.f;
        const unsigned short ah = bf16_rne(av), bh = bf16_rne(bv);
        ahi[r] = short(ah);
        alo[r] = short(bf16_rne(av - bf16_value(ah)));
        bhi[r] = short(bh);
        blo[r] = short(bf16_rne(bv - bf16_value(bh)));
      }
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ahi, bhi, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ahi, blo, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(alo, bhi, acc, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = bi * 16 + 4 * quad + r;
      if (i < M && col < NC) c_store(i, col, acc[r]);
    }
  }
}

// c_store(i, col, sum_k V[i][k] in(col)(k)) (TR false: rows of V_h, [.][LD] row-major) or, with
// TR, sum_k V[k][i] in(col)(k), for M rows and ncol columns.
template <int CM, int M, int KD, int LD, bool TR, typename real, class FB, class FC>
__device__ __forceinline__ void contract(const real *V, int ncol, int nwaves, FB in, FC c_store) {
  if constexpr (CM == kMfmaBf16x3)
    gemm_bf16x3(M, KD, ncol, [&](int i, int k) { return TR ? V[k * LD + i] : V[i * LD + k]; },
                [&](int k, int c) { return in(c)(k, k >> 2); }, c_store);
  else
    gemm_native<M, KD, real>(ncol, nwaves, [&](int row) { return V + (TR ? row : __umul24(unsigned(row), unsigned(LD))); },
                             TR ? LD : 1, in, c_store);
}

// Columns of an array [ncol][M], as contract's input and output.
template <int M, typename real>
__device__ __forceinline__ auto cols_in(const real *x) {
  return [x](int c) {
    const real *p = x + __umul24(unsigned(c), unsigned(M));
    return [p](int k, int) { return p[k]; };
  };
}
template <int M, typename real>
__device__ __forceinline__ auto cols_out(real *x) {
  return [x](int i, int c, real v) { x[__umul24(unsigned(c), unsigned(M)) + i] = v; };
}

// LDS carve-up of one tile (see tile_words()).
template <typename real, int N, int EC, int NTH>
struct Lds {
  static constexpr int NT = NTH;
  static constexpr int Np = dim_Np(N), Nq = dim_Nq(N), Nfq = dim_Nfq(N), Nh = dim_Nh(N);
  real *ref, *Vh, *ST, *FT, *wf, *nr, *ns;
  real *q0, *q1, *dH, *p, *raw, *nb, *U, *DU, *Minv, *wJ, *bq, *bh;
  real *R, *T, *Q, *VH;
  int32_t *pp;
  int E;                           // elements of a full tile: the stride of every array below
  // sm: the ref block (already loaded); tile: the tile region (after the largest ref block);
  // mw: reals of mass data per element (mass_words).
  // EC: E where the kernel is built for one tile size, so that every offset is an immediate;
  // 0: E is e.
  __device__ Lds(real *sm, real *tile, int e, int mw) : E(EC != 0 ? EC : e) {
    ref = sm;
    Vh = ref;
    ST = Vh + Nh * Np;
    FT = ST + 2 * Nh * Nq;
    wf = FT + 2 * Nq * Nfq;
    nr = wf + Nfq;
    ns = nr + Nfq;
    q0 = tile;                   // node records (see kNodeQuads)
    q1 = q0 + 4 * E * Nh;
    raw = q1 + 4 * E * Nh;
    nb = raw + ((E * raw_words(N) + 3) & ~3);
    Minv = nb + 4 * E * Nfq;     // the static block; every region up to here is 16-byte aligned
    wJ = Minv + E * mw;          // Minv: [E][Np][Np], or w/J [E][Nq] (weight-adjusted)
    bq = wJ + E * Nq;
    bh = bq + E * Nq;
    pp = reinterpret_cast<int32_t *>(bh + E * Nh);
    U = bh + E * (Nh + Nfq);
    DU = U + 3 * E * Np;
    dH = DU + 3 * E * Np;
    p = dH + E * Nh;
    // reuse: the residual, lift and projection temporaries live in the raw block (dead
    // after phase 1) and v'_h in the neighbour block (dead after the residual); the
    // node records and the state are left alone, so a resident tile keeps them
    R = raw;                      // the two parts of the residual [2][3][E][Nh]
    T = raw + 6 * E * Nh;         // [3][E][Np]
    Q = raw;                      // [3][E][Nq] projection's weighted entropy variables
    VH = nb;                      // [3][E][Np] v'_h (3 Np <= 4 Nfq for N <= 5)
  }
};

// Rows per thread of the residual phase: two in float where two rows' sums fit the registers
// and 2 divides Nq and Nfq.
template <typename real, int N> struct RowsPerThread { static constexpr int value = 1; };
template <> struct RowsPerThread<float, 1> { static constexpr int value = 2; };
template <> struct RowsPerThread<float, 3> { static constexpr int value = 2; };
template <> struct RowsPerThread<float, make_key(1, 2)> { static constexpr int value = 2; };   // DG-SBP: 6 + 6 nodes
template <> struct RowsPerThread<float, make_key(3, 2)> { static constexpr int value = 2; };   // 18 + 12
// The tile size a kind's kernel is built for (0: none), so that every LDS offset is an
// immediate: the size that is fastest for large meshes (FP32 N = 2, K = 65522: 43.7 us a stage
// at 14 so, 50.6 at 12 with run-time offsets).
template <typename real> __host__ __device__ constexpr int fixed_tile(int kind) {
  const bool f = sizeof(real) == 4;
  switch (kind) {
    case 1: return f ? 32 : 16;
    case 2: return f ? 14 : 7;
    case 3: return f ? 8 : 4;
    case 4: return 5;
    case 5: return 7;
    case make_key(1, 2): return f ? 16 : 8;
    case make_key(2, 2): return f ? 13 : 8;
    case make_key(3, 2): case make_key(4, 2): return f ? 8 : 4;
    default: return 0;
  }
}

// A second one: what small meshes (one tile for each of 1024 workgroups) or launches of
// several degrees, whose largest tile sets the LDS of all, take instead.  Per stage without and
// with: FP32 N = 1, K = 8192 4.87 -> 4.35 us, FP64 N = 2, K = 8192 8.47 -> 7.92, K = 1800 6.08 ->
// 5.53.
template <typename real> __host__ __device__ constexpr int other_tile(int kind) {
  const bool f = sizeof(real) == 4;
  return kind == 1 ? (f ? 16 : 12) : kind == 2 ? (f ? 12 : 8) : 0;
}
// EC of the kernel for several kinds whose tiles have those sizes (an ensemble of 45944
// elements, N = 2..4, FP32: 72.8 us a stage with run-time offsets, 66.2 with these).
constexpr int kFixedTiles = -1;

// What changes from stage to stage of a launch.
struct StageRun {
  int mode, in_buf, out_buf;
  double rk_a, rk_b;
};

// Weight-adjusted inverse of the curved mass matrix (the implementation remark after eq.
// (dgform) in Section 2.8): (M_h^k)^{-1} y ~ M^{-1} M_{1/J} M^{-1} y with M_{1/J} =
// V_q^T W diag(1/J) V_q; the reference mass matrix M is the identity for the orthonormal
// basis with the degree-2N volume rule, so this is V_q^T diag(w/J) V_q y, two contractions
// with V_q (the first Nq rows of V_h) and the per-element weights w/J (held where the
// stored inverse would be).  First factor, one task per (field, element, volume node):
// S[c][e][q] = (w/J)[e][q] sum_j V_q[q][j] Y[c][e][j].
template <typename real, int N, class LT>
__device__ __forceinline__ void wadg_first(const LT &L, const real *Y, real *S) {
  constexpr int Np = dim_Np(N), Nq = dim_Nq(N);
  const int E = L.E;
  contract<kMfmaNative, Nq, Np, Np, false, real>(L.Vh, 3 * E, threads<LT>() >> 6, cols_in<Np>(Y), [&](int q, int c, real v) {
    const int e = c - ((c >= E) + (c >= 2 * E)) * E;
    S[__umul24(unsigned(c), unsigned(Nq)) + q] = L.Minv[__umul24(unsigned(e), unsigned(Nq)) + q] * v;
  });
}

// Second factor: out[c][e][j] = sum_q V_q[q][j] S[c][e][q].
template <typename real, int N, class LT>
__device__ __forceinline__ void wadg_second(const LT &L, const real *S, real *out) {
  constexpr int Np = dim_Np(N), Nq = dim_Nq(N);
  contract<kMfmaNative, Np, Nq, Np, true, real>(L.Vh, 3 * L.E, threads<LT>() >> 6, cols_in<Nq, real>(S), cols_out<Np>(out));
}

// Node record i = e Nh + n (its metric quad q1 is copied there as it lies in HBM).
template <typename real, class LT>
__device__ __forceinline__ void write_record(const LT &L, int i, real h, real u, real v, real dH, real g) {
  typedef real real4 __attribute__((ext_vector_type(4)));
  reinterpret_cast<real4 *>(L.q0)[i] = real4{real(0.5) * h * u, real(0.5) * h * v, real(0.5) * u, real(0.5) * v};
  L.dH[i] = dH;
  L.p[i] = real(0.5) * g * h;
}

// The stored inverses applied to X [3][E][Np]: store(i, (Minv_e X[c][e])[j]), i = (c E + e) Np + j,
// one task per output, on the vector ALUs (the matrix differs from element to element).
template <typename real, int N, class LT, class F>
__device__ __forceinline__ void minv_rows(const LT &L, const real *X, F store) {
  constexpr int Np = dim_Np(N);
  const int nem = L.E * Np;
  for (int i = phase_tid(); i < 3 * nem; i += threads<LT>()) {
    const FieldTask<Np> k(i, nem);
    const real *Mi = L.Minv + __umul24(unsigned(k.r), unsigned(Np));   // row (e, j) of Minv_e
    const real *Xc = X + (i - k.j);                                    // X[c][e][0..Np)
    real a = 0, b = 0;
#pragma unroll 32
    for (int j = 0; j + 1 < Np; j += 2) {
      a += Mi[j] * Xc[j];
      b += Mi[j + 1] * Xc[j + 1];
    }
    if (Np & 1) a += Mi[Np - 1] * Xc[Np - 1];
    store(i, a + b);
  }
}

// Entropy projection of the tile states in L.U ([3][ne][Np]: eta, hu, hv) to the
// hybridized nodes (Section 2.6), written to out (tile-blocked [4][ne][Nh]: h~, u~, v~,
// H~ - Href) or, in a resident stage that is not the last, straight into the node records
// of the next stage (the same values the records phase would form from out):
//   q = V_q u_h; h = eta_q + (Href - b_q); v' = (g eta_q - |u|^2/2, u, v) = v(u_q) - (g Href, 0, 0)
//   (FP64); v'_h = Minv_k V_q^T diag(w J) v'_q (Minv_k the stored inverse, or the
//   weight-adjusted one); v~' = V_h v'_h;
//   H~ - Href = (v~1' + |v~23|^2/2)/g, h~ = (H~ - Href) + (Href - b~) (FP64).
// Subtracting the constant g Href is exact: the projection reproduces constants.  The rest
// depth Href - b comes from the static block, formed in double on the device from b (so in
// float it has the relative accuracy of the depth itself where the water is shallow).
template <typename real, int N, int CM, bool WADG, class LT>
__device__ __forceinline__ void project_tile(const InstDesc &d, int k0, int ne, LT &L, real *out,
                                             real *nbx_out, int32_t *flag, bool coherent, bool to_records = false) {
  constexpr int Np = dim_Np(N), Nq = dim_Nq(N), Nh = dim_Nh(N), Nfq = dim_Nfq(N);
  const double g = d.g;
  const int tid = phase_tid(), nth = threads<LT>();
  const int E = L.E, nc = 3 * E;               // contraction columns: (field, element)
  real *Stage = L.R;                           // [3][E][Nq] or [3][E][Nh] staging (free here)
  bool bad = false;
  contract<CM, Nq, Np, Np, false, real>(L.Vh, nc, nth >> 6, cols_in<Np, real>(L.U), cols_out<Nq>(Stage));   // u_q = V_q u_h
  __syncthreads();
  for (int i = tid; i < ne * Nq; i += nth) {
    const double eta = Stage[i], hu = Stage[E * Nq + i], hv = Stage[2 * E * Nq + i];
    const double h = eta + double(L.bq[i]);       // L.bq: rest depth Href - b
    const double rh = 1.0 / h, uu = hu * rh, vv = hv * rh;
    const double v1 = g * eta - 0.5 * (uu * uu + vv * vv);
    const double w = L.wJ[i];
    L.Q[i] = real(w * v1);
    L.Q[E * Nq + i] = real(w * uu);
    L.Q[2 * E * Nq + i] = real(w * vv);
    bad |= bad_value(h, hu, hv);
  }
  __syncthreads();
  contract<CM, Np, Nq, Np, true, real>(L.Vh, nc, nth >> 6, cols_in<Nq, real>(L.Q), cols_out<Np>(L.T));      // y = V_q^T (w J v')
  __syncthreads();
  // v'_h = Minv_k y (weight-adjusted: the first factor into L.Q, dead once y is formed)
  if constexpr (WADG) {
    wadg_first<real, N>(L, L.T, L.Q);
    __syncthreads();
    wadg_second<real, N>(L, L.Q, L.VH);
  } else {
    minv_rows<real, N>(L, L.T, [&](int i, real v) { L.VH[i] = v; });
  }
  __syncthreads();
  contract<CM, Nh, Np, Np, false, real>(L.Vh, nc, nth >> 6, cols_in<Np, real>(L.VH), cols_out<Nh>(Stage));  // v~ = V_h v_h
  __syncthreads();
  for (int i = tid; i < ne * Nh; i += nth) {
    const int e = int(unsigned(i) / unsigned(Nh)), n = i - __umul24(unsigned(e), unsigned(Nh));
    const double v1 = Stage[i], v2 = Stage[E * Nh + i], v3 = Stage[2 * E * Nh + i];
    const double dH = (v1 + 0.5 * (v2 * v2 + v3 * v3)) / g;
    const double h = dH + double(L.bh[i]);        // L.bh: rest depth Href - b
    if (to_records) {
      write_record<real>(L, i, real(h), real(v2), real(v3), real(dH), real(d.g));
    } else {
      real *ot = out + size_t(k0) * 4 * Nh + unsigned(i);   // tile-blocked [4][E][Nh]
      ot[0] = real(h);
      ot[E * Nh] = real(v2);
      ot[2 * E * Nh] = real(v3);
      ot[3 * E * Nh] = real(dH);
    }
    if (n >= Nq) {                 // face node: also fill the neighbour's face slot
      const int f = n - Nq;
      const uint32_t tgt = uint32_t(L.pp[__umul24(unsigned(e), unsigned(Nfq)) + f]);
      real *slot = nbx_out + size_t(tgt & ~kPushWall) * 4;
      double pu = v2, pv = v3;     // the velocity the exterior side of the face sees
      if (tgt & kPushWall) {
        // reflective wall (Section 2.9): the exterior state is this node's own with the
        // normal velocity reversed, u+ = u - 2 (u . nJ) nJ / |nJ|^2, h+ = h (so H+ = H),
        // written into this node's own slot; nJ from the metric factors (tile-blocked, as
        // fetched) and the reference normal of the face
        const real *gm = static_cast<const real *>(d.geo) + (size_t(k0) * Nh + unsigned(i)) * 4;
        const double nr = double(L.nr[f]), ns = double(L.ns[f]);
        const double nx = double(gm[0]) * nr + double(gm[1]) * ns;
        const double ny = double(gm[2]) * nr + double(gm[3]) * ns;
        const double c = 2.0 * (v2 * nx + v3 * ny) / (nx * nx + ny * ny);
        pu = v2 - c * nx;
        pv = v3 - c * ny;
      }
      if (coherent) {
        // multi-stage launches: device-coherent (sc1) 16-byte vector stores, since the
        // neighbour's workgroup may sit on another XCD, whose L2 does not see this one's.
        // The slot is 16-byte aligned; publish() waits for these stores (vmcnt) itself.
        // A vector store of more than 8 bytes reads its data registers after issue: a VALU
        // write to them must wait two cycles.  The compiler inserts that wait only for stores
        // it generates, not for these, so each statement carries its own s_nop (without it
        // the FP64 pair below had its first store's data overwritten by the second's address).
        if constexpr (sizeof(real) == 4) {
          typedef float f4 __attribute__((ext_vector_type(4)));
          const f4 val = {float(h), float(pu), float(pv), float(dH)};
          asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(slot), "v"(val) : "memory");
        } else {
          typedef double d2 __attribute__((ext_vector_type(2)));
          const d2 lo = {h, pu}, hi = {pv, dH};
          asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(slot), "v"(lo) : "memory");
          asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(slot + 2), "v"(hi) : "memory");
        }
      } else {
        typedef real real4 __attribute__((ext_vector_type(4)));
        const real4 val = {real(h), real(pu), real(pv), real(dH)};
        *reinterpret_cast<real4 *>(slot) = val;
      }
    }
    bad |= bad_value(h, v2, v3);
  }
  if (bad) atomicOr(flag, 1);
}

// Asynchronous global -> LDS copies (global_load_lds): every lane moves 16 bytes (or one
// word) from its own address straight into LDS at (wave-uniform base) + 16 (or 4) * lane,
// without staging in registers.  They are issued from asm statements, which the compiler's
// wait counting does not see, so nothing waits for them until wait_copies: the waits the
// compiler inserts for its own loads can only come out longer.
__device__ __forceinline__ uint32_t lds_byte(const void *p) {
  return uint32_t(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const void *)p));
}
template <bool COHERENT>
__device__ __forceinline__ void copy16(uint32_t lds, const void *src) {
  if constexpr (COHERENT)          // device-coherent: other XCDs' stores are visible
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off sc1" ::"s"(__builtin_amdgcn_readfirstlane(lds)), "v"(src) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(__builtin_amdgcn_readfirstlane(lds)), "v"(src) : "memory", "m0");
}
__device__ __forceinline__ void copy4(uint32_t lds, const void *src) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(__builtin_amdgcn_readfirstlane(lds)), "v"(src) : "memory", "m0");
}
// This wave's copies have landed in LDS.
__device__ __forceinline__ void wait_copies() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Copies `bytes` contiguous bytes (at most MAX where that is not 0, so that the rounds unroll)
// between 16-byte aligned places; a tail of single words where bytes is not a multiple of 16.
template <class LT, int MAX, bool COHERENT = false>
__device__ __forceinline__ void copy_block(void *dst, const void *src, int bytes) {
  const int nth = threads<LT>(), t = phase_tid(), lane16 = t * 16;
  const uint32_t lds = lds_byte(dst) + (wave_id() << 10);
  const char *p = static_cast<const char *>(src) + lane16;
  if constexpr (MAX != 0 && LT::NT != 0) {
#pragma unroll
    for (int o = 0; o < MAX; o += LT::NT * 16)
      if (o + lane16 + 16 <= bytes) copy16<COHERENT>(lds + o, p + o);
  } else {
    for (int o = 0; o < bytes; o += nth * 16)
      if (o + lane16 + 16 <= bytes) copy16<COHERENT>(lds + o, p + o);
  }
  if (MAX == 0 || MAX % 16 != 0) {
    const int tail = bytes & ~15;
    if (tail + 4 * t < bytes) copy4(lds_byte(dst) + tail, static_cast<const char *>(src) + tail + 4 * t);
  }
}

// Copies the tile's part of a state array [3][K][M] to [3][E][M] in LDS, one word per lane (its
// planes have no alignment beyond a value's).
template <class LT, int M, int EC, typename real>
__device__ __forceinline__ void copy_state(real *dst, const void *src, size_t splane, int k0, int ne, int E) {
  constexpr int W = sizeof(real) / 4;
  const int nth = threads<LT>(), plane = E * M * W, live = ne * M * W, t = phase_tid();
  const uint32_t lds = lds_byte(dst) + (wave_id() << 8);
  const uint32_t *s0 = static_cast<const uint32_t *>(src) + size_t(k0) * M * W;
  auto round = [&](int o) {
    const int i = o + t, c = (i >= plane) + (i >= 2 * plane), w = i - (c == 0 ? 0 : c == 1 ? plane : 2 * plane);
    if (c < 3 && w < live) copy4(lds + 4 * o, s0 + (c == 0 ? 0 : c == 1 ? splane * W : 2 * splane * W) + w);
  };
  if constexpr (EC != 0 && LT::NT != 0) {
#pragma unroll
    for (int o = 0; o < 3 * EC * M * W; o += LT::NT) round(o);
  } else {
    for (int o = 0; o < 3 * plane; o += nth) round(o);
  }
}

// Phase 0: fetch the tile's global data into LDS (all asynchronous; see above).  `index`: the
// tile's number within its instance.
template <typename real, int N, bool WADG, bool MULTI, int EC, class LT>
__device__ __forceinline__ void fetch_tile(const StageArgs &a, const StageRun &r, const InstDesc &d, int index, int k0,
                                           int ne, LT &L) {
  constexpr int Np = dim_Np(N), Nfq = dim_Nfq(N), Nh = dim_Nh(N), SW = stat_words(N, WADG), B = int(sizeof(real));
  const int E = L.E;
  const size_t splane = size_t(d.K) * Np;
  // the multi-stage build runs RK stages only, on the instance buffers (see stage_tile)
  const int mode = MULTI ? int(kStage) : r.mode;
  const void *ext_ut = MULTI ? nullptr : a.ext_ut, *ext_state = MULTI ? nullptr : a.ext_state;
  const void *ext_nbx = MULTI ? nullptr : a.ext_nbx;
  if (mode != kProject) {
    // u~ and the metric quads are stored tile-blocked ([4][E][Nh] and [E][Nh][4] per tile)
    const size_t base = size_t(k0) * 4 * Nh;
    const void *ut = ext_ut ? ext_ut : d.ut[r.in_buf];
    copy_block<LT, 4 * EC * Nh * B>(L.raw, static_cast<const real *>(ut) + base, 4 * E * Nh * B);
    copy_block<LT, 4 * EC * Nh * B>(L.q1, static_cast<const real *>(d.geo) + base, 4 * E * Nh * B);
    // neighbour values, pushed here by the neighbours' projections (in a multi-stage launch
    // during this kernel, maybe on another XCD)
    const real *nbx = static_cast<const real *>(ext_nbx ? ext_nbx : d.nbx[r.in_buf]) + size_t(k0) * Nfq * 4;
    copy_block<LT, EC * Nfq * 4 * B, MULTI>(L.nb, nbx, ne * Nfq * 4 * B);
  }
  if (mode != kRhs)
    copy_state<LT, Np, EC>(L.U, mode == kProject && ext_state ? ext_state : d.uh, splane, k0, ne, E);
  if (mode == kStage) copy_state<LT, Np, EC>(L.DU, d.du, splane, k0, ne, E);
  // static block (mass data, w J, rest depth, push targets): contiguous in HBM and in LDS
  copy_block<LT, EC * SW * B>(L.Minv, static_cast<const real *>(d.stat) + size_t(index) * stat_tile(N, E, WADG),
                              E * SW * B);
  wait_copies();
}

// Interface terms of a face node (Section 2.8) from its node record i and the neighbour's
// values nbp (h, u, v, H - Href): W_f [ nJ . f_S(u~, u~+) + 1/2 g h (H+ - Href) nJ ] minus,
// for the LF flux, the penalty 1/2 lambda sJ (u~+ - u~).
template <typename real, class LT>
__device__ __forceinline__ void interface_terms(const LT &L, int i, const real *nbp, real wf, real nrf, real nsf, real g,
                                                int flux, real &t0, real &t1, real &t2) {
  typedef real real4 __attribute__((ext_vector_type(4)));
  const real4 s0 = reinterpret_cast<const real4 *>(L.q0)[i], s1 = reinterpret_cast<const real4 *>(L.q1)[i];
  const real gh = L.p[i], dH = L.dH[i];          // gh/2, H - Href
  const real nJx = s1.x * nrf + s1.y * nsf, nJy = s1.z * nrf + s1.w * nsf;
  const real uu = real(2) * s0.z, vv = real(2) * s0.w, huu = real(2) * s0.x, hvv = real(2) * s0.y;
  const real hP = nbp[0], uP = nbp[1], vP = nbp[2], dHP = nbp[3];
  const real huP = hP * uP, hvP = hP * vP;
  const real hua = real(0.5) * (huu + huP), hva = real(0.5) * (hvv + hvP);
  const real ua = real(0.5) * (uu + uP), va = real(0.5) * (vv + vP);
  const real pr = gh * dHP;
  real f0v = nJx * hua + nJy * hva;
  real f1v = nJx * (hua * ua + pr) + nJy * hva * ua;
  real f2v = nJx * hua * va + nJy * (hva * va + pr);
  if (flux == 1) {
    const real sJ = sqrt(nJx * nJx + nJy * nJy);
    const real lm = fabs(uu * nJx + vv * nJy) + sqrt(real(2) * gh) * sJ;
    const real lp = fabs(uP * nJx + vP * nJy) + sqrt(g * hP) * sJ;
    const real c = real(0.5) * fmax(lm, lp);
    f0v -= c * (dHP - dH);
    f1v -= c * (huP - huu);
    f2v -= c * (hvP - hvv);
  }
  t0 = wf * f0v;
  t1 = wf * f1v;
  t2 = wf * f2v;
}

// Residual rows (Section 2.8, flux differencing plus interface terms).  Row m accumulates,
// over its columns n, c = Qx {hu} + Qy {hv} (a0), u_n c and v_n c (b1, b2), and dH_n Qx,
// dH_n Qy (d1, d2); the row factors are applied once at the end:
//   sum_n ({u} c + gh_m dH_n Qx) = u_m a0 + b1 + gh_m d1   (halves folded into the records)
// Volume rows run over all Nh columns (the diagonal of the skew operator is zero), face rows
// over the Nq volume columns (the surface-surface block is zero).  This function is one
// task: rows m0 .. m0+R-1 of element e, over T columns from n_lo on (one more with `more`),
// with the operator table Stab (already offset to the first of these rows of its row set)
// whose consecutive columns are LD2 reals apart; the sums go to part p of the residual block.
// The trip count is a constant so that the loads of several columns are in flight at once.
template <typename real, int N, int R, int T, int LD2, class LT>
__device__ __forceinline__ void row_sums(int e, int m0, int p, int n_lo, bool more, const real *Stab, LT &L) {
  constexpr int Nh = dim_Nh(N), UN = T <= 16 ? T : T % 9 == 0 ? 9 : T % 10 == 0 ? 10 : 8;
  typedef real real4 __attribute__((ext_vector_type(4)));
  const int i0 = __umul24(unsigned(e), unsigned(Nh));    // the element's first node
  const real4 *q0 = reinterpret_cast<const real4 *>(L.q0) + i0, *q1 = reinterpret_cast<const real4 *>(L.q1) + i0;
  const real *dH = L.dH + i0;
  real hu[R], hv[R], u[R], v[R], gh[R], rx[R], sx[R], ry[R], sy[R], a0[R], a1[R], a2[R];
  real b1[R], b2[R], d1[R], d2[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const real4 s0 = q0[m0 + r], s1 = q1[m0 + r];
    hu[r] = s0.x; hv[r] = s0.y; u[r] = s0.z; v[r] = s0.w;
    rx[r] = s1.x; sx[r] = s1.y; ry[r] = s1.z; sy[r] = s1.w;
    gh[r] = L.p[i0 + m0 + r];
    a0[r] = 0; b1[r] = 0; b2[r] = 0; d1[r] = 0; d2[r] = 0;
  }
  const real *Scol = Stab + __umul24(unsigned(n_lo), unsigned(LD2));
  const real4 *p0 = q0 + n_lo, *p1 = q1 + n_lo;
  const real *pd = dH + n_lo;
  auto column = [&](int j) {
    const real4 c0 = p0[j], c1 = p1[j];
    const real hun = c0.x, hvn = c0.y, un = c0.z, vn = c0.w, dHn = pd[j];
    const real *S = Scol + j * LD2;
    const real rxn = c1.x, sxn = c1.y, ryn = c1.z, syn = c1.w;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const real Sr = S[2 * r], Ss = S[2 * r + 1];
      const real Qx = (rx[r] + rxn) * Sr + (sx[r] + sxn) * Ss;
      const real Qy = (ry[r] + ryn) * Sr + (sy[r] + syn) * Ss;
      const real c = Qx * (hu[r] + hun) + Qy * (hv[r] + hvn);
      a0[r] += c;
      b1[r] += un * c;
      b2[r] += vn * c;
      d1[r] += dHn * Qx;
      d2[r] += dHn * Qy;
    }
  };
#pragma unroll UN
  for (int j = 0; j < T; ++j) column(j);
  if (more) column(T);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    a1[r] = u[r] * a0[r] + b1[r] + gh[r] * d1[r];
    a2[r] = v[r] * a0[r] + b2[r] + gh[r] * d2[r];
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int m = m0 + r;
    real *Rp = L.R + __umul24(unsigned(p), unsigned(3 * L.E * Nh)) + i0 + m;
    Rp[0] = a0[r];
    Rp[L.E * Nh] = a1[r];
    Rp[2 * L.E * Nh] = a2[r];
  }
}

// The tasks of the residual rows; every row's columns are summed in two parts.
//
// Kinds with few hybrid nodes cut volume rows (Nh columns) and face rows (Nq columns) into
// halves, R rows to a task, volume tasks first and the half slowest: a wave then runs one
// column range (the node records of its columns are read by several elements at once, the
// operator table's rows by consecutive row blocks).
//
// The wide kinds (N=5, and N+2 points at N=4 and 5) have more rows than threads at that cut.
// There the first tasks (padded to whole waves) take the Nq volume columns of a volume row,
// and the second ones its Nfq face columns and then half a face row (Nq >= 2 Nfq), so that
// all run about Nq columns: at N=5 and seven elements per workgroup 504 of 512 threads run
// 36 columns each, against 378 threads running 54 or 36.
template <typename real, int N, int R, class LT>
__device__ __forceinline__ void residual_tile(int ne, LT &L) {
  constexpr int Nq = dim_Nq(N), Nfq = dim_Nfq(N), Nh = dim_Nh(N);
  constexpr int VB = Nq / R, FB = Nfq / R;
  static_assert(Nq % R == 0 && Nfq % R == 0, "R must divide Nq and Nfq");
  const int tid = phase_tid(), nth = threads<LT>();
  if constexpr (wide_kind(N)) {
    static_assert(R == 1 && Nq >= 2 * Nfq, "a second task takes one half of a face row");
    const int rows = ne * Nq, second = (rows + 63) & ~63;
    for (int t = tid; t < second + rows; t += nth) {
      const bool b = t >= second;
      const int i = b ? t - second : t, e = int(unsigned(i) / unsigned(Nq)), m = i - __umul24(unsigned(e), unsigned(Nq));
      if (!b) {
        if (i < rows) row_sums<real, N, 1, Nq, 2 * Nq>(e, m, 0, 0, false, L.ST + 2 * m, L);
      } else {
        row_sums<real, N, 1, Nfq, 2 * Nq>(e, m, 1, Nq, false, L.ST + 2 * m, L);
        const int f = m >> 1, h = m & 1;
        if (m < 2 * Nfq)
          row_sums<real, N, 1, Nq / 2, 2 * Nfq>(e, Nq + f, h, h * (Nq / 2), Nq % 2 != 0 && h != 0, L.FT + 2 * f, L);
      }
    }
  } else {
    // task t = (half ne + e) rows + b, split in unsigned arithmetic by constants (see FieldTask)
    auto split = [&](int t, unsigned rows, int &p, int &e, int &b) {
      const int per = ne * rows;
      p = t >= per;
      const unsigned rest = unsigned(p ? t - per : t);
      e = int(rest / rows);
      b = int(rest) - __umul24(unsigned(e), rows);
    };
    // the face tasks start on a wave of their own where that adds no round: a wave with tasks of
    // both sorts runs both loops (DG-SBP N = 4, K = 32768 49.6 -> 47.3 us a stage, FP64 N = 4,
    // K = 20402 98.3 -> 95)
    const int nv = 2 * ne * VB, nf = 2 * ne * FB, whole = (nv + 63) & ~63;
    const int nv1 = (whole + nf + nth - 1) / nth > (nv + nf + nth - 1) / nth ? nv : whole;
    for (int t = tid; t < nv1 + nf; t += nth) {
      int p, e, b;
      if (t < nv1) {
        split(t, VB, p, e, b);
        if (t < nv)
          row_sums<real, N, R, Nh / 2, 2 * Nq>(e, b * R, p, p * (Nh / 2), Nh % 2 != 0 && p != 0, L.ST + 2 * b * R, L);
      } else {
        split(t - nv1, FB, p, e, b);
        row_sums<real, N, R, Nq / 2, 2 * Nfq>(e, Nq + b * R, p, p * (Nq / 2), Nq % 2 != 0 && p != 0, L.FT + 2 * b * R, L);
      }
    }
  }
}

// Residual r_h of column c = (field, element) at hybrid node k: its two parts and, on the face
// rows, the interface terms, which are added to the first part (FIRST), or to the sum of both: for
// the split-bf16 products, whose own error hides the difference, that is the faster order (N = 5,
// K = 131072 608 us a stage, 620 the other way).
template <typename real, int D, bool FIRST, class LT>
__device__ __forceinline__ auto residual_in(const LT &L) {
  constexpr int Nq = dim_Nq(D), Nfq = dim_Nfq(D), Nh = dim_Nh(D);
  const int E = L.E;
  const real *R = L.R, *nb = L.nb;
  return [=](int c) {
    const int f = (c >= E) + (c >= 2 * E), e = c - f * E;
    const real *p0 = R + __umul24(unsigned(c), unsigned(Nh)), *p1 = p0 + 3 * E * Nh;
    const real *pf = nb + __umul24(unsigned(e), unsigned(4 * Nfq)) + f;
    return [=](int k, int s) {     // s = k / 4, which settles most of the tests at compile time
      real v = FIRST ? p0[k] : p0[k] + p1[k];
      if (4 * s + 3 >= Nq) {
        const bool face = 4 * s >= Nq || k >= Nq;
        const real x = pf[face ? 4 * (k - Nq) : 0];
        v += face ? x : real(0);
      }
      return FIRST ? v + p1[k] : v;
    };
  };
}

// Descriptors, tiles and tile ranges are written by the host before a launch and only
// read by kernels.  Reading them through the constant address space lets the compiler use
// scalar loads (lgkmcnt); as vector loads they would share vmcnt with the asynchronous
// LDS copies, and every descriptor field needed between two copies would wait for all
// copies issued before it.
template <typename T>
__device__ __forceinline__ const T &read_const(const T *p, int i) {
  return *(const T *)((const __attribute__((address_space(4))) T *)p + i);
}

// Multi-stage launches: before stage `target` of tile t, wait until every tile holding a
// face neighbour of t has published `target` completed stages (their projection has pushed
// t's neighbour values, and they have finished reading the slots t is about to fill).
// Wave 0 polls, one neighbour per lane, with device-coherent loads and a bounded spin; the
// barrier then releases the other waves.  The neighbour values themselves are read with
// device-coherent copies (fetch_tile), so no cache-wide invalidation is needed.  Returns
// false (for the whole workgroup) if a wait gave up.
__device__ __forceinline__ bool wait_neighbours(const StageArgs &a, int t, int target) {
  int ok = 1;
  if (threadIdx.x < 64) {
    const int b = read_const(a.nbr_off, t), e = read_const(a.nbr_off, t + 1);
    for (int j = b + int(threadIdx.x); j < e; j += 64) {
      const int u = read_const(a.nbr_idx, j);
      int spins = 0;
      while (__hip_atomic_load(a.progress + progress_word(u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
        if (++spins > a.spin_limit) { ok = 0; break; }
        __builtin_amdgcn_s_sleep(1);
      }
    }
  }
  return __syncthreads_and(ok) != 0;
}

// The same wait for a resident tile, by every wave that calls it and for that wave alone: false,
// with flag bit 1 set, once a wait has given up (`waits` false: do not wait).
__device__ __forceinline__ bool poll_neighbours(const StageArgs &a, int t, int target, bool waits) {
  bool ok = waits;
  if (waits) {
    const int b = read_const(a.nbr_off, t), e = read_const(a.nbr_off, t + 1);
    for (int j = b + (int(threadIdx.x) & 63); j < e; j += 64) {
      const int u = read_const(a.nbr_idx, j);
      int spins = 0;
      while (__hip_atomic_load(a.progress + progress_word(u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
        if (++spins > a.spin_limit) { ok = false; break; }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    if (!ok) atomicOr(a.flag, 2);
    ok = __all(ok);
  }
  return ok;
}

// After a stage of tile t: every wave waits until its stores have completed (the pushed
// face values are device-coherent stores, so completion means visible to every XCD), then
// one thread publishes the tile's completed-stage count.  The tile's other outputs are read
// back only by this workgroup.
__device__ __forceinline__ void publish(const StageArgs &a, int t, int value) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(a.progress + progress_word(t), value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Four values through device-coherent 16-byte loads (the workgroup that stored them may sit on
// another XCD); each asm block waits for what it loads.
__device__ __forceinline__ void load_coherent(const float *p, float *v) {
  f32x4_t x;
  asm volatile("global_load_dwordx4 %0, %1, off sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(x) : "v"(p) : "memory");
  v[0] = x[0]; v[1] = x[1]; v[2] = x[2]; v[3] = x[3];
}
__device__ __forceinline__ void load_coherent(const double *p, double *v) {
  typedef double f64x2_t __attribute__((ext_vector_type(2)));
  f64x2_t x, y;
  asm volatile("global_load_dwordx4 %0, %2, off sc1\n\tglobal_load_dwordx4 %1, %2, off offset:16 sc1\n\ts_waitcnt vmcnt(0)"
               : "=&v"(x), "=&v"(y) : "v"(p) : "memory");
  v[0] = x[0]; v[1] = x[1]; v[2] = y[0]; v[3] = y[1];
}

// Neighbour values as fetch_tile left them in LDS.
template <typename real, class LT>
__device__ __forceinline__ auto fetched_neighbours(const LT &L) {
  const real *nb = L.nb;
  return [nb](int i, real *v) {
    typedef real real4 __attribute__((ext_vector_type(4)));
    const real4 x = reinterpret_cast<const real4 *>(nb)[i];
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
  };
}

// First of the interface tasks of this thread: in the modal kinds from the last wave on, since
// the pair loop gives its longer tasks (volume rows) to the first waves (FP32 N = 3, K = 20402
// 29.5 -> 28.8 us a stage, N = 1, K = 65522 23.4 -> 22.9).  FP64 N = 3, one launch per stage, pays
// (K = 8192 20.65 -> 21.2); without the reversal there it stays at 21.2, and the other FP64 kinds
// lose.  The wide kinds' last waves have the longer ones, and in DG-SBP at N = 3 the third wave has both sorts (K = 32768 34.3 us; 35.8
// from the last wave on).
template <int N, class LT>
__device__ __forceinline__ int interface_tid() {
  return wide_kind(N) || key_sbp(N) ? phase_tid() : phase_tid() ^ (threads<LT>() - 64);
}

// Phase 3: interface terms of the face rows (Section 2.8): W_f [ nJ . f_S(u~, u~+) + 1/2 g h
// (H+ - Href) nJ ] - LF penalty, one task per (element, face node), into the first three words
// of the node's four in the neighbour block (the lift adds them).  A pass of its own so that a
// resident tile can run the whole pair loop before it waits for its neighbours' values.
// neighbour(i, v): h, u, v, H - Href on the other side of face node i.
template <typename real, int N, class LT, class FN>
__device__ __forceinline__ void interface_tile(const InstDesc &d, int ne, LT &L, FN neighbour) {
  constexpr int Nq = dim_Nq(N), Nfq = dim_Nfq(N);
  for (int i = interface_tid<N, LT>(); i < ne * Nfq; i += threads<LT>()) {
    const int e = int(unsigned(i) / unsigned(Nfq)), f = i - __umul24(unsigned(e), unsigned(Nfq));
    real t0, t1, t2;
    real nbp[4];
    neighbour(i, nbp);
    interface_terms<real>(L, __umul24(unsigned(e), unsigned(dim_Nh(N))) + Nq + f, nbp, L.wf[f], L.nr[f], L.ns[f],
                          real(d.g), d.flux, t0, t1, t2);
    L.nb[4 * i] = t0;
    L.nb[4 * i + 1] = t1;
    L.nb[4 * i + 2] = t2;
  }
}

// From the residual and interface terms to the updated state: the lift, the mass inverse and
// (mode kStage) the LSRK update, or (kRhs) the right-hand side.  write: the state and RK
// register go to HBM too.  Elements beyond a ragged tile's ne are dropped.
template <typename real, int N, int CM, bool WADG, class LT>
__device__ __forceinline__ void lift_update(const StageArgs &a, const StageRun &r, const InstDesc &d, int mode, int k0,
                                            int ne, LT &L, bool write) {
  constexpr int Np = dim_Np(N), Nh = dim_Nh(N);
  const int E = L.E, nth = threads<LT>();
  // lift: y = V_h^T r_h
  contract<CM, Np, Nh, Np, true, real>(L.Vh, 3 * E, nth >> 6, residual_in<real, N, CM != kMfmaBf16x3>(L), cols_out<Np>(L.T));
  __syncthreads();
  // rhs = -Minv y; store it, or do the LSRK update
  const size_t splane = size_t(d.K) * Np;
  real *uh = static_cast<real *>(d.uh);
  real *du = static_cast<real *>(d.du);
  const real ra = real(r.rk_a), rdt = real(d.dt), rb = real(r.rk_b);
  // one output per (field, element, mode)
  auto update = [&](int i, real y) {
    const real rr = -y;
    const FieldTask<Np> k(i, E * Np);
    // global index: field c's plane, the tile's first element, then r (zero-extended)
    const size_t o = size_t(unsigned(k.c)) * splane + size_t(k0) * Np + unsigned(k.r);
    const bool in = k.r < ne * Np;
    if (mode == kRhs) {
      if (in) static_cast<real *>(a.ext_rhs)[o] = rr;
    } else {
      const real dn = ra * L.DU[i] + rdt * rr;
      const real un = L.U[i] + rb * dn;
      if (write && in) {
        du[o] = dn;
        uh[o] = un;
      }
      L.DU[i] = dn;
      L.U[i] = un;
    }
  };
  if constexpr (WADG) {            // first factor into the residual block (dead after the lift)
    wadg_first<real, N>(L, L.T, L.R);
    __syncthreads();
    wadg_second<real, N>(L, L.R, L.T);
    __syncthreads();
    for (int i = phase_tid(); i < 3 * E * Np; i += nth) update(i, L.T[i]);
  } else {
    minv_rows<real, N>(L, L.T, update);
  }
}

// One stage (or projection, or right-hand side) of a tile that is fetched for it.
template <typename real, int N, int CM, bool WADG, bool MULTI, int EC, int NT>
__device__ __forceinline__ void stage_tile(const StageArgs &a, const StageRun &r, const InstDesc &d, int index, int k0,
                                           int ne, real *sm, real *tile) {
  constexpr int Nh = dim_Nh(N);
  typedef Lds<real, N, EC, NT> LT;
  const int tid = phase_tid(), nth = threads<LT>();
  LT L(sm, tile, d.E, mass_words(N, WADG));
  const int E = L.E;
  // The multi-stage build runs only multi-stage launches (and their residency probe, which
  // returns before any tile): RK stages on the instance buffers.  Taking that as given here
  // compiles the projection-only and RHS paths and the external buffers out of it, whose
  // addresses would otherwise stay live in scalar registers (and spill) across the stage.
  const int mode = MULTI ? int(kStage) : r.mode;
  fetch_tile<real, N, WADG, MULTI, EC>(a, r, d, index, k0, ne, L);
  __syncthreads();
  if (!MULTI && mode == kProject) {
    project_tile<real, N, CM, WADG>(d, k0, ne, L, static_cast<real *>(a.ext_ut ? a.ext_ut : d.ut[r.out_buf]),
                                    static_cast<real *>(a.ext_nbx ? a.ext_nbx : d.nbx[r.out_buf]), a.flag, false);
    return;
  }
  // phase 1: node records from the fetched u~
  const real g = real(d.g);
  for (int i = tid; i < ne * Nh; i += nth)
    write_record<real>(L, i, L.raw[i], L.raw[E * Nh + i], L.raw[2 * E * Nh + i], L.raw[3 * E * Nh + i], g);
  __syncthreads();
  residual_tile<real, N, RowsPerThread<real, N>::value>(ne, L);
  interface_tile<real, N>(d, ne, L, fetched_neighbours<real>(L));
  __syncthreads();
  lift_update<real, N, CM, WADG>(a, r, d, mode, k0, ne, L, true);
  if (mode == kStage) {
    __syncthreads();
    project_tile<real, N, CM, WADG>(d, k0, ne, L, static_cast<real *>(d.ut[r.out_buf]), static_cast<real *>(d.nbx[r.out_buf]),
                                    a.flag, MULTI);
  }
}

// All stages of a multi-stage launch for a tile that stays in LDS: its records, metric
// factors, static block, state and RK register are fetched once, each projection writes the
// next stage's records, and only the last stage writes the state, RK register and u~ back.
// Between stages the tile waits for its face neighbours after its pair loop and reads their
// pushed values straight into the interface terms.  A wait that gives up sets flag bit 1;
// the workgroup then goes on without waiting any more (the state is undefined and the flag
// reports it), so every workgroup ends.
// Bound by the chain of its short phases, then by the neighbours' skew.  Measured per stage,
// before (one stage body for all launches, counts packed 32 to a line) and now: FP32 N = 3,
// K = 8192 8.66 -> 7.33 us, N = 2 K = 8192 7.3 -> 6.3, N = 1 K = 8192 6.05 -> 4.91, FP64
// N = 2 K = 8192 10.05 -> 8.65; with packed counts this loop alone made N = 1 7.1 us (each
// publish took its line from all the pollers of 32 tiles).  With the wait and the interface
// terms on the waves that have them, and no barrier before: N = 3, K = 512 5.56 -> 5.07, K = 8192
// 7.26 -> 7.1, N = 1, K = 8192 4.35 -> 4.07, FP64 N = 2 7.9 -> 7.45, N = 3, K = 3200 7.3 -> 6.8.
template <typename real, int N, int CM, bool WADG, int EC, int NT>
__device__ __forceinline__ void resident_tile(const StageArgs &a, const InstDesc &d, int t, int index, int k0, int ne,
                                              real *sm, real *tile) {
  constexpr int Nh = dim_Nh(N), Nfq = dim_Nfq(N);
  typedef Lds<real, N, EC, NT> LT;
  LT L(sm, tile, d.E, mass_words(N, WADG));
  const int E = L.E, nth = threads<LT>();
  const real g = real(d.g);
  StageRun r{kStage, a.in_buf, 1 - a.in_buf, 0.0, 0.0};
  fetch_tile<real, N, WADG, true, EC>(a, r, d, index, k0, ne, L);
  __syncthreads();
  for (int i = phase_tid(); i < ne * Nh; i += nth)
    write_record<real>(L, i, L.raw[i], L.raw[E * Nh + i], L.raw[2 * E * Nh + i], L.raw[3 * E * Nh + i], g);
  __syncthreads();
  bool waits = true;
#pragma unroll 1
  for (int s = 0, s5 = 0; s < a.nstages; ++s, s5 = s5 == 4 ? 0 : s5 + 1) {
    const bool last = s + 1 == a.nstages;
    r.rk_a = a.rk_a5[s5];
    r.rk_b = a.rk_b5[s5];
    residual_tile<real, N, RowsPerThread<real, N>::value>(ne, L);
    if (s > 0) {
      // a wave with interface tasks waits and runs them while others are in their pair loop
      if (__builtin_amdgcn_readfirstlane(interface_tid<N, LT>()) < ne * Nfq) {
        waits = poll_neighbours(a, t, a.stage0 + s, waits);
        const real *nbx = static_cast<const real *>(d.nbx[r.in_buf]) + size_t(k0) * Nfq * 4;
        interface_tile<real, N>(d, ne, L, [nbx](int i, real *v) {
          load_coherent(nbx + 4 * size_t(unsigned(i)), v);
        });
      }
    } else {
      interface_tile<real, N>(d, ne, L, fetched_neighbours<real>(L));
    }
    __syncthreads();
    // from here to its publish the tile is on its neighbours' critical path (their next
    // stage waits for its pushes), while the other workgroups on the CU that are still in
    // their pair loop have slack: raise this workgroup's wave priority until the publish
    __builtin_amdgcn_s_setprio(2);
    lift_update<real, N, CM, WADG>(a, r, d, kStage, k0, ne, L, last);
    __syncthreads();
    project_tile<real, N, CM, WADG>(d, k0, ne, L, static_cast<real *>(d.ut[r.out_buf]), static_cast<real *>(d.nbx[r.out_buf]),
                                    a.flag, true, !last);
    publish(a, t, a.stage0 + s + 1);
    __builtin_amdgcn_s_setprio(0);
    r.in_buf = r.out_buf;
    r.out_buf = 1 - r.in_buf;
  }
}

// Persistent stage kernel: block b walks a contiguous range of tiles.  Blocks are dealt
// to the XCDs round-robin, so block b's range is chosen as range number
// (b mod kXcds) * (gridDim / kXcds) + b / kXcds: each XCD owns a contiguous run of tiles.
// The reference-operator block stays in LDS and is reloaded only when the degree changes.
// With a.progress set, the launch runs a.nstages RK stages: each block takes its tiles
// through stage s before stage s + 1, and a tile starts a stage once its face neighbours'
// tiles have finished the previous one (see wait_neighbours), which the co-residency of
// all workgroups (cooperative launch) makes safe.  A wait that gives up sets flag bit 1
// and ends the workgroup; its neighbours' waits then give up in turn.
// V1: the build that also holds the variant-1 element kinds (N+2 points per direction and
// per face); launches whose instances are all of variant 0 use the build without them,
// whose register allocation those larger kinds do not affect.  KIND: a build for one
// variant-0 kind alone, used when every instance is of that kind: its registers are
// allocated for that kind's code only.  EC: a build of that for one tile size.
// Residency probe of a multi-stage grid (kProbe): every workgroup counts itself in and waits,
// with a bounded spin, until the whole grid has; a wait that gives up sets flag bit 2.  Run
// once at bind with the grid, workgroup size and LDS of the multi-stage launches: if every
// workgroup was resident at once, those launches go out as ordinary launches, else as
// cooperative ones.  The count is a word of the flag block of its own.
__device__ __forceinline__ void residency_probe(const StageArgs &a) {
  if (threadIdx.x == 0) {
    int32_t *count = a.flag + kProbeWord;
    __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int spins = 0;
    while (__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < int(gridDim.x)) {
      if (++spins > a.spin_limit) {
        atomicOr(a.flag, 4);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
}

// Threads of a kernel built for one kind, or for several with fixed tiles (as the host launches
// it; 0: not a constant).
__host__ __device__ constexpr int stage_kernel_threads(int kind, int tile) {
  return kind == 0 ? (tile == kFixedTiles ? kBlock : 0) : wide_kind(kind) ? kBlockWide : kBlock;
}

// Waves per SIMD that a kernel's registers have to allow.  Four, what the LDS of the default tile
// sizes leaves room for, except in the builds with run-time offsets: those also serve small tiles,
// of which more fit a CU (five workgroups where registers and LDS meet, six in FP32 at N = 4,
// and three of 512 threads at N = 5).  Left at four they took up to 101 registers, so that fewer
// workgroups than tiles were resident, K = 4608: FP32 N = 3, four elements to a tile 11.6 us a
// stage instead of 6.3, FP64 N = 2, four 18.6 instead of 7.4, FP32 N = 5, two 49.0 instead of 35.6.
// FP32 N = 4 is slower at six where LDS holds fewer: eight elements, K = 512 9.1 -> 10.4.  FP64
// N = 4 and 5 have no room in LDS for a fifth (a third at N = 5).
template <typename real> __host__ __device__ constexpr int stage_waves(int kind, int tile) {
  if (kind == 0 || key_variant(kind) != 0 || tile != 0) return 4;
  return kind <= 3 ? 5 : sizeof(real) == 4 ? 6 : 4;
}

template <typename real, int CM, bool WADG, bool MULTI, bool V1, int KIND = 0, int EC = 0>
__global__ void __launch_bounds__(kBlockWide) __attribute__((amdgpu_waves_per_eu(stage_waves<real>(KIND, EC))))
stage_kernel(StageArgs a) {
  if (MULTI && a.mode == kProbe) {
    residency_probe(a);
    return;
  }
  constexpr int NT = stage_kernel_threads(KIND, EC);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  real *sm = reinterpret_cast<real *>(smem_raw);
  real *tile = sm + (KIND != 0 ? (ref_words(KIND) + 3) & ~3 : a.ref_words_max);
  const int G = int(gridDim.x);
  const int chunk = (int(blockIdx.x) % kXcds) * (G / kXcds) + int(blockIdx.x) / kXcds;
  const int t0 = a.ranges ? read_const(a.ranges, chunk) : int((long long)chunk * a.ntiles / G);
  const int t1 = a.ranges ? read_const(a.ranges, chunk + 1) : int((long long)(chunk + 1) * a.ntiles / G);
  // MULTI: the multi-stage instantiation; the per-stage one compiles without the waits,
  // resident tiles and device-coherent pushes (and keeps the registers they would cost)
  const bool multi = MULTI && a.progress != nullptr;
  // resident: the launch has a workgroup for every tile (and then no ranges), so this one has at
  // most one
  const bool resident = multi && a.resident && t1 - t0 <= 1;
  const int nst = !multi ? 1 : resident ? (t1 > t0 ? 1 : 0) : a.nstages;
  int loaded_N = 0;
  for (int s = 0; s < nst; ++s) {
    StageRun r{a.mode, a.in_buf, a.out_buf, a.rk_a, a.rk_b};
    if (multi) {
      r.mode = kStage;
      r.in_buf = (a.in_buf + s) & 1;
      r.out_buf = 1 - r.in_buf;
      r.rk_a = a.rk_a5[s % 5];
      r.rk_b = a.rk_b5[s % 5];
    }
    for (int t = t0; t < t1; ++t) {
      if (multi && s > 0 && !wait_neighbours(a, t, a.stage0 + s)) {
        if (threadIdx.x == 0) atomicOr(a.flag, 2);
        return;
      }
      const Tile tl = read_const(a.tiles, t);
      const InstDesc &d = read_const(a.desc, tl.inst);
      if (KIND != 0 ? loaded_N == 0 : d.N != loaded_N) {
        // the reference block, copied with the tile's data (which fetch_tile waits for)
        if (KIND == 0) __syncthreads();
        constexpr int words = KIND != 0 ? (ref_words(KIND) + 3) & ~3 : 0;
        copy_block<Threads<NT>, words * int(sizeof(real))>(sm, d.ref, ((ref_words(d.N) + 3) & ~3) * int(sizeof(real)));
        loaded_N = KIND != 0 ? KIND : d.N;
      }
#define ESDG_STAGE_TILE(D, E)                                                                                  \
  if (MULTI && resident) resident_tile<real, D, CM, WADG, E, NT>(a, d, t, tl.index, tl.k0, tl.ne, sm, tile);   \
  else stage_tile<real, D, CM, WADG, MULTI, E, NT>(a, r, d, tl.index, tl.k0, tl.ne, sm, tile)
#define ESDG_STAGE_CASE(D)                                                                                     \
  case D: {                                                                                                    \
    constexpr int E1 = EC == kFixedTiles ? fixed_tile<real>(D) : EC;                                           \
    constexpr int E2 = EC == kFixedTiles ? other_tile<real>(D) : 0;                                            \
    if constexpr (E2 == 0) {                                                                                   \
      ESDG_STAGE_TILE(D, E1);                                                                                  \
    } else {                                                                                                   \
      if (d.E == E1) { ESDG_STAGE_TILE(D, E1); }                                                               \
      else if (d.E == E2) { ESDG_STAGE_TILE(D, E2); }                                                          \
      else { ESDG_STAGE_TILE(D, 0); }                                                                          \
    }                                                                                                          \
    break;                                                                                                     \
  }
      if constexpr (KIND != 0) {     // every tile is of this kind (the host's choice of kernel)
        switch (KIND) {
          ESDG_STAGE_CASE(KIND)
          default: break;
        }
      } else if constexpr (V1) {
        switch (d.N) {
          ESDG_STAGE_CASE(1) ESDG_STAGE_CASE(2) ESDG_STAGE_CASE(3) ESDG_STAGE_CASE(4) ESDG_STAGE_CASE(5)
          ESDG_STAGE_CASE(9) ESDG_STAGE_CASE(10) ESDG_STAGE_CASE(11) ESDG_STAGE_CASE(12) ESDG_STAGE_CASE(13)
          default: break;
        }
      } else {
        switch (d.N) {
          ESDG_STAGE_CASE(1) ESDG_STAGE_CASE(2) ESDG_STAGE_CASE(3) ESDG_STAGE_CASE(4) ESDG_STAGE_CASE(5)
          default: break;
        }
      }
#undef ESDG_STAGE_TILE
#undef ESDG_STAGE_CASE
      if (multi && !resident) publish(a, t, a.stage0 + s + 1);
      else __syncthreads();
    }
  }
}

// FP64 diagnostics per tile: mass (3), entropy, entropy rate, sum |entropy-rate terms|.
// Everything but the state and the RHS (widened exactly from the bulk precision) is double:
// V_q, w J and the bathymetry come from double copies kept for the diagnostics.
template <typename real, int D>
__device__ void diag_tile(const InstDesc &d, int k0, int ne, double *acc) {
  constexpr int Np = dim_Np(D), Nq = dim_Nq(D), Nh = dim_Nh(D);
  const real *uh = static_cast<const real *>(d.uh);
  const real *rh = static_cast<const real *>(d.rhs_scratch);
  const double *wJq = static_cast<const double *>(d.wJq);
  const size_t splane = size_t(d.K) * Np;
  const double g = d.g;
  for (int i = threadIdx.x; i < ne * Nq; i += blockDim.x) {
    const int e = i / Nq, q = i - e * Nq, k = k0 + e;
    double u[3] = {0, 0, 0}, r[3] = {0, 0, 0};
    if constexpr (key_sbp(D)) {    // nodal state: the values at the volume nodes themselves
      for (int c = 0; c < 3; ++c) {
        u[c] = double(uh[c * splane + size_t(k) * Np + q]);
        r[c] = double(rh[c * splane + size_t(k) * Np + q]);
      }
    } else {
      for (int j = 0; j < Np; ++j) {
        const double v = d.Vqd[q * Np + j];
        for (int c = 0; c < 3; ++c) {
          u[c] += v * double(uh[c * splane + size_t(k) * Np + j]);
          r[c] += v * double(rh[c * splane + size_t(k) * Np + j]);
        }
      }
    }
    const double w = wJq[size_t(k) * Nq + q], b = d.bd[size_t(k) * Nh + q];
    const double h = u[0] + (d.Href - b), uu = u[1] / h, vv = u[2] / h;
    acc[0] += w * h;
    acc[1] += w * u[1];
    acc[2] += w * u[2];
    acc[3] += w * (0.5 * h * (uu * uu + vv * vv) + 0.5 * g * h * h + g * h * b);
    const double t0 = w * (g * (h + b) - 0.5 * (uu * uu + vv * vv)) * r[0];
    const double t1 = w * uu * r[1], t2 = w * vv * r[2];
    acc[4] += t0 + t1 + t2;
    acc[5] += fabs(t0) + fabs(t1) + fabs(t2);
  }
}

template <typename real>
__global__ void __launch_bounds__(kBlock) diag_kernel(DiagArgs a) {
  __shared__ double red[kBlock][6];
  const int t = blockIdx.x;
  if (t >= a.ntiles) return;
  const Tile tl = read_const(a.tiles, t);
  const InstDesc &d = read_const(a.desc, tl.inst);
  double acc[6] = {0, 0, 0, 0, 0, 0};
  switch (d.N) {
#define ESDG_DIAG_CASE(D) \
  case D: diag_tile<real, D>(d, tl.k0, tl.ne, acc); break;
    ESDG_DIAG_CASE(1) ESDG_DIAG_CASE(2) ESDG_DIAG_CASE(3) ESDG_DIAG_CASE(4) ESDG_DIAG_CASE(5)
    ESDG_DIAG_CASE(9) ESDG_DIAG_CASE(10) ESDG_DIAG_CASE(11) ESDG_DIAG_CASE(12) ESDG_DIAG_CASE(13)
    ESDG_DIAG_CASE(17) ESDG_DIAG_CASE(18) ESDG_DIAG_CASE(19) ESDG_DIAG_CASE(20)
#undef ESDG_DIAG_CASE
    default: break;
  }
  for (int c = 0; c < 6; ++c) red[threadIdx.x][c] = acc[c];
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if (int(threadIdx.x) < s)
      for (int c = 0; c < 6; ++c) red[threadIdx.x][c] += red[threadIdx.x + s][c];
    __syncthreads();
  }
  if (threadIdx.x == 0)
    for (int c = 0; c < 6; ++c) a.partials[size_t(t) * 6 + c] = red[0][c];
}

// The rest depth Href - b of every tile of an instance, rounded once from double into the
// static block (Href changes at every set_state).  One workgroup per tile.
template <typename real>
__global__ void __launch_bounds__(kBlock) rest_depth_kernel(DiagArgs a) {
  const int t = blockIdx.x;
  if (t >= a.ntiles) return;
  const Tile tl = read_const(a.tiles, t);
  const InstDesc &d = read_const(a.desc, tl.inst);
  const int D = d.N, Nq = dim_Nq(D), Nh = dim_Nh(D), ne = tl.ne, E = d.E;
  const bool wadg = a.wadg != 0;
  real *st = static_cast<real *>(const_cast<void *>(d.stat)) + size_t(tl.index) * stat_tile(D, E, wadg);
  // modal kinds: Href - b at the volume nodes, then at the hybrid nodes, after the mass data
  // and w J; DG-SBP: at the volume nodes, after 1/(w J)
  real *dq = st + E * (key_sbp(D) ? Nq : mass_words(D, wadg) + Nq);
  real *dh = dq + E * Nq;
  for (int i = threadIdx.x; i < ne * Nq; i += blockDim.x) {
    const int e = i / Nq, q = i - e * Nq;
    dq[i] = real(d.Href - d.bd[size_t(tl.k0 + e) * Nh + q]);
  }
  if (!key_sbp(D))
    for (int i = threadIdx.x; i < ne * Nh; i += blockDim.x) {
      const int e = i / Nh, n = i - e * Nh;
      dh[i] = real(d.Href - d.bd[size_t(tl.k0 + e) * Nh + n]);
    }
}

// ---------------------------------------------------------------- DG-SBP (Section 3)
// The DG-SBP scheme with traditional SBP operators obtained from the hybridized ones
// (Section 3.2): Q_SBP = [I; I_f]^T Q_h [I; I_f] on a volume rule whose boundary nodes are
// the face nodes, diagonal mass matrix W J, nodal state at the volume nodes, no entropy
// projection.  Per element,
//   (W J) du/dt = -[I; I_f]^T r_h,
// where r_h is the hybridized residual of the modal kernel (skew form, zero block skipped,
// folded source, interface terms) evaluated with the face values taken from the volume
// nodes they coincide with: each face row is added to its volume node's row.

// LDS carve-up of one DG-SBP tile (see tile_words()).  EC: E where the kernel is built for one
// tile size, else 0.
template <typename real, int D, int EC>
struct LdsSbp {
  static constexpr int Nq = dim_Nq(D), Nfq = dim_Nfq(D), Nh = dim_Nh(D), NT = kBlock;
  real *ref, *ST, *FT, *wf, *nr, *ns, *fvol, *vface;
  real *q0, *q1, *dH, *p, *R, *nb, *U, *DU, *iwJ, *dep, *geo;
  int32_t *pp;
  int E;
  __device__ LdsSbp(real *sm, real *tile, int e) : E(EC != 0 ? EC : e) {
    ref = sm;
    ST = ref;
    FT = ST + 2 * Nh * Nq;
    wf = FT + 2 * Nq * Nfq;
    nr = wf + Nfq;
    ns = nr + Nfq;
    fvol = ns + Nfq;              // volume node of face node f (integer-valued reals)
    vface = fvol + Nfq;           // face node of volume node n, or -1
    q0 = tile;
    q1 = q0 + 4 * E * Nh;
    R = q1 + 4 * E * Nh;          // two parts of the residual [2][3][E][Nh]
    nb = R + ((6 * E * Nh + 3) & ~3);   // 16-byte aligned, as the static block after it
    iwJ = nb + 4 * E * Nfq;       // static block: 1/(w J) | rest depth | metrics [4][E][Nq] | push targets
    dep = iwJ + E * Nq;
    geo = dep + E * Nq;
    pp = reinterpret_cast<int32_t *>(geo + 4 * E * Nq);
    U = geo + E * (4 * Nq + Nfq);
    DU = U + 3 * E * Nq;
    dH = DU + 3 * E * Nq;
    p = dH + E * Nh;
  }
};

// Face node f of element e (its volume node is entry j of the tile): the values (h, u, v,
// H - Href) of its state, pushed into the neighbour's slot (a reflective wall node, Section
// 2.9, writes the mirror state into its own slot).  True for a non-physical state.
template <typename real, int D, class LT>
__device__ __forceinline__ bool sbp_push(const LT &L, int e, int f, int j, double eta, double hu, double hv,
                                         real *nbx_out) {
  constexpr int Nq = dim_Nq(D), Nfq = dim_Nfq(D);
  typedef real real4 __attribute__((ext_vector_type(4)));
  const double h = eta + double(L.dep[j]);
  const double u = hu / h, v = hv / h;
  double pu = u, pv = v;
  const uint32_t tgt = uint32_t(L.pp[__umul24(unsigned(e), unsigned(Nfq)) + f]);
  if (tgt & kPushWall) {
    const double nr = double(L.nr[f]), ns = double(L.ns[f]);
    const double nx = double(L.geo[j]) * nr + double(L.geo[L.E * Nq + j]) * ns;
    const double ny = double(L.geo[2 * L.E * Nq + j]) * nr + double(L.geo[3 * L.E * Nq + j]) * ns;
    const double c = 2.0 * (u * nx + v * ny) / (nx * nx + ny * ny);
    pu = u - c * nx;
    pv = v - c * ny;
  }
  *reinterpret_cast<real4 *>(nbx_out + size_t(tgt & ~kPushWall) * 4) = real4{real(h), real(pu), real(pv), real(eta)};
  return bad_value(h, hu, hv);
}

// One DG-SBP tile: fetch, node records, residual and interface terms, then one task per volume
// node for the update and, at a boundary node, its push.  Bound by the chain of those phases
// and the pair loop's vector work.  Measured per stage with one kernel for all degrees and
// tile sizes, records and pushes in phases of their own, and now: FP32 K = 32768 N = 1..4
// 17.7, 28, 41.6, 54 -> 14.9, 20.3, 34, 49 us; FP64 N = 4, K = 8192 30 -> 25.6.
template <typename real, int D, int EC>
__device__ __forceinline__ void sbp_tile(const StageArgs &a, const InstDesc &d, int index, int k0, int ne, real *sm,
                                         real *tile) {
  constexpr int Nq = dim_Nq(D), Nfq = dim_Nfq(D), Nh = dim_Nh(D), SW = stat_words(D);
  typedef LdsSbp<real, D, EC> LT;
  typedef real real4 __attribute__((ext_vector_type(4)));
  LT L(sm, tile, d.E);
  const int E = L.E;
  const int tid = phase_tid(), nth = kBlock;
  const size_t splane = size_t(d.K) * Nq;
  // fetch: state, RK register, static block, neighbour values
  copy_state<LT, Nq, EC>(L.U, a.ext_state ? a.ext_state : d.uh, splane, k0, ne, E);
  if (a.mode == kStage) copy_state<LT, Nq, EC>(L.DU, d.du, splane, k0, ne, E);
  copy_block<LT, EC * SW * int(sizeof(real))>(L.iwJ, static_cast<const real *>(d.stat) + size_t(index) * stat_tile(D, E, false),
                                              E * SW * int(sizeof(real)));
  if (a.mode != kProject) {
    const real *nbx = static_cast<const real *>(a.ext_nbx ? a.ext_nbx : d.nbx[a.in_buf]) + size_t(k0) * Nfq * 4;
    copy_block<LT, EC * Nfq * 4 * int(sizeof(real))>(L.nb, nbx, ne * Nfq * 4 * int(sizeof(real)));
  }
  wait_copies();
  __syncthreads();
  real *nbx_out = static_cast<real *>(a.ext_nbx ? a.ext_nbx : d.nbx[a.out_buf]);
  bool bad = false;
  if (a.mode == kProject) {
    for (int i = tid; i < ne * Nfq; i += nth) {
      const int e = int(unsigned(i) / unsigned(Nfq)), f = i - e * Nfq, j = e * Nq + int(L.fvol[f]);
      bad |= sbp_push<real, D>(L, e, f, j, L.U[j], L.U[E * Nq + j], L.U[2 * E * Nq + j], nbx_out);
    }
    if (bad) atomicOr(a.flag, 1);
    return;
  }
  // node records, from the nodal state (h in double from eta and the rest depth; H - Href is
  // eta itself); the face nodes' are those of the volume nodes they coincide with
  const real g = real(d.g);
  for (int i = tid; i < ne * Nh; i += nth) {
    const int e = int(unsigned(i) / unsigned(Nh)), n = i - e * Nh, q = n < Nq ? n : int(L.fvol[n - Nq]);
    const int j = e * Nq + q;
    const double eta = L.U[j], hu = L.U[E * Nq + j], hv = L.U[2 * E * Nq + j];
    const double h = eta + double(L.dep[j]);
    const double u = hu / h, v = hv / h;
    reinterpret_cast<real4 *>(L.q0)[i] = real4{real(0.5 * hu), real(0.5 * hv), real(0.5 * u), real(0.5 * v)};
    reinterpret_cast<real4 *>(L.q1)[i] = real4{L.geo[j], L.geo[E * Nq + j], L.geo[2 * E * Nq + j], L.geo[3 * E * Nq + j]};
    L.dH[i] = real(eta);
    L.p[i] = real(0.5) * g * real(h);
    bad |= bad_value(h, hu, hv);
  }
  __syncthreads();
  residual_tile<real, D, RowsPerThread<real, D>::value>(ne, L);
  interface_tile<real, D>(d, ne, L, fetched_neighbours<real>(L));
  __syncthreads();
  // du/dt = -(W J)^{-1} [I; I_f]^T r_h; store it, or do the LSRK update and push
  const real ra = real(a.rk_a), rdt = real(d.dt), rb = real(a.rk_b);
  for (int j = tid; j < ne * Nq; j += nth) {
    const int e = int(unsigned(j) / unsigned(Nq)), n = j - e * Nq;
    const int vf = int(L.vface[n]);
    const real iw = L.iwJ[j];
    real un[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const auto rh = residual_in<real, D, true>(L)(c * E + e);
      real r = rh(n, n >> 2);
      if (vf >= 0) r += rh(Nq + vf, (Nq + vf) >> 2);
      const real rr = -r * iw;
      const size_t o = size_t(c) * splane + size_t(k0) * Nq + j;
      if (a.mode == kRhs) {
        static_cast<real *>(a.ext_rhs)[o] = rr;
      } else {
        const int l = c * E * Nq + j;
        const real dn = ra * L.DU[l] + rdt * rr;
        un[c] = L.U[l] + rb * dn;
        static_cast<real *>(d.du)[o] = dn;
        static_cast<real *>(d.uh)[o] = un[c];
      }
    }
    if (a.mode == kStage && vf >= 0) bad |= sbp_push<real, D>(L, e, vf, j, un[0], un[1], un[2], nbx_out);
  }
  if (bad) atomicOr(a.flag, 1);
}

// One launch per RK stage (or per projection / RHS) for every DG-SBP tile; persistent,
// XCD-aligned chunks as in stage_kernel.  KIND, EC: as in stage_kernel.
template <typename real, int KIND = 0, int EC = 0>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4)))
sbp_stage_kernel(StageArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  real *sm = reinterpret_cast<real *>(smem_raw);
  real *tile = sm + (KIND != 0 ? (ref_words(KIND) + 3) & ~3 : a.ref_words_max);
  const int G = int(gridDim.x);
  const int chunk = (int(blockIdx.x) % kXcds) * (G / kXcds) + int(blockIdx.x) / kXcds;
  const int t0 = a.ranges ? read_const(a.ranges, chunk) : int((long long)chunk * a.ntiles / G);
  const int t1 = a.ranges ? read_const(a.ranges, chunk + 1) : int((long long)(chunk + 1) * a.ntiles / G);
  int loaded = 0;
  for (int t = t0; t < t1; ++t) {
    const Tile tl = read_const(a.tiles, t);
    const InstDesc &d = read_const(a.desc, tl.inst);
    if (KIND != 0 ? loaded == 0 : d.N != loaded) {
      // the reference block, copied with the tile's data (which sbp_tile waits for)
      constexpr int words = KIND != 0 ? (ref_words(KIND) + 3) & ~3 : 0;
      copy_block<Threads<kBlock>, words * int(sizeof(real))>(sm, d.ref, ((ref_words(d.N) + 3) & ~3) * int(sizeof(real)));
      loaded = KIND != 0 ? KIND : d.N;
    }
    if constexpr (KIND != 0) {
      sbp_tile<real, KIND, EC>(a, d, tl.index, tl.k0, tl.ne, sm, tile);
    } else {
      switch (d.N) {
#define ESDG_SBP_CASE(N) \
  case make_key(N, 2): sbp_tile<real, make_key(N, 2), 0>(a, d, tl.index, tl.k0, tl.ne, sm, tile); break;
        ESDG_SBP_CASE(1) ESDG_SBP_CASE(2) ESDG_SBP_CASE(3) ESDG_SBP_CASE(4)
#undef ESDG_SBP_CASE
        default: break;
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- instantiation units
// This file is compiled once per (precision, mass inverse) with ESDG_UNIT_REAL and
// ESDG_UNIT_WADG defined, instantiating the stage kernels of that combination only, and
// once with ESDG_UNIT_HOST for the DG-SBP, diagnostics and rest-depth kernels and the host
// launchers; the five objects compile in parallel.  Each unit exports the stage kernels of
// its combination by contraction mode and launch kind.
#define ESDG_CAT4(a, b, c, d) a##b##c##d
#define ESDG_UNIT_FN(R, W) ESDG_CAT4(stage_fn_unit_, R, _, W)
const void *stage_fn_unit_float_0(int cm, bool multi, bool v1, int kind, int tile);
const void *stage_fn_unit_float_1(int cm, bool multi, bool v1, int kind, int tile);
const void *stage_fn_unit_double_0(int cm, bool multi, bool v1, int kind, int tile);
const void *stage_fn_unit_double_1(int cm, bool multi, bool v1, int kind, int tile);

#if defined(ESDG_UNIT_REAL)
template <bool V1>
static const void *unit_fn(int cm, bool multi, int tile) {
  using real = ESDG_UNIT_REAL;
  constexpr bool W = ESDG_UNIT_WADG != 0;
  if constexpr (std::is_same<real, float>::value) {
    if (cm == kMfmaBf16x3)
      return multi ? reinterpret_cast<const void *>(&stage_kernel<float, kMfmaBf16x3, W, true, V1>)
                   : reinterpret_cast<const void *>(&stage_kernel<float, kMfmaBf16x3, W, false, V1>);
  }
  if constexpr (!V1)
    if (tile == kFixedTiles)
      return multi ? reinterpret_cast<const void *>(&stage_kernel<real, kMfmaNative, W, true, false, 0, kFixedTiles>)
                   : reinterpret_cast<const void *>(&stage_kernel<real, kMfmaNative, W, false, false, 0, kFixedTiles>);
  return multi ? reinterpret_cast<const void *>(&stage_kernel<real, kMfmaNative, W, true, V1>)
               : reinterpret_cast<const void *>(&stage_kernel<real, kMfmaNative, W, false, V1>);
}
template <int K, int EC>
static const void *tile_fn(bool multi) {
  using real = ESDG_UNIT_REAL;
  constexpr bool W = ESDG_UNIT_WADG != 0;
  return multi ? reinterpret_cast<const void *>(&stage_kernel<real, kMfmaNative, W, true, false, K, EC>)
               : reinterpret_cast<const void *>(&stage_kernel<real, kMfmaNative, W, false, false, K, EC>);
}
template <int K>
static const void *kind_fn(bool multi, int tile) {
  using real = ESDG_UNIT_REAL;
  if (tile == fixed_tile<real>(K)) return tile_fn<K, fixed_tile<real>(K)>(multi);
  if constexpr (other_tile<real>(K) != 0)
    if (tile == other_tile<real>(K)) return tile_fn<K, other_tile<real>(K)>(multi);
  return tile_fn<K, 0>(multi);
}
const void *ESDG_UNIT_FN(ESDG_UNIT_REAL, ESDG_UNIT_WADG)(int cm, bool multi, bool v1, int kind, int tile) {
  if (cm != kMfmaBf16x3 && !v1) {  // one variant-0 kind: that kind's own build
    switch (kind) {
      case 1: return kind_fn<1>(multi, tile);
      case 2: return kind_fn<2>(multi, tile);
      case 3: return kind_fn<3>(multi, tile);
      case 4: return kind_fn<4>(multi, tile);
      case 5: return kind_fn<5>(multi, tile);
      default: break;
    }
  }
  return v1 ? unit_fn<true>(cm, multi, tile) : unit_fn<false>(cm, multi, tile);
}
#endif

#if defined(ESDG_UNIT_HOST)
// ---------------------------------------------------------------- host launchers

// The stage kernel for a precision, contraction mode, mass inverse and launch kind (one
// launch per stage, or all stages of a step call in one multi-stage launch).  One launch
// per stage runs the per-stage instantiation, built without the waits, resident tiles and
// coherent pushes.
static const void *stage_fn(bool fp64, int cm, bool wadg, bool multi, bool v1, int kind, int tile) {
  if (fp64)
    return wadg ? stage_fn_unit_double_1(cm, multi, v1, kind, tile) : stage_fn_unit_double_0(cm, multi, v1, kind, tile);
  return wadg ? stage_fn_unit_float_1(cm, multi, v1, kind, tile) : stage_fn_unit_float_0(cm, multi, v1, kind, tile);
}

template <typename real, int K>
static const void *sbp_kind_fn(int tile) {
  constexpr int EC = fixed_tile<real>(K);
  return tile == EC ? reinterpret_cast<const void *>(&sbp_stage_kernel<real, K, EC>)
                    : reinterpret_cast<const void *>(&sbp_stage_kernel<real, K>);
}
template <typename real>
static const void *sbp_fn(int kind, int tile) {
  switch (kind) {
    case make_key(1, 2): return sbp_kind_fn<real, make_key(1, 2)>(tile);
    case make_key(2, 2): return sbp_kind_fn<real, make_key(2, 2)>(tile);
    case make_key(3, 2): return sbp_kind_fn<real, make_key(3, 2)>(tile);
    case make_key(4, 2): return sbp_kind_fn<real, make_key(4, 2)>(tile);
    default: return reinterpret_cast<const void *>(&sbp_stage_kernel<real>);
  }
}
// StageArgs.tile of a launch of several kinds with E elements to a tile of kind D (epb): the
// kernel with fixed tiles holds one size for each of N = 3, 4 and 5 (of which nothing fits
// better, see fixed_tile) and any for N = 1 and 2.
int mixed_tile(bool fp64, const std::map<int, int> &epb);
int mixed_tile(bool fp64, const std::map<int, int> &epb) {
  for (const auto &kv : epb) {
    if (key_variant(kv.first) != 0) return 0;
    if (kv.first > 2 && kv.second != (fp64 ? fixed_tile<double>(kv.first) : fixed_tile<float>(kv.first))) return 0;
  }
  return kFixedTiles;
}

static const void *sbp_fn(bool fp64, int kind, int tile) {
  return fp64 ? sbp_fn<double>(kind, tile) : sbp_fn<float>(kind, tile);
}

// Workgroups of the per-stage or multi-stage kernel (the DG-SBP kernel with sbp) that stay
// resident on the whole device with lds_bytes of dynamic LDS each.
hipError_t stage_max_blocks(bool fp64, int cm, bool wadg, bool sbp, bool v1, int kind, int tile, bool multi,
                            size_t lds_bytes, int block, int *out) {
  int dev = 0, ncu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  // The occupancy query does not round the LDS request up to the allocation granule; a
  // workgroup count it reports can then fail to fit, and the persistent grid's surplus
  // blocks only start when others finish (for a multi-stage launch, which needs every
  // workgroup resident at once, their neighbours then wait for stages that cannot come).
  // So cap it with 1 KiB granules of the CU's LDS, counting the kernel's own static LDS
  // (the multi-stage build's workgroup reduction) on top of the dynamic request.
  int lds_cu = 0;
  e = hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev);
  if (e != hipSuccess) return e;
  const void *fn = sbp ? sbp_fn(fp64, kind, tile) : stage_fn(fp64, cm, wadg, multi, v1, kind, tile);
  int n = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, block, lds_bytes);
  if (e != hipSuccess) return e;
  hipFuncAttributes fa{};
  e = hipFuncGetAttributes(&fa, fn);
  if (e != hipSuccess) return e;
  const size_t granule = 1024, total = lds_bytes + fa.sharedSizeBytes;
  const size_t need = (total + granule - 1) / granule * granule;
  if (need > 0 && lds_cu > 0) n = std::min<long long>(n, (long long)(size_t(lds_cu) / need));
  *out = ncu * (n > 0 ? n : 1);
  return hipSuccess;
}

hipError_t set_stage_lds_limit(bool fp64, int cm, bool wadg, bool sbp, bool v1, int kind, int tile,
                               size_t lds_bytes) {
  if (sbp) return hipFuncSetAttribute(sbp_fn(fp64, kind, tile), hipFuncAttributeMaxDynamicSharedMemorySize, int(lds_bytes));
  hipError_t e = hipFuncSetAttribute(stage_fn(fp64, cm, wadg, false, v1, kind, tile),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, int(lds_bytes));
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(stage_fn(fp64, cm, wadg, true, v1, kind, tile), hipFuncAttributeMaxDynamicSharedMemorySize,
                             int(lds_bytes));
}

// Persistent grid: at most max_blocks (what stays resident), at most one block per tile,
// always a whole number of XCD rounds (blocks whose range is empty just exit).
int stage_grid(int ntiles, int max_blocks);
int stage_grid(int ntiles, int max_blocks) {
  int g = ntiles < max_blocks ? ntiles : max_blocks;
  return ((g + kXcds - 1) / kXcds) * kXcds;
}

hipError_t launch_stage(bool fp64, bool sbp, const StageArgs &a, int max_blocks, size_t lds_bytes, int block,
                        hipStream_t stream) {
  if (a.ntiles <= 0) return hipSuccess;
  const int grid = stage_grid(a.ntiles, max_blocks);
  StageArgs arg = a;
  void *params[] = {&arg};
  return hipLaunchKernel(sbp ? sbp_fn(fp64, a.kind, a.tile)
                             : stage_fn(fp64, a.contraction, a.wadg != 0, false, a.v1 != 0, a.kind, a.tile),
                         dim3(grid),
                         dim3(sbp ? kBlock : block), params, lds_bytes, stream);
}

// Multi-stage launch: every workgroup of the grid must be resident at once (tiles wait on
// their neighbours' progress), which the cooperative launch guarantees or refuses.
hipError_t launch_stage_fused(bool fp64, const StageArgs &a, int max_blocks, size_t lds_bytes, int block,
                              bool cooperative, hipStream_t stream) {
  if (a.ntiles <= 0) return hipSuccess;
  const int grid = stage_grid(a.ntiles, max_blocks);
  StageArgs arg = a;
  void *params[] = {&arg};
  const void *fn = stage_fn(fp64, a.contraction, a.wadg != 0, true, a.v1 != 0, a.kind, a.tile);
  if (cooperative) return hipLaunchCooperativeKernel(fn, dim3(grid), dim3(block), params, lds_bytes, stream);
  return hipLaunchKernel(fn, dim3(grid), dim3(block), params, lds_bytes, stream);
}

hipError_t launch_diag(bool fp64, const DiagArgs &a, hipStream_t stream) {
  if (a.ntiles <= 0) return hipSuccess;
  if (fp64)
    hipLaunchKernelGGL(diag_kernel<double>, dim3(a.ntiles), dim3(kBlock), 0, stream, a);
  else
    hipLaunchKernelGGL(diag_kernel<float>, dim3(a.ntiles), dim3(kBlock), 0, stream, a);
  return hipGetLastError();
}

// Rest depth of the tiles a.tiles[0 .. a.ntiles) (one instance's) into their static blocks.
hipError_t launch_rest_depth(bool fp64, const DiagArgs &a, hipStream_t stream) {
  if (a.ntiles <= 0) return hipSuccess;
  if (fp64)
    hipLaunchKernelGGL(rest_depth_kernel<double>, dim3(a.ntiles), dim3(kBlock), 0, stream, a);
  else
    hipLaunchKernelGGL(rest_depth_kernel<float>, dim3(a.ntiles), dim3(kBlock), 0, stream, a);
  return hipGetLastError();
}

#endif  // ESDG_UNIT_HOST

}  // namespace esdg
