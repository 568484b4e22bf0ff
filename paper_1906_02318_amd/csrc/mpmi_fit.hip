// Koopman fit in FP64 (Sec. IV-A: the model is learned from transition data;
// least squares as in extended DMD).  Three launches:
//   1. gram:   every workgroup lifts tiles of 64 rows into LDS (psi computed on
//              the fly, never materialised in HBM) and accumulates its share
//              of Z^T Z restricted to the first D rows, Z = [Psi | targets], in
//              16 x 16 blocks on the FP64 matrix cores, one or two waves
//              lifting the next tile while the others accumulate;
//   2. reduce: partial sums added in a fixed order (deterministic);
//   3. solve:  RMS column scaling, ridge, blocked Cholesky of the scaled Gram
//              matrix, the triangular solves of all right-hand sides at once
//              and unscaling, and the extreme eigenvalues (power iteration
//              on the Gram matrix and on its inverse) for
//              the condition number.
#include <hip/hip_runtime.h>

#include "mpmi_launch.hpp"

namespace mpmi {

constexpr int kFitRows = 64;       // rows per LDS tile
constexpr int kFitBlocks = 256;    // maximum partial-sum workgroups
constexpr int kFitThreads = 256;  // the solve kernel: four waves share its block products
static_assert(kFitThreads == 4 * 64 && kFitThreads == 4 * MPMI_MAX_DIM, "solve_kernel's work split");

static_assert(MPMI_MAX_STATE <= 16, "the state's target columns are one 16-column block");

// psi(x, u) of one transition in FP64, the FP32 path's feature order,
// written to z (an LDS row) from the row's state xr[n] and input ur[m].  The
// fixed bases take their atoms into registers by constant index.
// Atom q of a custom basis at w = [xr; ur], FP64.
__device__ __forceinline__ double custom_atom(const mpmi_system& sys, int q, const double* __restrict__ xr,
                                              const double* __restrict__ ur) {
  const int kd = sys.atom_kind[q], v = sys.atom_var[q];
  const double w = v < sys.n_state ? xr[v] : ur[v - sys.n_state];
  if (kd == MPMI_ATOM_VAR) return w;
  if (kd == MPMI_ATOM_SIN) return sin(w);
  if (kd == MPMI_ATOM_COS) return cos(w);
  return 1.0;
}

// HALF 0 writes the features without a sine or cosine (custom bases: the
// first half), HALF 1 the others: two waves lift a tile.  The sine and cosine
// of an angle come from one call.
template <int HALF>
__device__ __forceinline__ void lift_row(const mpmi_system& sys, const double* __restrict__ xr,
                                         const double* __restrict__ ur, double* z) {
  const int basis = sys.basis, n = sys.n_state, m = sys.n_input;
  if (basis == MPMI_BASIS_CUSTOM) {
    const int mid = sys.dim / 2;
    for (int f = HALF ? mid : 0; f < (HALF ? sys.dim : mid); ++f)
      z[f] = custom_atom(sys, sys.feat_a[f], xr, ur) * custom_atom(sys, sys.feat_b[f], xr, ur);
    return;
  }
  if (basis == MPMI_BASIS_LINEAR) {
    if constexpr (HALF == 0) {
      for (int k = 0; k < n; ++k) z[k] = xr[k];
      for (int k = 0; k < m; ++k) z[n + k] = ur[k];
    }
    return;
  }
  if (basis == MPMI_BASIS_BALANCE_BOT) {
    if constexpr (HALF == 0) {
      const double w[5] = {xr[0], xr[1], xr[2], xr[3], ur[0]};
      int f = 0;
      z[f++] = 1.0;
#pragma unroll
      for (int k = 0; k < 5; ++k) z[f++] = w[k];
#pragma unroll
      for (int k = 0; k < 5; ++k)
#pragma unroll
        for (int l = k; l < 5; ++l) z[f++] = w[k] * w[l];
    }
    return;
  }
  if constexpr (HALF == 0) {
    const double w[8] = {xr[0], xr[1], xr[2], xr[3], xr[4], xr[5], ur[0], ur[1]};
    int f = 0;
    z[f++] = 1.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) z[f++] = w[k];
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
      for (int l = k; l < 8; ++l) z[f++] = w[k] * w[l];
  } else {
    int f = 45;
    double sp, cp, sd, cd;
    sincos(xr[2], &sp, &cp);
    sincos(ur[0], &sd, &cd);
    const double vx = xr[3], vy = xr[4], r = xr[5], a = ur[1];
    z[f++] = sp; z[f++] = cp; z[f++] = sd; z[f++] = cd;
    z[f++] = sp * vx; z[f++] = sp * vy; z[f++] = sp * r; z[f++] = sp * a;
    z[f++] = cp * vx; z[f++] = cp * vy; z[f++] = cp * r; z[f++] = cp * a;
    z[f++] = sd * vx; z[f++] = sd * vy; z[f++] = sd * r;
    z[f++] = cd * vx; z[f++] = cd * vy; z[f++] = cd * r;
    z[f++] = a * sd;
  }
}

// Accumulation on v_mfma_f64_16x16x4f64.  A tile of 64 rows of Z = [Psi | RHS]
// sits in LDS as 16-column blocks (Psi padded with zero columns to PB
// blocks, the right-hand sides to RB); an MFMA k-step takes four rows, and its
// A and B operands are the same read of a column block (lane l: row l / 16,
// column l % 16).  On gfx950 the instruction is a chain of four FMAs in k order
// (measured: 51,200 results of operands of mixed magnitude, none different),
// so every entry sums the rows in their order, one rounding each, exactly as a
// scalar FMA loop does.  Only the blocks on and above the diagonal of
// Psi' Psi are formed (a product commutes, so the mirrored entry has the same
// bits).  MFMA and vector FP64 run at the same rate here; what the MFMA saves
// is LDS reads: at most two 8-byte reads per 16 FMAs of a lane against 10 per
// 24 for a 4 x 6 register block, which bound the kernel before.  MW waves share
// the blocks and LW waves lift the next tile meanwhile (waves 0 and 1: Psi;
// waves 2 and 3 of the lifted operator: its right-hand sides); the row stride
// is odd, so a wave's writes of one feature use every bank.  The times
// stand at fit_columns.
constexpr int kPsiBlocks = MPMI_MAX_DIM / 16;  // 4
static_assert(MPMI_MAX_DIM == 64, "four 16-column blocks of features");
static_assert(kFitRows == 64, "a lifting wave takes one row per lane");

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// Lane l's element of column block cb of the four rows of k-step ks: both the
// A operand (row = feature) and the B operand (column) of the Gram products.
template <int STRIDE>
__device__ __forceinline__ double gram_frag(const double (*Z)[STRIDE], int ks, int cb, int lane) {
  return Z[4 * ks + (lane >> 4)][16 * cb + (lane & 15)];
}

// Right-hand sides: ny columns, either Y itself (LIFTED false; ny = n <= 8)
// or, for the lifted operator, the ny = D features psi(Y_t, U_t) (the input
// held over the step), lifted on the fly like the rows of Psi.
// PB: column blocks of Psi, as many as its features fill (one, two or four).  With four for every
// basis the products of zeros bound small ones: 3 features of [x; u], 2,000,000
// rows, 620 us and the lifted operator 792 (592 both by scalar FMAs), now 302 and
// 248; the balance bot's 21 557 and 705, now 385 and 311.
template <bool LIFTED, int PB>
struct GramShape {
  static constexpr int RB = LIFTED ? PB : 1;              // right-hand-side blocks
  static constexpr int kGram = PB * (PB + 1) / 2;         // blocks on and above the diagonal
  static constexpr int kTiles = kGram + PB * RB;
  static constexpr int MW = PB == 1 ? 2 : LIFTED ? 8 : 4;  // waves on the products
  static constexpr int LW = LIFTED ? 4 : 2;               // waves lifting
  static constexpr int kPerWave = (kTiles + MW - 1) / MW;
  static constexpr int kStride = 16 * (PB + RB) + 1;
  static constexpr int kThreads = 64 * (MW + LW);
};

template <bool LIFTED, int PB>
__global__ void __launch_bounds__((GramShape<LIFTED, PB>::kThreads))
gram_kernel(mpmi_system sys, int D, int ny, const double* __restrict__ X, const double* __restrict__ U,
            const double* __restrict__ Y, long long T, double* __restrict__ part) {
  using GS = GramShape<LIFTED, PB>;
  __shared__ __attribute__((aligned(16))) double Z[2][kFitRows][GS::kStride];
  const int n = sys.n_state, m = sys.n_input;
  const int C = D + ny;
  const int E = D * C;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool lifter = wave < GS::LW;
  const int mw = wave - GS::LW;
  // This wave's blocks: number q is (I, J), J < PB a feature block (I <= J, in
  // column order), J >= PB right-hand-side block J - PB.
  f64x4_t acc[GS::kPerWave];
  int bi[GS::kPerWave], bj[GS::kPerWave];
  bool on[GS::kPerWave];
#pragma unroll
  for (int k = 0; k < GS::kPerWave; ++k) {
    // A wave with fewer blocks repeats block 0 and drops it: no branch stands
    // between the products and their LDS reads.
    const int q0 = mw + GS::MW * k, q = q0 < 0 || q0 >= GS::kTiles ? 0 : q0;
    int i, j;
    if (q < GS::kGram) {
      j = q < 1 ? 0 : (q < 3 ? 1 : (q < 6 ? 2 : 3));
      i = q - j * (j + 1) / 2;
    } else {
      i = (q - GS::kGram) % PB;
      j = PB + (q - GS::kGram) / PB;
    }
    bi[k] = i;
    bj[k] = j;
    on[k] = !lifter && q == q0;
    acc[k] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  }
  const long long ntiles = (T + kFitRows - 1) / kFitRows;
  // This workgroup's tiles: blockIdx.x + k * gridDim.x, k = 0 .. count - 1.
  const long long count = blockIdx.x < ntiles ? (ntiles - 1 - blockIdx.x) / gridDim.x + 1 : 0;
  auto lift_tile = [&](long long k, int buf) {
    const long long r = (blockIdx.x + k * gridDim.x) * kFitRows + lane;
    double* z = Z[buf][lane];
    double* y = z + 16 * PB;
    if (r >= T) {
      for (int q = wave; q < GS::kStride - 1; q += GS::LW) z[q] = 0.0;
      return;
    }
    if (wave == 0) {
      lift_row<0>(sys, X + r * n, U + r * m, z);
      for (int q = D; q < 16 * PB; ++q) z[q] = 0.0;
      if constexpr (!LIFTED) {
        for (int q = 0; q < ny; ++q) y[q] = Y[r * n + q];
        for (int q = ny; q < 16 * GS::RB; ++q) y[q] = 0.0;
      }
    } else if (wave == 1) {
      lift_row<1>(sys, X + r * n, U + r * m, z);
    } else if (wave == 2) {
      lift_row<0>(sys, Y + r * n, U + r * m, y);
      for (int q = D; q < 16 * GS::RB; ++q) y[q] = 0.0;
    } else {
      lift_row<1>(sys, Y + r * n, U + r * m, y);
    }
  };
  if (lifter && count > 0) lift_tile(0, 0);
  __syncthreads();
  for (long long k = 0; k < count; ++k) {
    if (lifter) {
      if (k + 1 < count) lift_tile(k + 1, (int)((k + 1) & 1));
    } else {
      const double(*z)[GS::kStride] = Z[(int)(k & 1)];
      // The next k-step's operands are read before this one's products; the
      // scheduling barrier keeps the reads there (left to itself the compiler
      // reads each pair just before its product and waits for it).
      double fa[2][GS::kPerWave], fb[2][GS::kPerWave];
#pragma unroll
      for (int q = 0; q < GS::kPerWave; ++q) {
        fa[0][q] = gram_frag<GS::kStride>(z, 0, bi[q], lane);
        fb[0][q] = gram_frag<GS::kStride>(z, 0, bj[q], lane);
      }
#pragma unroll
      for (int ks = 0; ks < kFitRows / 4; ++ks) {
        const int cur = ks & 1;
        if (ks + 1 < kFitRows / 4)
#pragma unroll
          for (int q = 0; q < GS::kPerWave; ++q) {
            fa[cur ^ 1][q] = gram_frag<GS::kStride>(z, ks + 1, bi[q], lane);
            fb[cur ^ 1][q] = gram_frag<GS::kStride>(z, ks + 1, bj[q], lane);
          }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < GS::kPerWave; ++q)
          acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[cur][q], fb[cur][q], acc[q], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
  }
  if (lifter) return;
  // Result layout: lane l holds column l % 16 of rows 4 r + l / 16.
  double* out = part + (size_t)blockIdx.x * E;
#pragma unroll
  for (int q = 0; q < GS::kPerWave; ++q) {
    if (!on[q]) continue;
    const bool rhs = bj[q] >= PB;
    const int col = 16 * (bj[q] - (rhs ? PB : 0)) + (lane & 15);
    if (col >= (rhs ? ny : D)) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * bi[q] + 4 * r + (lane >> 4);
      if (row >= D) continue;
      out[row * C + (rhs ? D + col : col)] = acc[q][r];
      if (!rhs && bi[q] != bj[q]) out[col * C + row] = acc[q][r];
    }
  }
}

// tot[e] = sum over the parts of part[p][e], in a fixed order: the
// kReduceWays threads of element e sum parts p = q, q + kReduceWays, ...
// (q = 0 .. kReduceWays - 1), then one of them adds the partial sums in q
// order.  A workgroup covers kReduceElems elements (lanes of one q read
// consecutive elements); the grid spreads the ~4,500 elements of the race
// car over ~280 workgroups.
constexpr int kReduceElems = 16, kReduceWays = 16;
__global__ void __launch_bounds__(kReduceElems * kReduceWays)
reduce_kernel(int nparts, int E, const double* __restrict__ part, double* __restrict__ tot) {
  __shared__ double qs[kReduceWays][kReduceElems];
  const int el = threadIdx.x % kReduceElems, q = threadIdx.x / kReduceElems;
  const int e = blockIdx.x * kReduceElems + el;
  double s = 0.0;
  if (e < E) {
#pragma unroll 4
    for (int p = q; p < nparts; p += kReduceWays) s += part[(size_t)p * E + e];
  }
  qs[q][el] = s;
  __syncthreads();
  if (q == 0 && e < E) {
    double t = qs[0][el];
#pragma unroll
    for (int k = 1; k < kReduceWays; ++k) t += qs[k][el];
    tot[e] = t;
  }
}

// Value of x in lane k (k wave-uniform), to every lane of the wave.
__device__ __forceinline__ double lane_bcast(double x, int k) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, k);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), k);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// ---------------------------------------------------------------------------
// The solve: 64 x 64 matrices in LDS as 16-wide panels.  Inside a panel the
// 16 steps run in one wave's registers; everything a panel does to the rest of
// a matrix is a product of 16-wide blocks on v_mfma_f64_16x16x4f64.  That
// instruction adds its four products in k order with one rounding each (see
// the Gram kernel), so a blocked factorisation or substitution gives every
// entry the same FMAs in the same order as the step-by-step loop.
//
// Two workgroups run side by side: workgroup 0 factors, solves and estimates
// the least eigenvalue, workgroup 1 the largest.  One workgroup took 92 us
// (race car, D = 64): the factorisation 27 (a barrier per two columns), the
// inverse of the factor 22, its product 6, and twice 60 serial steps of power
// iteration, 28 and 24.  Its bound is the serial chain of 64 pivots, not
// arithmetic: all of its products are ~2 MFLOP.
// ---------------------------------------------------------------------------
constexpr int kMs = MPMI_MAX_DIM + 2;  // LDS row stride of a 64 x 64 matrix
typedef double MatRow[kMs];

// One 16 x 16 block acc += A B over 4 NS k-steps of four: a(i, k) the value of
// lane (row i, k), b(k, j) that of lane (k, column j).  The operands of four
// k-steps are read before their products, the next four meanwhile.
template <int NS, class FA, class FB>
__device__ __forceinline__ f64x4_t block_fma(f64x4_t acc, FA a, FB b) {
  const int lane = threadIdx.x & 63, k0 = lane >> 4, ij = lane & 15;
  double fa[2][4], fb[2][4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    fa[0][q] = a(ij, 4 * q + k0);
    fb[0][q] = b(4 * q + k0, ij);
  }
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    if (s + 1 < NS)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        fa[(s + 1) & 1][q] = a(ij, 16 * (s + 1) + 4 * q + k0);
        fb[(s + 1) & 1][q] = b(16 * (s + 1) + 4 * q + k0, ij);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[s & 1][q], fb[s & 1][q], acc, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
  return acc;
}

// Cholesky of the D x D matrix in A (lower triangle), right-looking in panels
// of 16 columns.  With c_k column k before its own step and d_k its pivot,
// step k subtracts c_ik (c_jk / d_k) from every entry (i, j) with i >= j > k;
// the columns stay unscaled (c_k below the diagonal, pivots in piv[]).  Wave
// 0 holds a panel as one row per lane; step k's multipliers reach the panel's
// other columns by lane broadcast, and Tp[j][k] keeps them for the block
// products.  Called by the whole workgroup (four waves).
__device__ __forceinline__ void factor(MatRow* A, double (*Tp)[18], double* piv, int D, double pivot_floor, int* bad) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int p = 0; 16 * p < D; ++p) {
    const int c0 = 16 * p;
    if (wave == 0) {
      double a[16], pv = 1.0;
      bool low = false;
#pragma unroll
      for (int k = 0; k < 16; ++k) a[k] = A[lane][c0 + k];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        // A pivot below the floor marks the fit singular and is replaced by 1
        // (so is a column past D: all zero, its multipliers stay zero).
        double d = lane_bcast(a[k], c0 + k);
        const bool ok = d > pivot_floor;
        low |= !ok & (c0 + k < D);
        d = ok ? d : 1.0;
        pv = lane == c0 + k ? d : pv;
        // 1 / d: the hardware estimate and two Newton steps (d > 0, normal).
        double rd = __builtin_amdgcn_rcp(d);
        rd = fma(rd, fma(-d, rd, 1.0), rd);
        rd = fma(rd, fma(-d, rd, 1.0), rd);
        const double t = a[k] * rd;
#pragma unroll
        for (int j = k + 1; j < 16; ++j) a[j] = fma(-a[k], lane_bcast(t, c0 + j), a[j]);
        Tp[lane][k] = t;
      }
#pragma unroll
      for (int k = 0; k < 16; ++k) A[lane][c0 + k] = a[k];
      if (lane >= c0 && lane < c0 + 16) piv[lane] = pv;
      if (low && lane == 0) *bad = 1;
    }
    __syncthreads();
    // Blocks (I, J), I >= J > p, spread over the waves.
    int q = 0;
    for (int J = p + 1; J < 4; ++J)
      for (int I = J; I < 4; ++I, ++q) {
        if ((q & 3) != wave || 16 * I >= D) continue;
        f64x4_t acc;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = A[16 * I + 4 * r + (lane >> 4)][16 * J + (lane & 15)];
        acc = block_fma<1>(acc, [&](int i, int k) { return -A[16 * I + i][c0 + k]; },
                        [&](int k, int j) { return Tp[16 * J + j][k]; });
#pragma unroll
        for (int r = 0; r < 4; ++r) A[16 * I + 4 * r + (lane >> 4)][16 * J + (lane & 15)] = acc[r];
      }
    __syncthreads();
  }
}

// One step of a DPP sum over a quad: x plus the lane CTRL selects.
template <int CTRL>
__device__ __forceinline__ double quad_add(double x) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)b, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
  return x + __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// The Rayleigh quotient (w . v) / (v . v), w = A v, of the last of 60 steps of
// power iteration from v0 on the symmetric matrix in M (zero past D).  Four
// lanes hold a row, 16 columns each in registers; the iterate goes from one
// LDS buffer to the other, so a step is eight broadcast reads, 16 FMAs, a quad
// sum and one barrier.  M is taken times the power of two that brings its
// trace, which bounds its eigenvalues, into [1, 2) (exact; the quotient scales
// with it): the iterate shrinks by at most 2^-6 a step along the leading
// eigenvector and needs no normalisation.  Called by the whole workgroup; the
// same value in every thread.
__device__ __forceinline__ double power_rayleigh(const MatRow* M, double v0, double (*v)[MPMI_MAX_DIM]) {
  const int t = threadIdx.x, lane = t & 63, row = t >> 2, c = 16 * (t & 3);
  double tr = M[lane][lane];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) tr += __shfl_xor(tr, o, 64);
  const int e = tr > 0.0 && tr < 1e300 ? ilogb(tr) : 0;
  const double sc = ldexp(1.0, -e);
  double m[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) m[k] = M[row][c + k] * sc;
  if (t < MPMI_MAX_DIM) v[0][t] = v0;
  __syncthreads();
  for (int it = 0; it < 60; ++it) {
    const double* x = v[it & 1] + c;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
    for (int k = 0; k < 16; k += 4) {
      s0 = fma(m[k], x[k], s0);
      s1 = fma(m[k + 1], x[k + 1], s1);
      s2 = fma(m[k + 2], x[k + 2], s2);
      s3 = fma(m[k + 3], x[k + 3], s3);
    }
    const double s = quad_add<0x4E>(quad_add<0xB1>((s0 + s1) + (s2 + s3)));  // lanes xor 1, then xor 2
    if ((t & 3) == 0) v[(it + 1) & 1][row] = s;
    __syncthreads();
  }
  // v[1] holds the iterate before the last step, v[0] the last product.
  double a = v[1][lane] * v[0][lane], b = v[1][lane] * v[1][lane];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, 64);
    b += __shfl_xor(b, o, 64);
  }
  return ldexp(a / b, e);
}

// tot holds [D][C]: G = columns 0..D-1, A = columns D..D+ny-1.  RB: 16-column
// blocks of right-hand sides (ny <= 16 RB).  K [D][ny].
template <int RB>
__global__ void __launch_bounds__(kFitThreads)
solve_kernel(int ny, int D, long long T, double ridge, const double* __restrict__ tot, double* __restrict__ K,
             FitInfo* __restrict__ info) {
  constexpr int kXs = 16 * RB + MPMI_MAX_DIM + 2;  // right-hand sides, then the identity
  __shared__ __attribute__((aligned(16))) double A[MPMI_MAX_DIM][kMs];   // G_s, then the factor
  __shared__ __attribute__((aligned(16))) double X[MPMI_MAX_DIM][kXs];
  __shared__ __attribute__((aligned(16))) double M[MPMI_MAX_DIM][kMs];   // G_s^-1 (workgroup 1: G_s)
  __shared__ double Tp[MPMI_MAX_DIM][18];
  __shared__ double sc[MPMI_MAX_DIM], rinv[MPMI_MAX_DIM], piv[MPMI_MAX_DIM];
  __shared__ __attribute__((aligned(16))) double vv[2][MPMI_MAX_DIM];
  __shared__ int bad;
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int C = D + ny;
  // Loads use clamped (valid) indices so that none waits behind a branch, and
  // all are issued before the scale factors are formed.
  constexpr int kRowsPerWave = MPMI_MAX_DIM / 4;
  double a[kRowsPerWave];
  const int jc = min(lane, D - 1);
#pragma unroll
  for (int r = 0; r < kRowsPerWave; ++r) a[r] = tot[(size_t)min(wave + 4 * r, D - 1) * C + jc];
  constexpr int kRhs = 4 * RB;  // right-hand-side entries per thread
  double b[kRhs];
#pragma unroll
  for (int r = 0; r < kRhs; ++r) {
    const int i = (t + kFitThreads * r) / (16 * RB), j = (t + kFitThreads * r) % (16 * RB);
    b[r] = tot[(size_t)min(i, D - 1) * C + D + min(j, ny - 1)];
  }
  if (t == 0) bad = 0;
  if (t < MPMI_MAX_DIM) {
    const double g = tot[(size_t)jc * C + jc];
    const double s = sqrt(g / (double)T);
    sc[t] = s > 0.0 ? s : 1.0;
    piv[t] = 1.0;
  }
  __syncthreads();
  MatRow* const Gs = blockIdx.x == 0 ? A : M;
#pragma unroll
  for (int r = 0; r < kRowsPerWave; ++r) {
    const int i = wave + 4 * r;
    Gs[i][lane] = (i < D && lane < D) ? a[r] / (sc[i] * sc[lane]) + (i == lane ? ridge : 0.0) : 0.0;
  }
  if (blockIdx.x != 0) {
    __syncthreads();
    const double lmax = power_rayleigh(M, t < D ? 1.0 + 0.01 * t : 0.0, vv);
    if (t == 0) info->lmax = lmax;
    return;
  }
#pragma unroll
  for (int r = 0; r < kRhs; ++r) {
    const int i = (t + kFitThreads * r) / (16 * RB), j = (t + kFitThreads * r) % (16 * RB);
    X[i][j] = (i < D && j < ny) ? b[r] / sc[i] : 0.0;
  }
#pragma unroll
  for (int r = 0; r < kRowsPerWave; ++r) X[wave + 4 * r][16 * RB + lane] = wave + 4 * r == lane ? 1.0 : 0.0;
  __syncthreads();
  factor(A, Tp, piv, D, 1e-14 * (double)T, &bad);
  // The columns scaled into the factor: L_ik = c_i / sqrt(d_k), L_kk = sqrt(d_k).
  {
    const double lkk = sqrt(piv[lane]), rs = 1.0 / lkk;
#pragma unroll
    for (int r = 0; r < kRowsPerWave; ++r) {
      const int i = wave + 4 * r;
      const double v = A[i][lane];
      A[i][lane] = (i < D && lane <= i) ? (i == lane ? lkk : v * rs) : 0.0;
    }
    if (wave == 0) rinv[lane] = lane < D ? rs : 0.0;
  }
  __syncthreads();
  // Forward substitution L Z = [B | I], in place, a panel of 16 rows at a time:
  // one column per lane inside the panel (wave w: columns 64 w ..), then
  // block products for the rows below.
  constexpr int kCols = 16 * RB + MPMI_MAX_DIM, kColBlocks = kCols / 16;
  for (int p = 0; p < 4; ++p) {
    const int c0 = 16 * p;
    if (t < kCols) {
      // The panel's diagonal block, a row in each of lanes 0 .. 15, is read
      // by lane broadcast.
      double x[16], l[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        x[k] = X[c0 + k][t];
        l[k] = A[c0 + (lane & 15)][c0 + k];
      }
      const double ri = rinv[c0 + (lane & 15)];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        x[k] *= lane_bcast(ri, k);
#pragma unroll
        for (int i = k + 1; i < 16; ++i) x[i] = fma(-lane_bcast(l[k], i), x[k], x[i]);
      }
#pragma unroll
      for (int k = 0; k < 16; ++k) X[c0 + k][t] = x[k];
    }
    __syncthreads();
    for (int q = wave; q < (3 - p) * kColBlocks; q += 4) {
      const int I = p + 1 + q / kColBlocks, J = q % kColBlocks;
      f64x4_t acc;
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] = X[16 * I + 4 * r + (lane >> 4)][16 * J + (lane & 15)];
      acc = block_fma<1>(acc, [&](int i, int k) { return -A[16 * I + i][c0 + k]; },
                      [&](int k, int j) { return X[c0 + k][16 * J + j]; });
#pragma unroll
      for (int r = 0; r < 4; ++r) X[16 * I + 4 * r + (lane >> 4)][16 * J + (lane & 15)] = acc[r];
    }
    __syncthreads();
  }
  // G_s^-1 = L^-T L^-1 (the smallest eigenvalue of G_s is 1 / its largest):
  // block (I, J), I <= J, sums over rows k >= 16 J, L^-1 being zero above its
  // diagonal.
  {
    int q = 0;
    for (int J = 0; J < 4; ++J)
      for (int I = 0; I <= J; ++I, ++q) {
        if ((q & 3) != wave) continue;
        f64x4_t acc{0.0, 0.0, 0.0, 0.0};
        for (int k0 = 16 * J; k0 < MPMI_MAX_DIM; k0 += 16)
          acc = block_fma<1>(acc, [&](int i, int k) { return X[k0 + k][16 * RB + 16 * I + i]; },
                             [&](int k, int j) { return X[k0 + k][16 * RB + 16 * J + j]; });
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * I + 4 * r + (lane >> 4), col = 16 * J + (lane & 15);
          const bool in = row < D && col < D;
          M[row][col] = in ? acc[r] : 0.0;
          M[col][row] = in ? acc[r] : 0.0;
        }
      }
  }
  // Backward substitution L^T Y = Z on the right-hand sides, rows from the
  // last up.
  for (int p = 3; p >= 0; --p) {
    const int c0 = 16 * p;
    if (t < 16 * RB) {
      double x[16], l[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        x[k] = X[c0 + k][t];
        l[k] = A[c0 + (lane & 15)][c0 + k];
      }
      const double ri = rinv[c0 + (lane & 15)];
#pragma unroll
      for (int k = 15; k >= 0; --k) {
        x[k] *= lane_bcast(ri, k);
#pragma unroll
        for (int i = 0; i < k; ++i) x[i] = fma(-lane_bcast(l[i], k), x[k], x[i]);
      }
#pragma unroll
      for (int k = 0; k < 16; ++k) X[c0 + k][t] = x[k];
    }
    __syncthreads();
    for (int q = wave; q < p * RB; q += 4) {
      const int I = q / RB, J = q % RB;
      f64x4_t acc;
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] = X[16 * I + 4 * r + (lane >> 4)][16 * J + (lane & 15)];
      // k-steps from the panel's last row up: the order of a step-by-step loop
      acc = block_fma<1>(acc, [&](int i, int k) { return -A[c0 + 15 - k][16 * I + i]; },
                      [&](int k, int j) { return X[c0 + 15 - k][16 * J + j]; });
#pragma unroll
      for (int r = 0; r < 4; ++r) X[16 * I + 4 * r + (lane >> 4)][16 * J + (lane & 15)] = acc[r];
    }
    __syncthreads();
  }
  for (int e = t; e < D * ny; e += kFitThreads) {
    const int i = e / ny, j = e % ny;
    K[e] = X[i][j] / sc[i];
  }
  __syncthreads();
  const double lmin_inv = power_rayleigh(M, t < D ? 1.0 - 0.01 * t : 0.0, vv);
  if (t == 0) {
    info->status = bad ? MPMI_ESINGULAR : MPMI_OK;
    info->lmin_inv = lmin_inv;
  }
}

// Workspace: partial sums, then totals.
constexpr int kFitColsMax = 2 * MPMI_MAX_DIM;  // the lifted operator's D + D columns
size_t fit_workspace_bytes() { return (size_t)(kFitBlocks + 1) * MPMI_MAX_DIM * kFitColsMax * sizeof(double); }

// One least-squares solve: targets Y (ny = n), or psi(Y, U) for the lifted
// operator (ny = dim).  Race car, T = 50,000, one MI355X: Gram 22 us (29 with
// 4 x 6 vector blocks and one lifting wave), reduction 4.5, solve 45 (91);
// lifted operator 30 + 4.5 + 50 us (eight rounds of 29 + 4.6 + 91 when it was
// solved eight columns at a time).  The Gram pass is bound by the lift of a
// tile (two waves, 3.7 us against 2.3 us of products); 256 workgroups fix the
// order of the sums.
template <bool LIFTED, int PB>
static hipError_t fit_columns(const mpmi_system& sys, int dim, int ny, const double* X, const double* U,
                              const double* Y, int64_t T, double ridge, double* K_out, void* work, FitInfo* info,
                              hipStream_t st) {
  const int E = dim * (dim + ny);
  long long ntiles = (T + kFitRows - 1) / kFitRows;
  const int nparts = (int)(ntiles < kFitBlocks ? ntiles : kFitBlocks);
  double* part = (double*)work;
  double* tot = part + (size_t)kFitBlocks * MPMI_MAX_DIM * kFitColsMax;
  using GS = GramShape<LIFTED, PB>;
  gram_kernel<LIFTED, PB><<<nparts, GS::kThreads, 0, st>>>(sys, dim, ny, X, U, Y, (long long)T, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  reduce_kernel<<<(E + kReduceElems - 1) / kReduceElems, kReduceElems * kReduceWays, 0, st>>>(nparts, E, part, tot);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  solve_kernel<GS::RB><<<2, kFitThreads, 0, st>>>(ny, dim, (long long)T, ridge, tot, K_out, info);
  return hipGetLastError();
}

hipError_t launch_fit(const mpmi_system& sys, int dim, const double* X, const double* U, const double* Y,
                      int64_t T, double ridge, double* K_out, void* work, FitInfo* info, hipStream_t st) {
  auto fit = dim <= 16 ? fit_columns<false, 1> : dim <= 32 ? fit_columns<false, 2> : fit_columns<false, kPsiBlocks>;
  return fit(sys, dim, sys.n_state, X, U, Y, T, ridge, K_out, work, info, st);
}

// The lifted operator K (dim x dim, targets psi(Y_t, U_t)): the same scaled
// least-squares problem with dim target columns, in one pass over the data
// and one factorisation.  It was solved eight columns at a time, each chunk
// forming the Gram matrix and its factor again.
hipError_t launch_fit_lifted(const mpmi_system& sys, int dim, const double* X, const double* U, const double* Y,
                             int64_t T, double ridge, double* K_out, void* work, FitInfo* info, hipStream_t st) {
  auto fit = dim <= 16 ? fit_columns<true, 1> : dim <= 32 ? fit_columns<true, 2> : fit_columns<true, kPsiBlocks>;
  return fit(sys, dim, dim, X, U, Y, T, ridge, K_out, work, info, st);
}

}  // namespace mpmi
