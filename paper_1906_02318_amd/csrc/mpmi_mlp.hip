// Learned proposal network: forward, mixture loss, backward, Adam and the
// mixture sampler, all hand-written for gfx950.
//
// Shape (fixed): 8 standardised inputs -> 256 -> 256 -> 256 -> 80, GELU (tanh
// form) on the hidden layers; the 80 outputs are 16 x {logit, mu_0, mu_1,
// log sigma_0, log sigma_1} of a diagonal-Gaussian mixture over the input
// normalised to [-1, 1]^2.  Weights are BF16 (FP32 master copy for Adam);
// every product accumulates in FP32.
//
// The dense products run on BF16 matrix cores.  The forward and the backward
// dX products run layer after layer inside one fused row-block kernel
// (v_mfma_f32_32x32x16_bf16, activations in LDS); the weight-gradient products,
// contractions over the batch, as tiles over parts of it
// (v_mfma_f32_16x16x32_bf16).  A training gradient is four launches: weights
// packed, the fused pass, the weight gradients, the sums of their parts.
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>

#include <algorithm>

#include "mpmi_device.hpp"
#include "mpmi_launch.hpp"

namespace mpmi {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr float kGeluC = 0.7978845608028654f;  // sqrt(2/pi)
constexpr float kGeluA = 0.044715f;

__device__ __forceinline__ uint16_t f2bf(float f) { return (uint16_t)bf16_bits_rne_u(f); }
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ float gelu_f(float z) {
  return 0.5f * z * (1.0f + tanhf(kGeluC * fmaf(kGeluA * z * z, z, z)));
}
struct GemmArgs {
  const uint16_t* A;  // bf16
  const uint16_t* B;  // bf16
  int M, N, K;
  int lda, ldb;
  int ta, tb;          // A(m,k) = ta ? A[k*lda+m] : A[m*lda+k]; B(k,n) = tb ? B[n*ldb+k] : B[k*ldb+n]
  float* out;          // [M][N]
  bool vec_a, vec_b;   // 16-byte loads allowed (leading dimension a multiple of 8, 16-byte aligned base)
};

// C = op(A) op(B) on v_mfma_f32_16x16x32_bf16, a stand-alone product (the
// network's run in mlp_fused_kernel and mlp_dw_kernel).  A 256-thread workgroup owns a
// 64 x 64 tile of C, each wave a 32 x 32 quarter as 2 x 2 MFMA blocks.  Per
// 32-wide k step every thread moves one 16-byte chunk (8 BF16) of A and one
// of B from global memory into LDS, in the operand order the MFMA reads (row
// or column, then k): a chunk along k (row-major A, transposed B) is stored
// as one 16-byte LDS write, a chunk along m or n as eight 2-byte writes.  The
// next stage's chunks (several k steps) are loaded into registers while the
// current stage's MFMAs run (see kGemmSub).  Chunks that
// are contiguous, aligned and wholly inside the matrix take one
// 16-byte load; others (ragged edges, odd leading dimensions) load element by
// element.
constexpr int kGemmKP = 40;  // padded k extent of an LDS row (80 B, keeps 16-B alignment)

struct GemmChunk {
  uint4 a, b;
};

// Eight BF16 values p[0], p[s], ..., p[7 s], those with index >= lim zero,
// packed as a 16-byte chunk; one 16-byte load when all eight are in range
// and contiguous and aligned (vec).
__device__ __forceinline__ uint4 load_chunk(const uint16_t* __restrict__ p, size_t s, int idx, int lim, bool vec) {
  if (vec && idx + 8 <= lim) return *reinterpret_cast<const uint4*>(p);
  uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (idx + i < lim) w[i >> 1] |= (uint32_t)p[(size_t)i * s] << ((i & 1) * 16);
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// This thread's chunks of the k step at k0: A row-major -- row t / 4, k
// (t % 4) * 8 .. +8; A transposed -- k t / 8, rows (t % 8) * 8 .. +8; B
// transposed -- column t / 4, k (t % 4) * 8 .. +8; B row-major -- k t / 8,
// columns (t % 8) * 8 .. +8.  Values outside the matrix (or past kend) are 0.
__device__ __forceinline__ void gemm_load(const GemmArgs& g, int m0, int n0, int k0, int kend, GemmChunk* c) {
  const int t = threadIdx.x;
  c->a = make_uint4(0u, 0u, 0u, 0u);
  c->b = make_uint4(0u, 0u, 0u, 0u);
  if (!g.ta) {
    const int m = m0 + (t >> 2), k = k0 + (t & 3) * 8;
    if (m < g.M && k < kend) c->a = load_chunk(g.A + (size_t)m * g.lda + k, 1, k, kend, g.vec_a);
  } else {
    const int k = k0 + (t >> 3), m = m0 + (t & 7) * 8;
    if (m < g.M && k < kend) c->a = load_chunk(g.A + (size_t)k * g.lda + m, 1, m, g.M, g.vec_a);
  }
  if (g.tb) {
    const int n = n0 + (t >> 2), k = k0 + (t & 3) * 8;
    if (n < g.N && k < kend) c->b = load_chunk(g.B + (size_t)n * g.ldb + k, 1, k, kend, g.vec_b);
  } else {
    const int k = k0 + (t >> 3), n = n0 + (t & 7) * 8;
    if (n < g.N && k < kend) c->b = load_chunk(g.B + (size_t)k * g.ldb + n, 1, n, g.N, g.vec_b);
  }
}

__device__ __forceinline__ void gemm_store(const GemmArgs& g, const GemmChunk& c, uint16_t (*As)[kGemmKP],
                                           uint16_t (*Bs)[kGemmKP]) {
  const int t = threadIdx.x;
  const uint32_t wa[4] = {c.a.x, c.a.y, c.a.z, c.a.w};
  const uint32_t wb[4] = {c.b.x, c.b.y, c.b.z, c.b.w};
  if (!g.ta) {
    *reinterpret_cast<uint4*>(&As[t >> 2][(t & 3) * 8]) = c.a;
  } else {
    const int k = t >> 3, m = (t & 7) * 8;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      As[m + 2 * i][k] = (uint16_t)(wa[i] & 0xffffu);
      As[m + 2 * i + 1][k] = (uint16_t)(wa[i] >> 16);
    }
  }
  if (g.tb) {
    *reinterpret_cast<uint4*>(&Bs[t >> 2][(t & 3) * 8]) = c.b;
  } else {
    const int k = t >> 3, n = (t & 7) * 8;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      Bs[n + 2 * i][k] = (uint16_t)(wb[i] & 0xffffu);
      Bs[n + 2 * i + 1][k] = (uint16_t)(wb[i] >> 16);
    }
  }
}

// A stage is kGemmSub k-steps of 32 (128 values of k): every thread issues
// the loads of the whole next stage (kGemmSub 16-byte chunks of A and of B)
// into registers before the MFMAs of the current one, so a product with
// K = 256 takes two memory round trips instead of eight (a single stage of
// 256, one round trip, measured the same at batch 4,096: launch and epilogue
// latency, not the round trips, bound those products).  One LDS buffer
// (40 KB, several workgroups per CU): the registers are stored into it
// after a barrier that ends the current stage's reads.
constexpr int kGemmSub = 4;

__global__ void __launch_bounds__(256) gemm_bf16_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(16))) uint16_t As[kGemmSub][64][kGemmKP];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[kGemmSub][64][kGemmKP];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64, kend = g.K;
  constexpr int kStage = 32 * kGemmSub;
  f32x4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  GemmChunk c[kGemmSub];
#pragma unroll
  for (int q = 0; q < kGemmSub; ++q) gemm_load(g, m0, n0, 32 * q, kend, &c[q]);
#pragma unroll
  for (int q = 0; q < kGemmSub; ++q) gemm_store(g, c[q], As[q], Bs[q]);
  __syncthreads();
  for (int k0 = 0; k0 < kend; k0 += kStage) {
    const bool more = k0 + kStage < kend;
    if (more) {
#pragma unroll
      for (int q = 0; q < kGemmSub; ++q) gemm_load(g, m0, n0, k0 + kStage + 32 * q, kend, &c[q]);
    }
    const int kq = (lane >> 4) * 8;
#pragma unroll
    for (int q = 0; q < kGemmSub; ++q) {
      if (k0 + 32 * q >= kend) break;  // uniform: a ragged last stage
      bf16x8_t af[2], bfr[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        af[i] = *reinterpret_cast<const bf16x8_t*>(&As[q][wm * 32 + i * 16 + (lane & 15)][kq]);
        bfr[i] = *reinterpret_cast<const bf16x8_t*>(&Bs[q][wn * 32 + i * 16 + (lane & 15)][kq]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
    if (more) {  // uniform
      __syncthreads();  // the stage's reads are done
#pragma unroll
      for (int q = 0; q < kGemmSub; ++q) gemm_store(g, c[q], As[q], Bs[q]);
      __syncthreads();
    }
  }
  // D fragment: lane holds column (lane & 15), rows (lane >> 4) * 4 + r.
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int mb = m0 + wm * 32 + i * 16 + (lane >> 4) * 4;
      const int n = n0 + wn * 32 + j * 16 + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (mb + r < g.M && n < g.N) g.out[(size_t)(mb + r) * g.N + n] = acc[i][j][r];
    }
}

// Max and sum over a 16-lane group (one sample's mixture components), the
// same bits in every lane: DPP rotations by 8, 4, 2 and 1 within the row (after
// each, the values repeat with that period, so a lane adds what its xor
// partner would give it).
template <int CTRL>
__device__ __forceinline__ float row_ror(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float group16_max(float v) {
  v = fmaxf(v, row_ror<0x128>(v));
  v = fmaxf(v, row_ror<0x124>(v));
  v = fmaxf(v, row_ror<0x122>(v));
  return fmaxf(v, row_ror<0x121>(v));
}
__device__ __forceinline__ float group16_sum(float v) {
  v += row_ror<0x128>(v);
  v += row_ror<0x124>(v);
  v += row_ror<0x122>(v);
  return v + row_ror<0x121>(v);
}

// Adam (Kingma & Ba 2015) with bias correction on the FP32 master weights,
// refreshing the BF16 copy used by the products.
__global__ void adam_kernel(float* __restrict__ w, uint16_t* __restrict__ w16, float* __restrict__ mom,
                            float* __restrict__ vel, const float* __restrict__ grad, int n, float lr, float b1,
                            float b2, float omb1, float omb2, float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float g = grad[i];
  const float m = b1 * mom[i] + omb1 * g;
  const float v = b2 * vel[i] + omb2 * g * g;
  mom[i] = m;
  vel[i] = v;
  const float wi = w[i] - lr * (m / c1) / (sqrtf(v / c2) + eps);
  w[i] = wi;
  w16[i] = f2bf(wi);
}

// The mixture of one head in the form the draws use, built once per
// workgroup in LDS: cdf[k] = (sum_{i<=k} e_i) / (sum_i e_i) with e_i =
// exp(logit_i - max logit), summed in component order, and sig = exp of the
// clamped log sigmas.
struct MdnTable {
  float e[kMlpComp], w[kMlpComp], cdf[kMlpComp], sig[kMlpComp][2], acc;
};

// Called by every thread of the workgroup (three barriers); head is readable
// by all of them.
__device__ __forceinline__ void mdn_table_build(const float* head, MdnTable* t) {
  const int j = threadIdx.x;
  if (j < kMlpComp) {
    float lmax = -INFINITY;
    for (int k = 0; k < kMlpComp; ++k) lmax = fmaxf(lmax, head[5 * k]);
    t->e[j] = expf(head[5 * j] - lmax);
  } else if (j < 3 * kMlpComp) {
    const int k = (j - kMlpComp) >> 1, q = (j - kMlpComp) & 1;
    t->sig[k][q] = expf(fminf(fmaxf(head[5 * k + 3 + q], kLogSigMin), kLogSigMax));
  }
  __syncthreads();
  if (j == 0) {
    float acc = 0.0f;
    for (int k = 0; k < kMlpComp; ++k) {
      acc += t->e[k];
      t->w[k] = acc;
    }
    t->acc = acc;
  }
  __syncthreads();
  if (j < kMlpComp) t->cdf[j] = t->w[j] / t->acc;
  __syncthreads();
}

// Proposal p: component by inverse CDF at r0, Box-Muller normals from r1,
// r2, mu + sigma z clipped to [-1, 1], mapped to the input box.  Writes cand
// [1][m][P] (EXPLICIT layout, m = 2).
__device__ __forceinline__ void mdn_draw(const ModelDev* __restrict__ md, const float* head, const MdnTable* t,
                                         int P, int p, uint64_t seed, uint64_t tick, int loop,
                                         float* __restrict__ cand) {
  const uint64_t pre = hash_prefix(seed, tick, (uint64_t)(uint32_t)loop, (uint64_t)p);
  const uint64_t h0 = hash_finish(pre, 0), h1 = hash_finish(pre, 1), h2 = hash_finish(pre, 2);
  const float r0 = (float)((double)(h0 >> 40) * 0x1p-24);
  int kc = 0;
#pragma unroll
  for (int k = 0; k < kMlpComp; ++k) kc += (t->cdf[k] <= r0) ? 1 : 0;
  kc = kc < kMlpComp ? kc : kMlpComp - 1;
  const float r1 = (float)(((double)(h1 >> 40) + 1.0) * 0x1p-24);
  const float r2 = (float)((double)(h2 >> 40) * 0x1p-24);
  const float rad = sqrtf(-2.0f * logf(r1));
  float sn, cs;
  sincosf(6.283185307179586f * r2, &sn, &cs);
  const float z[2] = {rad * cs, rad * sn};
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    float un = fmaf(t->sig[kc][j], z[j], head[5 * kc + 1 + j]);
    un = fminf(fmaxf(un, -1.0f), 1.0f);
    const float lo = md->sys.u_lo[j], hi = md->sys.u_hi[j];
    cand[(size_t)j * P + p] = fmaf(0.5f * (hi - lo), un, 0.5f * (lo + hi));
  }
}

__global__ void __launch_bounds__(256)
mdn_sample_kernel(const ModelDev* __restrict__ md, const float* __restrict__ Yrow, int P, uint64_t seed,
                  uint64_t tick, int loop, float* __restrict__ cand) {
  __shared__ MdnTable tab;
  mdn_table_build(Yrow, &tab);
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < P) mdn_draw(md, Yrow, &tab, P, p, seed, tick, loop, cand);
}

// Offsets of (W_l, b_l) in the flat parameter vector (per layer W[in][out]
// then b[out]), as plain constants: device code must not call a recursive
// function (it would need a call stack of unbounded depth).
constexpr size_t kMlpW0 = 0;
constexpr size_t kMlpB0 = kMlpW0 + (size_t)kMlpIn * kMlpHid;
constexpr size_t kMlpW1 = kMlpB0 + kMlpHid;
constexpr size_t kMlpB1 = kMlpW1 + (size_t)kMlpHid * kMlpHid;
constexpr size_t kMlpW2 = kMlpB1 + kMlpHid;
constexpr size_t kMlpB2 = kMlpW2 + (size_t)kMlpHid * kMlpHid;
constexpr size_t kMlpW3 = kMlpB2 + kMlpHid;
constexpr size_t kMlpB3 = kMlpW3 + (size_t)kMlpHid * kMlpOut;
static_assert(kMlpB3 + kMlpOut == MPMI_MLP_PARAMS, "parameter layout");

// ---------------------------------------------------------------------------
// The fused row-block pass.  A workgroup of 8 waves takes blocks of 32 batch
// rows through every layer with the activations in LDS: the forward pass
// (inputs standardised, three GELU layers, the linear head) and, when
// training, the mixture loss and the three dX products with GELU' straight
// after it, so nothing of the forward pass that only the backward pass reads
// leaves the chip: GELU'(z), formed in FP32 beside GELU(z) from the same
// exponential, stays in the registers of the lane that uses it.
//
// A product is taken transposed, W^T (outputs x K) times the block's
// activations (K x 32 rows) on v_mfma_f32_32x32x16_bf16, wave w forming
// outputs 32 w .. 32 w + 31: a lane then holds one batch row and runs of four
// consecutive outputs, which go to the next layer's row-major LDS buffer as
// 8-byte writes.  The weights stream from L2 straight into the operand
// registers through a ring of six k-steps; a layer's last k-steps load the
// next layer's first ones, and the layers are separated by barriers that wait
// for LDS only (__syncthreads would drain the loads in flight).  The operands
// of the weight-gradient products leave row-major, copied from LDS in 16-byte
// stores.
//
// Bound: at large batches vector arithmetic (~18 instruction slots per
// activation, two of its instructions transcendental) beside the weights each
// block reads from L2 (0.6 MB) and the MFMAs; two workgroups per CU overlap one's
// epilogues with the other's products.  Batch
// 65,536: 106 us for both passes (137 forward + 261 backward when they were two
// kernels, FP32 pre-activations going through memory between them); batch
// 4,096, 128 blocks of one round: 22 us, the latency of a block (18 + 22).
// Vector instructions take 0.6 of its cycles, the MFMAs 0.2.
// ---------------------------------------------------------------------------
typedef float f32x16_t __attribute__((ext_vector_type(16)));
constexpr int kFuseRows = 32;
constexpr int kFuseLd = 264;  // LDS row stride in BF16: 256 + 8, rows 16 B apart in bank order
constexpr int kFuseWaves = 8;
constexpr int kFuseThreads = 64 * kFuseWaves;
static_assert(kMlpHid == 32 * kFuseWaves, "32 outputs per wave");
constexpr int kYLd = 100;  // LDS row stride of the FP32 head (three 32-wide tiles and padding)
constexpr int kHeadWaves = (kMlpOut + 31) / 32;
constexpr int kRing = 6;

// Workgroup barrier over LDS only: waits for this wave's LDS accesses, not
// for its global loads (__syncthreads' fence also drains the vector-memory
// counter, which would retire the weights in flight).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Two FP32 -> two BF16, round to nearest even (v_cvt_pk_bf16_f32), packed.
__device__ __forceinline__ uint32_t cvt2_bf16(float a, float b) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const bf16x2_t v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}

// GELU and its derivative (tanh form) at z.  With s = 1 / (1 + exp(-2 y)) =
// (1 + tanh y) / 2, y = sqrt(2/pi) (z + 0.044715 z^3): GELU = z s and
// GELU' = s + 2 z s (1 - s) y'(z) -- one hardware exponential and one
// reciprocal for both, and no cancellation in 1 + tanh y for negative z.
// The gradient's error against 64 bits is what it was with tanhf (6.5e-5 at
// batch 4,096, 1.8e-5 at 65,536: the BF16 roundings').
__device__ __forceinline__ float gelu_both(float z, float* grad) {
  constexpr float kLog2e = 1.4426950408889634f;
  constexpr float k1 = -2.0f * kGeluC * kLog2e, k3 = k1 * kGeluA;
  constexpr float q0 = 2.0f * kGeluC, q2 = 6.0f * kGeluC * kGeluA;
  const float z2 = z * z;
  const float s = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(z * fmaf(k3, z2, k1)));
  const float zs = z * s;
  *grad = fmaf(fmaf(-zs, s, zs), fmaf(q2, z2, q0), s);
  return zs;
}

// The weights as the products read them.  A product's A operand is cut into
// chunks of 1 KB, chunk (tile w, k-step ks) the 64 lanes' 16 bytes of output
// tile w: lane l holds output 32 w + l % 32, k-values 16 ks + 8 (l / 32) .. + 7.
// Read as they lie in the matrix, those 16 bytes come from 32 rows 512 bytes
// apart and a wave's four k-steps share cache lines that eight waves push out
// of the 32 KB L1 between them: the weights then came from L2 several times
// over (65,536 rows: 172 us; the packed order 110).  Products in the
// order they run: the forward layers 0 .. 2 (A = W^T), the head, and backward
// through layers 3, 2, 1 (A = W).  Entries past a matrix are zero (layer 0 has
// 8 inputs of 16, the head 80 outputs of 96).
constexpr int kProducts = 7;
struct PackedProduct {
  int tiles, ksteps, first;  // first chunk
  int w, din, dout;          // offset and shape of W [din][dout]
  bool fwd;
};
constexpr int kKh = kMlpHid / 16, kKo = kMlpOut / 16;  // k-steps of the hidden and head widths
constexpr PackedProduct kPacked[kProducts] = {
    {kFuseWaves, 1, 0, (int)kMlpW0, kMlpIn, kMlpHid, true},
    {kFuseWaves, kKh, kFuseWaves, (int)kMlpW1, kMlpHid, kMlpHid, true},
    {kFuseWaves, kKh, kFuseWaves * (1 + kKh), (int)kMlpW2, kMlpHid, kMlpHid, true},
    {kHeadWaves, kKh, kFuseWaves * (1 + 2 * kKh), (int)kMlpW3, kMlpHid, kMlpOut, true},
    {kFuseWaves, kKo, kFuseWaves * (1 + 2 * kKh) + kHeadWaves * kKh, (int)kMlpW3, kMlpHid, kMlpOut, false},
    {kFuseWaves, kKh, kFuseWaves * (1 + 2 * kKh + kKo) + kHeadWaves * kKh, (int)kMlpW2, kMlpHid, kMlpHid, false},
    {kFuseWaves, kKh, kFuseWaves * (1 + 3 * kKh + kKo) + kHeadWaves * kKh, (int)kMlpW1, kMlpHid, kMlpHid, false},
};
constexpr int kForwardChunks = kPacked[4].first;
constexpr int kPackedChunks = kPacked[6].first + kFuseWaves * kKh;
constexpr int kChunk = 512;  // BF16 values

// One wave per chunk of the first gridDim.x * 4.  loss_zero (optional) is
// zeroed for the fused pass to accumulate into.
__global__ void __launch_bounds__(256)
mlp_pack_weights_kernel(const uint16_t* __restrict__ w16, uint16_t* __restrict__ packed, float* __restrict__ loss_zero) {
  if (loss_zero && blockIdx.x == 0 && threadIdx.x == 0) *loss_zero = 0.0f;
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (c >= kPackedChunks) return;
#pragma unroll
  for (int q = 0; q < kProducts; ++q) {
    constexpr auto& P = kPacked;
    if (c < P[q].first || c >= P[q].first + P[q].tiles * P[q].ksteps) continue;  // uniform across the wave
    const int tile = (c - P[q].first) / P[q].ksteps, ks = (c - P[q].first) % P[q].ksteps;
    const int o = 32 * tile + (lane & 31), k = 16 * ks + 8 * (lane >> 5);
    const int din = P[q].din, dout = P[q].dout;
    const uint16_t* W = w16 + P[q].w;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (!P[q].fwd) {
      v = *reinterpret_cast<const uint4*>(W + (size_t)o * dout + k);
    } else if (o < dout && k < din) {
      uint32_t w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        w[i] = (uint32_t)W[(size_t)(k + 2 * i) * dout + o] | ((uint32_t)W[(size_t)(k + 2 * i + 1) * dout + o] << 16);
      v = make_uint4(w[0], w[1], w[2], w[3]);
    }
    *reinterpret_cast<uint4*>(packed + (size_t)c * kChunk + 8 * lane) = v;
  }
}

// A wave's chunks of one product: a uniform base and this lane's 16 bytes.
struct Weights {
  const uint16_t* base;
  uint32_t off;
  __device__ __forceinline__ uint4 step(int ks) const {
    return *reinterpret_cast<const uint4*>(base + off + kChunk * ks);
  }
};

// acc += the product of KS k-steps of 16 with the LDS block A (row-major, this
// lane's row).  ring[q % kRing] holds k-step q of the running product; a slot
// whose last use is over takes the next product's k-step of the same number
// (NKS of them, at `next`; none when NKS is 0).
template <int KS, int NKS>
__device__ __forceinline__ f32x16_t stream_product(f32x16_t acc, uint4 (&ring)[kRing], const uint16_t (*A)[kFuseLd],
                                                   Weights cur, Weights next, int lane) {
#pragma unroll
  for (int q = KS; q < kRing; ++q)  // slots this product does not use
    if (q < NKS) ring[q] = next.step(q);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const bf16x8_t b = *reinterpret_cast<const bf16x8_t*>(&A[lane & 31][16 * ks + 8 * (lane >> 5)]);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, ring[ks % kRing]), b, acc, 0, 0, 0);
    if (ks + kRing < KS)
      ring[ks % kRing] = cur.step(ks + kRing);
    else if (ks % kRing < NKS)
      ring[ks % kRing] = next.step(ks % kRing);
  }
  return acc;
}
template <int KS>
__device__ __forceinline__ void ring_fill(uint4 (&ring)[kRing], Weights w) {
#pragma unroll
  for (int q = 0; q < kRing && q < KS; ++q) ring[q] = w.step(q);
}

// Output of accumulator element r of this lane: 8 (r / 4) + 4 (lane / 32) +
// r % 4 within the wave's 32; the lane's batch row is lane % 32.
__device__ __forceinline__ int out_base(int t) { return 32 * (t >> 6) + 4 * ((t >> 5) & 1); }

// Start of a forward product's sum: the biases of this lane's outputs.
__device__ __forceinline__ f32x16_t bias_start(const float* bias, int t) {
  f32x16_t acc;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 b = *reinterpret_cast<const float4*>(bias + out_base(t) + 8 * q);
    acc[4 * q] = b.x; acc[4 * q + 1] = b.y; acc[4 * q + 2] = b.z; acc[4 * q + 3] = b.w;
  }
  return acc;
}
__device__ __forceinline__ f32x16_t zero_start() {
  f32x16_t acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  return acc;
}

// Epilogue of a hidden layer: GELU(z) in BF16 to the next LDS buffer,
// GELU' to g.
template <bool TRAIN>
__device__ __forceinline__ void hidden_epilogue(const f32x16_t& z, uint16_t (*hout)[kFuseLd],
                                                float (&g)[16], int t) {
  const int row = t & 31, n0 = out_base(t);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float h[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float gr = 0.0f;
      h[r] = gelu_both(z[4 * q + r], &gr);
      if (TRAIN) {
        // Formed here: left alone, the compiler moves the derivative to its
        // use, three layers on, and keeps three values for it instead of one.
        asm volatile("" : "+v"(gr));
        g[4 * q + r] = gr;
      }
    }
    *reinterpret_cast<uint2*>(&hout[row][n0 + 8 * q]) = make_uint2(cvt2_bf16(h[0], h[1]), cvt2_bf16(h[2], h[3]));
  }
}

// One halving step of column_sum: lane i and the lane CTRL pairs it with
// exchange half of their N values; `high` lanes keep the upper half.
template <int N, int CTRL>
__device__ __forceinline__ void halve(float (&v)[16], bool high) {
#pragma unroll
  for (int k = 0; k < N / 2; ++k) {
    const float keep = high ? v[N / 2 + k] : v[k], send = high ? v[k] : v[N / 2 + k];
    v[k] = keep + __builtin_bit_cast(
                      float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, send), CTRL, 0xF, 0xF, true));
  }
}
// Sums over the 32 lanes of a half wave of 16 values per lane, in a fixed
// order: lane l returns the sum of value l % 16.  Four exchanges within a row
// of 16 lanes (mirror, half mirror, quad mirror, neighbour), each halving the
// values a lane keeps, then the two rows of the half wave.
__device__ __forceinline__ float column_sum(float (&v)[16], int lane) {
  halve<16, 0x140>(v, (lane & 8) != 0);  // row_mirror
  halve<8, 0x141>(v, (lane & 4) != 0);   // row_half_mirror
  halve<4, 0x1B>(v, (lane & 2) != 0);    // quad_perm 3,2,1,0
  halve<2, 0xB1>(v, (lane & 1) != 0);    // quad_perm 1,0,3,2
  return v[0] + __shfl_xor(v[0], 16);
}

// Epilogue of a dX product: dz = acc GELU' in BF16 to the next LDS buffer
// (zero for rows past the batch, whose gradient of the loss is), and its FP32 column sum over the block
// added to cs (lane l: output out_base(t) + 8 ((l % 16) / 4) + l % 4).
__device__ __forceinline__ void dx_epilogue(const f32x16_t& acc, const float (&g)[16], uint16_t (*dout)[kFuseLd],
                                            float* cs, int t) {
  const int row = t & 31, n0 = out_base(t);
  float v[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = acc[r] * g[r];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *reinterpret_cast<uint2*>(&dout[row][n0 + 8 * q]) =
        make_uint2(cvt2_bf16(v[4 * q], v[4 * q + 1]), cvt2_bf16(v[4 * q + 2], v[4 * q + 3]));
  *cs += column_sum(v, t & 63);
}

// Mixture negative log-likelihood of T under the head ys and its gradient, one
// lane per (sample, component): the 16 lanes of a sample form the two
// log-sum-exps by shuffles within their group.  dNLL/dY / B replaces ys (FP32)
// and goes to ds in BF16; rows past the batch are zero.  Returns the lane's
// share of the block's NLL.
__device__ __forceinline__ float mixture_loss(float (*ys)[kYLd], uint16_t (*ds)[kFuseLd], const float* __restrict__ T,
                                              int r0, int B, float inv_b, int t) {
  static_assert(kMlpComp == 16 && kFuseRows * kMlpComp == kFuseThreads, "one lane per (sample, component)");
  const int sl = t >> 4, k = t & 15;
  const bool valid = r0 + sl < B;  // uniform across each 16-lane group
  const int bb = valid ? r0 + sl : 0;
  float* y = &ys[sl][5 * k];
  const float t0 = T[2 * bb], t1 = T[2 * bb + 1];
  const float logit = y[0], mu0 = y[1], mu1 = y[2], q0 = y[3], q1 = y[4];
  const float lmax0 = group16_max(logit);
  const float lse_logit = lmax0 + logf(group16_sum(expf(logit - lmax0)));
  const float l0 = fminf(fmaxf(q0, kLogSigMin), kLogSigMax);
  const float l1 = fminf(fmaxf(q1, kLogSigMin), kLogSigMax);
  const float is0 = expf(-l0), is1 = expf(-l1);
  const float d0 = (t0 - mu0) * is0;
  const float d1 = (t1 - mu1) * is1;
  const float lp = logit - lse_logit;
  const float a = lp - (0.5f * (d0 * d0 + d1 * d1) + l0 + l1 + kLog2Pi);
  const float amax = group16_max(a);
  const float lse = amax + logf(group16_sum(expf(a - amax)));
  const float gam = expf(a - lse);
  const float pi = expf(lp);
  float gk[5];
  gk[0] = pi - gam;
  gk[1] = -gam * d0 * is0;
  gk[2] = -gam * d1 * is1;
  gk[3] = (q0 > kLogSigMin && q0 < kLogSigMax) ? gam * (1.0f - d0 * d0) : 0.0f;
  gk[4] = (q1 > kLogSigMin && q1 < kLogSigMax) ? gam * (1.0f - d1 * d1) : 0.0f;
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    const float v = valid ? gk[q] * inv_b : 0.0f;
    y[q] = v;
    ds[sl][5 * k + q] = (uint16_t)cvt2_bf16(v, 0.0f);
  }
  return valid && k == 0 ? -lse : 0.0f;
}

// The block's first W columns (a multiple of 8) from LDS to dst [B][W].
template <int W>
__device__ __forceinline__ void store_block(const uint16_t (*a)[kFuseLd], uint16_t* __restrict__ dst, int r0, int B,
                                            int t) {
  constexpr int C = W / 8;
#pragma unroll
  for (int i = 0; i < (kFuseRows * C + kFuseThreads - 1) / kFuseThreads; ++i) {
    const int e = t + i * kFuseThreads, row = e / C, c = e % C;
    if (row < kFuseRows && r0 + row < B)
      *reinterpret_cast<uint4*>(dst + (size_t)(r0 + row) * W + 8 * c) = *reinterpret_cast<const uint4*>(&a[row][8 * c]);
  }
}

// Blocks blockIdx.x, + gridDim.x, ... of 32 rows.  TRAIN false: Y [B][80].
// TRAIN true: the operands of the weight gradients (h_l at h[l], the gradient
// of layer l's output at d[l], row-major), the workgroup's column sums of the
// latter at bsum + (l gridDim.x + blockIdx.x) 256, and its share of the mean
// NLL added into *loss_sum (zeroed by an earlier launch).
struct FusedArgs {
  const uint16_t* packed;  // weights in the products' order
  const float *bias32, *mean, *stdv, *X, *T;
  int B;
  float* Y;
  uint16_t *h[4], *d[4];
  float *bsum, *loss_sum;
};

template <bool TRAIN>
__global__ void __launch_bounds__(kFuseThreads, 4)
mlp_fused_kernel(FusedArgs g) {
  __shared__ __attribute__((aligned(16))) uint16_t hs[2][kFuseRows][kFuseLd];
  __shared__ __attribute__((aligned(16))) float ys[kFuseRows][kYLd];
  __shared__ __attribute__((aligned(16))) float bs[3 * kMlpHid + 32 * kHeadWaves];
  __shared__ float wave_nll[kFuseWaves];
  constexpr int KH = kKh, KO = kKo;
  const int B = g.B;
  for (int e = threadIdx.x; e < 3 * kMlpHid + 32 * kHeadWaves; e += kFuseThreads) {
    const int l = e / kMlpHid, n = e % kMlpHid;
    const size_t off = l == 0 ? kMlpB0 : (l == 1 ? kMlpB1 : (l == 2 ? kMlpB2 : kMlpB3));
    bs[e] = l < 3 || n < kMlpOut ? g.bias32[off + n] : 0.0f;
  }
  float cs1 = 0.0f, cs2 = 0.0f, cs3 = 0.0f, csh = 0.0f, nll = 0.0f;
  uint4 ring[kRing];
  const int nblk = (B + kFuseRows - 1) / kFuseRows;
  for (int blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    // The thread number is made anew for every block: addresses formed from it
    // outside the loop would be held across it in registers the block needs.
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    // Waves past the head's tiles repeat its last one and drop it.
    const bool head = wave < kHeadWaves;
    const int head_wave = min(wave, kHeadWaves - 1);
    auto product = [&](int q, int w) {
      return Weights{g.packed + (size_t)(kPacked[q].first + w * kPacked[q].ksteps) * kChunk, (uint32_t)(8 * lane)};
    };
    const Weights p0 = product(0, wave), p1 = product(1, wave), p2 = product(2, wave), ph = product(3, head_wave);
    const Weights q3 = product(4, wave), q2 = product(5, wave), q1 = product(6, wave);
    const int r0 = blk * kFuseRows;
    ring[0] = p0.step(0);
    // standardised inputs, k 8 .. 15 zero (the first product's k-step)
    {
      const int r = t >> 4, k = t & 15, b = r0 + r;
      uint16_t v = 0;
      if (k < kMlpIn && b < B) v = f2bf((g.X[(size_t)b * kMlpIn + k] - g.mean[k]) / g.stdv[k]);
      hs[0][r][k] = v;
    }
    lds_barrier();
    float g1[16], g2[16], g3[16];
    f32x16_t acc = stream_product<1, KH>(bias_start(bs, t), ring, hs[0], p0, p1, lane);
    if (TRAIN) store_block<kMlpIn>(hs[0], g.h[0], r0, B, t);
    hidden_epilogue<TRAIN>(acc, hs[1], g1, t);
    lds_barrier();
    acc = stream_product<KH, KH>(bias_start(bs + kMlpHid, t), ring, hs[1], p1, p2, lane);
    if (TRAIN) store_block<kMlpHid>(hs[1], g.h[1], r0, B, t);
    hidden_epilogue<TRAIN>(acc, hs[0], g2, t);
    lds_barrier();
    acc = stream_product<KH, KH>(bias_start(bs + 2 * kMlpHid, t), ring, hs[0], p2, ph, lane);
    if (TRAIN) store_block<kMlpHid>(hs[0], g.h[2], r0, B, t);
    hidden_epilogue<TRAIN>(acc, hs[1], g3, t);
    lds_barrier();
    // the head: 80 outputs, linear, FP32 to LDS
    if (head) {
      acc = stream_product<KH, 0>(bias_start(bs + 3 * kMlpHid, t), ring, hs[1], ph, ph, lane);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        *reinterpret_cast<float4*>(&ys[lane & 31][out_base(t) + 8 * q]) =
            make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
      }
    }
    if (TRAIN) {
      ring_fill<KO>(ring, q3);
      store_block<kMlpHid>(hs[1], g.h[3], r0, B, t);
    }
    lds_barrier();
    if constexpr (!TRAIN) {
      for (int e = t; e < kFuseRows * kMlpOut; e += kFuseThreads) {
        const int row = e / kMlpOut, n = e % kMlpOut;
        if (r0 + row < B) g.Y[(size_t)(r0 + row) * kMlpOut + n] = ys[row][n];
      }
      continue;  // the next block writes ys after three more barriers
    }
    nll += mixture_loss(ys, hs[0], g.T, r0, B, 1.0f / (float)B, t);
    lds_barrier();
    acc = stream_product<KO, KH>(zero_start(), ring, hs[0], q3, q2, lane);
    store_block<kMlpOut>(hs[0], g.d[3], r0, B, t);
    if (t < kMlpOut) {  // the head's bias gradient: rows in order
#pragma unroll 4
      for (int r = 0; r < kFuseRows; ++r) csh += ys[r][t];
    }
    dx_epilogue(acc, g3, hs[1], &cs3, t);
    lds_barrier();
    acc = stream_product<KH, KH>(zero_start(), ring, hs[1], q2, q1, lane);
    store_block<kMlpHid>(hs[1], g.d[2], r0, B, t);
    dx_epilogue(acc, g2, hs[0], &cs2, t);
    lds_barrier();
    acc = stream_product<KH, 0>(zero_start(), ring, hs[0], q1, q1, lane);
    store_block<kMlpHid>(hs[0], g.d[1], r0, B, t);
    dx_epilogue(acc, g1, hs[1], &cs1, t);
    lds_barrier();
    store_block<kMlpHid>(hs[1], g.d[0], r0, B, t);
  }
  if constexpr (TRAIN) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const size_t ld = (size_t)gridDim.x * kMlpHid;
    float* const bsum = g.bsum + (size_t)blockIdx.x * kMlpHid;
    if ((lane & 31) < 16) {
      const int n = out_base(t) + 8 * ((lane & 15) >> 2) + (lane & 3);
      bsum[n] = cs1;
      bsum[ld + n] = cs2;
      bsum[2 * ld + n] = cs3;
    }
    if (t < kMlpOut) bsum[3 * ld + t] = csh;
    nll += __shfl_xor(nll, 16);
    nll += __shfl_xor(nll, 32);
    if (lane == 0) wave_nll[wave] = nll;
    __syncthreads();
    if (t == 0) {
      float s = 0.0f;
      for (int w = 0; w < kFuseWaves; ++w) s += wave_nll[w];
      atomicAdd(g.loss_sum, s / (float)B);
    }
  }
}

// ---------------------------------------------------------------------------
// Weight gradients: dW_l [kin][nout] = h_l^T d_l, contractions over the batch,
// split over row ranges (parts), every layer in one launch.  Both operands are
// row-major [B][width], so a stage of 32 or 64 batch rows is copied as it lies into
// LDS and the transposing LDS read (ds_read_b64_tr_b16: 16 lanes fetch a 4 x 16
// tile, lane s row s / 4, columns 4 (s % 4) .. + 3, and lane s receives column
// s) gives a lane the consecutive k-values of its column.  A workgroup forms a
// 64 MW x 128 tile on v_mfma_f32_16x16x32_bf16, a wave 64 x 64 of it; the next
// stage is loaded into registers while the current one is multiplied.
// LDS rows are padded by 32 bytes: the 16 row segments one read touches then
// fall in distinct banks.
//
// Bound: reading the operands (0.21 GB at batch 65,536).  Batch
// 65,536: 47-53 us, 4 TB/s (124 us with 64 x 64 tiles reading batch-minor copies,
// each operand four times); batch 4,096: 14 us (13), latency.
// ---------------------------------------------------------------------------
typedef short s16x4_t __attribute__((ext_vector_type(4)));
constexpr int kDwN = 128, kDwPad = 16;

// One output tile family: A [B][wa] (columns m0 .. of the 64 MW a workgroup
// takes, M of them in all), B [B][wb] (columns n0 .. n0 + 127); element (m, n)
// of part z goes to part[z * size + m * sm + n * sn].
struct DwTile {
  const uint16_t *A, *B;
  int wa, wb, m0, n0, M, N, sm, sn, size;
  float* part;
};
struct DwGroup {
  DwTile t[12];  // at most 4 + 4 + 2 + 2 tiles of 128 x 128
  int n_tiles, rows, rows_per_part;
};

template <int STRIDE>
__device__ __forceinline__ bf16x8_t tr_frag(const uint16_t (*S)[STRIDE], int c0) {
  const int lane = threadIdx.x & 63, g = lane >> 4, s = lane & 15;
  typedef __attribute__((address_space(3))) s16x4_t lds_s16x4;
  struct { s16x4_t lo, hi; } v;
  v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)&S[8 * g + (s >> 2)][c0 + 4 * (s & 3)]);
  v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)&S[8 * g + 4 + (s >> 2)][c0 + 4 * (s & 3)]);
  return __builtin_bit_cast(bf16x8_t, v);
}

// MW m-waves of 64 columns and two n-waves; stages of kDwRows rows.
template <int MW, int kDwRows>
__global__ void __launch_bounds__(128 * MW)
mlp_dw_kernel(DwGroup g) {
  constexpr int kThreads = 128 * MW, kM = 64 * MW;
  constexpr int LA = kM + kDwPad, LB = kDwN + kDwPad;
  constexpr int CA = kDwRows * kM / 8 / kThreads, CB = kDwRows * kDwN / 8 / kThreads;  // 16-byte chunks per thread
  static_assert(CA * kThreads * 8 == kDwRows * kM && CB * kThreads * 8 == kDwRows * kDwN, "whole chunks");
  __shared__ __attribute__((aligned(16))) uint16_t As[2][kDwRows][LA];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][kDwRows][LB];
  // Consecutive workgroups take consecutive parts of one tile (a part's tiles
  // then lie a multiple of n_parts apart: on one XCD when that is a multiple of
  // 8, so an operand two tiles share is in its L2).
  const int parts = (g.rows + g.rows_per_part - 1) / g.rows_per_part;
  const int tile = blockIdx.x / parts, z = blockIdx.x % parts;
  const DwTile& T = g.t[tile];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
  const int kbeg = z * g.rows_per_part, kend = min(g.rows, kbeg + g.rows_per_part);
  const int wa = T.wa, wb = T.wb;
  // This wave's 16-column blocks inside the product (uniform).
  const int mb = min(4, (T.M - T.m0 - 64 * wm + 15) / 16), nb = min(4, (T.N - T.n0 - 64 * wn + 15) / 16);
  uint4 ra[CA], rb[CB];
  auto load = [&](int k0) {
#pragma unroll
    for (int i = 0; i < CA; ++i) {
      const int e = t + i * kThreads, row = k0 + e / (kM / 8), col = T.m0 + 8 * (e % (kM / 8));
      ra[i] = row < kend && col < T.M ? *reinterpret_cast<const uint4*>(T.A + (size_t)row * wa + col)
                                      : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int i = 0; i < CB; ++i) {
      const int e = t + i * kThreads, row = k0 + e / (kDwN / 8), col = T.n0 + 8 * (e % (kDwN / 8));
      rb[i] = row < kend && col < T.N ? *reinterpret_cast<const uint4*>(T.B + (size_t)row * wb + col)
                                      : make_uint4(0u, 0u, 0u, 0u);
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int i = 0; i < CA; ++i) {
      const int e = t + i * kThreads;
      *reinterpret_cast<uint4*>(&As[buf][e / (kM / 8)][8 * (e % (kM / 8))]) = ra[i];
    }
#pragma unroll
    for (int i = 0; i < CB; ++i) {
      const int e = t + i * kThreads;
      *reinterpret_cast<uint4*>(&Bs[buf][e / (kDwN / 8)][8 * (e % (kDwN / 8))]) = rb[i];
    }
  };
  f32x4_t acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  load(kbeg);
  store(0);
  lds_barrier();
  int buf = 0;
  for (int k0 = kbeg; k0 < kend; k0 += kDwRows, buf ^= 1) {
    const bool more = k0 + kDwRows < kend;  // uniform
    if (more) load(k0 + kDwRows);
    if (mb > 0 && nb > 0) {
#pragma unroll
      for (int ks = 0; ks < kDwRows / 32; ++ks) {
        bf16x8_t fa[4], fb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          fa[i] = tr_frag<LA>(As[buf] + 32 * ks, 64 * wm + 16 * i);
          fb[i] = tr_frag<LB>(Bs[buf] + 32 * ks, 64 * wn + 16 * i);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (j >= nb) break;  // uniform
#pragma unroll
          for (int i = 0; i < 4; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
      }
    }
    if (more) {
      store(buf ^ 1);
      lds_barrier();
    }
  }
  float* const dst = T.part + (size_t)z * T.size;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m = T.m0 + 64 * wm + 16 * i + 4 * (lane >> 4), n = T.n0 + 64 * wn + 16 * j + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (m + r < T.M && n < T.N) dst[(size_t)(m + r) * T.sm + (size_t)n * T.sn] = acc[i][j][r];
    }
}

// Sums of the weight gradients' parts and of the bias gradients' parts, in one
// launch, each in a fixed order.  The first wblocks workgroups take four
// consecutive weights per lane: wave q of the four sums parts q, q + 4, ...
// and the four sums are added in q order.  The rest take 16 columns each of
// a layer's bias gradient (columns of cs_part [cs_parts][256]), thread group q
// of the 16 summing rows q, q + 16, ..., then the groups in order.  Loads go
// out eight at a time: one at a time, each add waited for a round trip to
// memory (8 us at 16 parts, 31 at 64).
struct ReduceGroup {
  const float* part[4];
  const float* cs_part[4];
  float* out[4];
  float* cs_out[4];
  int wbase[5], cbase[5];  // first float4 of a layer's weights; first 16-column block of its bias
  int parts, cs_parts, wblocks;
};

__global__ void __launch_bounds__(256) mlp_reduce_kernel(ReduceGroup rg) {
  __shared__ float4 s4[4][64];
  __shared__ float s1[16][16];
  const int t = threadIdx.x;
  if ((int)blockIdx.x < rg.wblocks) {  // uniform
    const int q = t >> 6, e = blockIdx.x * 64 + (t & 63);
    int l = 0;
    while (l < 3 && e >= rg.wbase[l + 1]) ++l;
    const int idx = e - rg.wbase[l], stride = rg.wbase[l + 1] - rg.wbase[l];
    const bool in = e < rg.wbase[4];
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (in) {
      const float4* p = reinterpret_cast<const float4*>(rg.part[l]) + idx;
      int z = q;
      for (; z + 28 < rg.parts; z += 32) {
        float4 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = p[(size_t)(z + 4 * k) * stride];
#pragma unroll
        for (int k = 0; k < 8; ++k) { s.x += v[k].x; s.y += v[k].y; s.z += v[k].z; s.w += v[k].w; }
      }
#pragma unroll 4
      for (; z < rg.parts; z += 4) {
        const float4 v = p[(size_t)z * stride];
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
      }
    }
    s4[q][t & 63] = s;
    __syncthreads();
    if (q == 0 && in) {
      float4 a = s4[0][t];
#pragma unroll
      for (int k = 1; k < 4; ++k) { a.x += s4[k][t].x; a.y += s4[k][t].y; a.z += s4[k][t].z; a.w += s4[k][t].w; }
      // a layer's output starts at any float of the flat gradient
      float* o = rg.out[l] + (size_t)4 * idx;
      o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
    }
    return;
  }
  const int cb = (int)blockIdx.x - rg.wblocks;
  int l = 0;
  while (l < 3 && cb >= rg.cbase[l + 1]) ++l;
  const int n = 16 * (cb - rg.cbase[l]) + (t & 15), q = t >> 4;
  float s = 0.0f;
  const float* p = rg.cs_part[l] + n;
  int r = q;
  for (; r + 112 < rg.cs_parts; r += 128) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = p[(size_t)(r + 16 * k) * kMlpHid];
#pragma unroll
    for (int k = 0; k < 8; ++k) s += v[k];
  }
#pragma unroll 4
  for (; r < rg.cs_parts; r += 16) s += p[(size_t)r * kMlpHid];
  s1[q][t & 15] = s;
  __syncthreads();
  if (t < 16) {
    float a = s1[0][t];
#pragma unroll
    for (int k = 1; k < 16; ++k) a += s1[k][t];
    rg.cs_out[l][n] = a;
  }
}

// Forward pass of the one row [x_t; u_user] in a workgroup of 1,024
// threads, then draws from its head: each of the launch's workgroups runs the
// same forward (bit-identical; workgroup 0 stores the head) and draws its
// share of the P proposals, kRowDraws per workgroup and pass.  Roundings are the
// batched path's (standardised input and activations to BF16, BF16 weights, FP32
// accumulation and biases), but not every FP32 operation: here the bias is added
// last, not first, and GELU takes tanhf, not the hardware exponential and
// reciprocal, so an activation that lies at a BF16 rounding boundary can round
// the other way in the two.  In a layer of DIN
// inputs and DOUT units, thread t takes units [8g, 8g + 8) (g = t % (DOUT/8))
// over inputs [8s, 8s + 8) (s = t / (DOUT/8)): eight 16-byte weight loads and
// 64 FMAs; its eight partial sums go to LDS, where one thread per unit adds
// the DIN/8 partials in order.  Each layer's weight loads are issued before
// the previous layer's reduction, so their latency overlaps it.  A serving
// tick needs one row, for which a GEMM tile per layer is mostly idle.
constexpr int kRowThreads = 1024;
constexpr int kRowDraws = 256;
constexpr int kRowMaxGroups = 64;

template <int DIN, int DOUT>
struct RowSlice {
  static constexpr int G = DOUT / 8, S = DIN / 8;
  static_assert(DOUT % 8 == 0 && DIN % 8 == 0 && G * S <= kRowThreads, "row layer shape");
  uint4 w[8];
  __device__ __forceinline__ bool active() const { return (int)threadIdx.x < G * S; }
  __device__ __forceinline__ void load(const uint16_t* __restrict__ W) {
    if (!active()) return;
    const int g = threadIdx.x % G, sl = threadIdx.x / G;
#pragma unroll
    for (int r = 0; r < 8; ++r) w[r] = *reinterpret_cast<const uint4*>(W + (size_t)(8 * sl + r) * DOUT + 8 * g);
  }
  // red[s][DOUT]: this thread's eight partial sums.
  __device__ __forceinline__ void partial(const float* hin, float* red) const {
    if (!active()) return;
    const int g = threadIdx.x % G, sl = threadIdx.x / G;
    float acc[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc[u] = 0.0f;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const float h = hin[8 * sl + r];
      const uint32_t q[4] = {w[r].x, w[r].y, w[r].z, w[r].w};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        acc[2 * u] = fmaf(h, __uint_as_float(q[u] << 16), acc[2 * u]);
        acc[2 * u + 1] = fmaf(h, __uint_as_float(q[u] & 0xffff0000u), acc[2 * u + 1]);
      }
    }
    float4* dst = reinterpret_cast<float4*>(red + (size_t)sl * DOUT + 8 * g);
    dst[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
    dst[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
  }
};

// Unit j's pre-activation: the DIN/8 partials in order, then the bias.
template <int DIN, int DOUT>
__device__ __forceinline__ float row_unit(const float* red, float bias, int j) {
  float v = 0.0f;
#pragma unroll 8
  for (int sl = 0; sl < DIN / 8; ++sl) v += red[sl * DOUT + j];
  return v + bias;
}

__global__ void __launch_bounds__(kRowThreads)
mlp_row_forward_kernel(const float* __restrict__ x_t, const float* __restrict__ u_user,
                       const uint16_t* __restrict__ w16, const float* __restrict__ w32,
                       const float* __restrict__ mean, const float* __restrict__ stdv,
                       float* __restrict__ Y, const ModelDev* __restrict__ md, int P, uint64_t seed,
                       uint64_t tick, int loop, float* __restrict__ cand) {
  __shared__ __attribute__((aligned(16))) float red[(kMlpHid / 8) * kMlpHid];
  __shared__ __attribute__((aligned(16))) float bufA[kMlpHid], bufB[kMlpHid], head[kMlpOut];
  const int j = threadIdx.x;
  // Global loads in the order they are consumed (the vector-memory counter
  // retires loads in issue order): input row and biases, then the weights of
  // layers 0 and 1; layer l + 2's weights are issued before layer l + 1's
  // products.
  float xin = 0.0f, b0 = 0.0f, b1 = 0.0f, b2 = 0.0f, b3 = 0.0f;
  float xm = 0.0f, xs = 1.0f;
  if (j < kMlpIn) {
    xin = j < 6 ? x_t[j] : u_user[j - 6];
    xm = mean[j];
    xs = stdv[j];
  }
  if (j < kMlpHid) {
    b0 = w32[kMlpB0 + j];
    b1 = w32[kMlpB1 + j];
    b2 = w32[kMlpB2 + j];
  }
  if (j < kMlpOut) b3 = w32[kMlpB3 + j];
  RowSlice<kMlpIn, kMlpHid> s0;
  RowSlice<kMlpHid, kMlpHid> s1;
  s0.load(w16 + kMlpW0);
  s1.load(w16 + kMlpW1);
  if (j < kMlpIn) bufA[j] = bf2f(f2bf((xin - xm) / xs));
  lds_barrier();
  s0.partial(bufA, red);
  lds_barrier();
  if (j < kMlpHid) bufB[j] = bf2f(f2bf(gelu_f(row_unit<kMlpIn, kMlpHid>(red, b0, j))));
  lds_barrier();
  RowSlice<kMlpHid, kMlpHid> s2;
  s2.load(w16 + kMlpW2);
  s1.partial(bufB, red);
  lds_barrier();
  if (j < kMlpHid) bufA[j] = bf2f(f2bf(gelu_f(row_unit<kMlpHid, kMlpHid>(red, b1, j))));
  lds_barrier();
  RowSlice<kMlpHid, kMlpOut> s3;
  s3.load(w16 + kMlpW3);
  s2.partial(bufA, red);
  lds_barrier();
  if (j < kMlpHid) bufB[j] = bf2f(f2bf(gelu_f(row_unit<kMlpHid, kMlpHid>(red, b2, j))));
  lds_barrier();
  s3.partial(bufB, red);
  lds_barrier();
  if (j < kMlpOut) {
    const float v = row_unit<kMlpHid, kMlpOut>(red, b3, j);
    head[j] = v;
    if (blockIdx.x == 0) Y[j] = v;
  }
  if (P <= 0) return;
  __shared__ MdnTable tab;
  lds_barrier();
  mdn_table_build(head, &tab);
  for (int p = blockIdx.x * kRowDraws + j; j < kRowDraws && p < P; p += gridDim.x * kRowDraws)
    mdn_draw(md, head, &tab, P, p, seed, tick, loop, cand);
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Rows of the batch per part of the weight-gradient products: at most 64 parts
// (40 or 32 parts at 65,536 leave compute units idle: step 169 us against 178
// and 185), at least 256 rows while that fills the chip (4,096: 192 workgroups
// of 128 x 128 tiles, step 40.5 us; 384 rows 43, 128 rows 41 but 53 against 49
// at 8,192), and 128 below, where few parts are a longer chain each.
constexpr int kMlpSplits = 64;
static int dw_rows_per_part(int B) {
  const int per = B <= 2048 ? 128 : 256;
  return std::max(per, (B + kMlpSplits - 1) / kMlpSplits + 31) / 32 * 32;
}

// What leaves the fused pass is what later launches read: the BF16 activations
// and gradients row-major (index l: the input of layer l, and the gradient of
// its output) for the weight-gradient products, and the bias gradients' parts.
// Each layer has its own split partial buffers.
struct MlpWork {
  uint16_t *packed, *h[4], *d[4];
  float *Y, *loss, *bsum;
  float* part[4];
};

// Workgroups of the fused pass: one block of rows each up to two per compute
// unit, which the registers allow; further blocks go to the same workgroups.
constexpr int kFuseGroups = 512;
static int fuse_groups(int B) { return std::min((B + kFuseRows - 1) / kFuseRows, kFuseGroups); }

constexpr int kMlpDims[5] = {kMlpIn, kMlpHid, kMlpHid, kMlpHid, kMlpOut};

static MlpWork carve(void* base, int B) {
  char* p = (char*)base;
  MlpWork w;
  auto take = [&](size_t bytes) { char* r = p; p += align256(bytes); return (void*)r; };
  w.packed = (uint16_t*)take((size_t)kPackedChunks * kChunk * 2);
  for (int l = 0; l < 4; ++l) {
    w.h[l] = (uint16_t*)take((size_t)B * kMlpDims[l] * 2);
    w.d[l] = (uint16_t*)take((size_t)B * kMlpDims[l + 1] * 2);
  }
  w.Y = (float*)take((size_t)kMlpOut * 4);  // the serving tick's head
  w.loss = (float*)take(4);
  w.bsum = (float*)take((size_t)4 * fuse_groups(B) * kMlpHid * 4);  // bias-gradient parts (the head uses 80)
  for (int l = 0; l < 4; ++l) w.part[l] = (float*)take((size_t)kMlpSplits * kMlpDims[l] * kMlpDims[l + 1] * 4);
  return w;
}

size_t mlp_workspace_bytes(int B) {
  char* base = nullptr;
  MlpWork w = carve((void*)base, B);
  return (size_t)((char*)w.part[3] - base) + align256((size_t)kMlpSplits * kMlpHid * kMlpOut * 4);
}

// Offsets of (W_l, b_l) in the flat parameter vector.
static void layer_offsets(size_t* ow, size_t* ob) {
  const int dims[5] = {kMlpIn, kMlpHid, kMlpHid, kMlpHid, kMlpOut};
  size_t o = 0;
  for (int l = 0; l < 4; ++l) {
    ow[l] = o;
    o += (size_t)dims[l] * dims[l + 1];
    ob[l] = o;
    o += dims[l + 1];
  }
}

// The weights packed (the forward products' alone without training), then
// the fused pass.
template <bool TRAIN>
static hipError_t fused_pass(const uint16_t* w16, const MlpWork& w, FusedArgs a, float* loss_zero, hipStream_t st) {
  const int chunks = TRAIN ? kPackedChunks : kForwardChunks;
  mlp_pack_weights_kernel<<<(chunks + 3) / 4, 256, 0, st>>>(w16, w.packed, loss_zero);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  a.packed = w.packed;
  mlp_fused_kernel<TRAIN><<<fuse_groups(a.B), kFuseThreads, 0, st>>>(a);
  return hipGetLastError();
}

// Biases are kept in FP32 (they add to FP32 accumulators): the FP32 master
// vector is passed alongside the BF16 weights.
hipError_t launch_mlp_forward(const uint16_t* w16, const float* w32, const float* mean, const float* stdv,
                              const float* X, int B, float* Y, void* work, hipStream_t st) {
  FusedArgs a{};
  a.bias32 = w32; a.mean = mean; a.stdv = stdv; a.X = X; a.B = B; a.Y = Y;
  return fused_pass<false>(w16, carve(work, B), a, nullptr, st);
}

// One gradient: weights packed, the fused pass, every layer's weight
// gradient in one launch and the sums of their parts in another.  The loss
// accumulates straight into *loss (or the workspace).
hipError_t launch_mlp_grad(const uint16_t* w16, const float* w32, const float* mean, const float* stdv,
                           const float* X, const float* T, int B, float* grad, float* loss, void* work,
                           hipStream_t st) {
  const MlpWork w = carve(work, B);
  FusedArgs a{};
  a.bias32 = w32; a.mean = mean; a.stdv = stdv; a.X = X; a.T = T; a.B = B;
  for (int l = 0; l < 4; ++l) {
    a.h[l] = w.h[l];
    a.d[l] = w.d[l];
  }
  a.bsum = w.bsum;
  a.loss_sum = loss ? loss : w.loss;
  hipError_t e = fused_pass<true>(w16, w, a, a.loss_sum, st);
  if (e != hipSuccess) return e;
  // The first layer has eight inputs: its gradient is formed transposed (the
  // 256 outputs on the tile's long side).
  // Tiles of 128 x 128 while the parts are few (256 x 128 at 4,096: step 44.7 us
  // against 43.4), of 256 x 128, one read of the wide operand less, above
  // (128 x 128 at 12,001: 60 against 55; at 32,768: 95 against 86).
  const int mw = B <= 8192 ? 2 : 4;
  DwGroup g{};
  ReduceGroup rg{};
  g.rows = B;
  g.rows_per_part = dw_rows_per_part(B);
  const int parts = (B + g.rows_per_part - 1) / g.rows_per_part;
  size_t ow[4], ob[4];
  layer_offsets(ow, ob);
  for (int l = 0; l < 4; ++l) {
    const int kin = kMlpDims[l], nout = kMlpDims[l + 1];
    DwTile d{};
    d.A = l ? w.h[l] : w.d[0];
    d.B = l ? w.d[l] : w.h[0];
    d.wa = d.M = l ? kin : nout;
    d.wb = d.N = l ? nout : kin;
    d.sm = l ? nout : 1;
    d.sn = l ? 1 : nout;
    d.size = kin * nout;
    d.part = w.part[l];
    for (d.m0 = 0; d.m0 < d.M; d.m0 += 64 * mw)
      for (d.n0 = 0; d.n0 < d.N; d.n0 += kDwN) g.t[g.n_tiles++] = d;
    rg.part[l] = w.part[l];
    rg.cs_part[l] = w.bsum + (size_t)l * fuse_groups(B) * kMlpHid;
    rg.out[l] = grad + ow[l];
    rg.cs_out[l] = grad + ob[l];
    rg.wbase[l + 1] = rg.wbase[l] + kin * nout / 4;
    rg.cbase[l + 1] = rg.cbase[l] + nout / 16;
  }
  rg.parts = parts;
  rg.cs_parts = fuse_groups(B);
  rg.wblocks = (rg.wbase[4] + 63) / 64;
  if (mw == 4) mlp_dw_kernel<4, 32><<<g.n_tiles * parts, 512, 0, st>>>(g);
  else mlp_dw_kernel<2, 64><<<g.n_tiles * parts, 256, 0, st>>>(g);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  mlp_reduce_kernel<<<rg.wblocks + rg.cbase[4], 256, 0, st>>>(rg);
  return hipGetLastError();
}

hipError_t launch_mlp_adam(float* w32, uint16_t* w16, float* m, float* v, const float* grad, int step, float lr,
                           hipStream_t st) {
  // Constants and their complements rounded once from FP64 (1 - 0.999f in
  // FP32 would carry a 1e-5 relative error into the second moment).
  const double b1 = 0.9, b2 = 0.999;
  const float c1 = (float)(1.0 - pow(b1, step)), c2 = (float)(1.0 - pow(b2, step));
  adam_kernel<<<(kMlpParams + 255) / 256, 256, 0, st>>>(w32, w16, m, v, grad, kMlpParams, lr, (float)b1, (float)b2,
                                                        (float)(1.0 - b1), (float)(1.0 - b2), 1e-8f, c1, c2);
  return hipGetLastError();
}

hipError_t launch_mdn_sample(const void* model, const float* Yrow, int P, uint64_t seed, uint64_t tick, int loop,
                             float* cand, hipStream_t st) {
  mdn_sample_kernel<<<(P + 255) / 256, 256, 0, st>>>((const ModelDev*)model, Yrow, P, seed, tick, loop, cand);
  return hipGetLastError();
}

hipError_t launch_mlp_row_forward(const float* x_t, const float* u_user, const uint16_t* w16, const float* w32,
                                  const float* mean, const float* stdv, void* work, float* head_out, float** head,
                                  const void* model, int P, uint64_t seed, uint64_t tick, int loop, float* cand,
                                  hipStream_t st) {
  const MlpWork w = carve(work, 1);
  *head = head_out ? head_out : w.Y;
  int groups = P > 0 ? (P + kRowDraws - 1) / kRowDraws : 1;
  groups = groups < kRowMaxGroups ? groups : kRowMaxGroups;
  mlp_row_forward_kernel<<<groups, kRowThreads, 0, st>>>(x_t, u_user, w16, w32, mean, stdv, *head,
                                                         (const ModelDev*)model, P, seed, tick, loop, cand);
  return hipGetLastError();
}

hipError_t launch_gemm_test(const uint16_t* A, const uint16_t* B, int M, int N, int K, int ta, int tb, float* C,
                            hipStream_t st) {
  GemmArgs g{};
  g.A = A; g.B = B; g.M = M; g.N = N; g.K = K; g.ta = ta; g.tb = tb;
  g.lda = ta ? M : K;
  g.ldb = tb ? K : N;
  g.out = C;
  g.vec_a = g.lda % 8 == 0 && ((uintptr_t)A & 15) == 0;
  g.vec_b = g.ldb % 8 == 0 && ((uintptr_t)B & 15) == 0;
  gemm_bf16_kernel<<<dim3((N + 63) / 64, (M + 63) / 64), 256, 0, st>>>(g);
  return hipGetLastError();
}

}  // namespace mpmi
