// Latency form of the fused tick: each candidate spread over SPLIT lanes.
//
// With few candidates per tick a wave's 60-step serial chain, not the chip's
// throughput, sets the tick time: a wave issues one instruction per four
// cycles, so the step's instruction count is its latency.  Here lane h of a
// group of SPLIT computes output columns [h J, h J + J) of every step
// (J = ceil(n / SPLIT)) from the full feature set, and the group rebuilds the
// full next state with cross-lane permutes, so each lane's contraction is
// J / n of the one-lane form, at the price of redundant feature and safety
// work.  The caller, the autotuner or the library (tick_lanes, by candidate
// count) picks SPLIT.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "mpmi_device.hpp"
#include "mpmi_launch.hpp"
#include "mpmi_tick_common.hpp"

namespace mpmi {

// LDS rows of 8 floats; column j of a row sits at (j / J) * A + (j % J), A = 4
// when J = 3 (so a lane's three columns are one aligned float4), else J.
template <int J>
struct SplitLayout {
  static constexpr int A = (J == 3) ? 4 : J;
  static __device__ __forceinline__ int pos(int j) { return (j / J) * A + (j % J); }
};

constexpr int kSplitRows = 64 + 27;  // full rows + per-step rows (race car is the larger)

// Row r of the table: K row r (r < D), or the per-step row r - D (the
// quadratic state features, then for the race car the heading terms).
template <int BASIS>
__device__ __forceinline__ int split_row(int r) {
  constexpr int D = (BASIS == MPMI_BASIS_RACE_CAR) ? 64 : 21;
  if (r < D) return r;
  const int q = r - D;
  if (BASIS == MPMI_BASIS_RACE_CAR) {
    if (q < 21) {
      int k = 0, t = q;
      while (t >= 6 - k) { t -= 6 - k; ++k; }
      return quad_index(k, k + t, 8);
    }
    constexpr int trig_rows[6] = {49, 50, 51, 53, 54, 55};
    return trig_rows[q - 21];
  }
  int k = 0, t = q;
  while (t >= 4 - k) { t -= 4 - k; ++k; }
  return quad_index(k, k + t, 5);
}

// One pass over the table: every entry is written once, with its K value or
// zero (positions no column maps to), so one barrier suffices; D and R are
// the basis' constants, so the loads start without a round trip.
template <int BASIS, int J>
__device__ __forceinline__ void stage_K_split(const ModelDev* __restrict__ md, float* sK8) {
  constexpr int NS = Dims<BASIS>::N;
  constexpr int D = (BASIS == MPMI_BASIS_RACE_CAR) ? 64 : 21;
  constexpr int R = (BASIS == MPMI_BASIS_RACE_CAR) ? kRcStepRows : 10;
  constexpr int A = SplitLayout<J>::A;
  for (int e = threadIdx.x; e < (D + R) * 8; e += blockDim.x) {
    const int r = e >> 3, p = e & 7;
    const int j = (p / A) * J + (p % A);  // the column at position p, if p % A < J
    float v = 0.0f;
    if (p % A < J && j < NS) v = md->K[split_row<BASIS>(r)][j];
    sK8[e] = v;
  }
  __syncthreads();
}

// Loads J consecutive floats at an aligned LDS position.
template <int J>
__device__ __forceinline__ void ldsJ(const float* p, float* out) {
  if constexpr (J == 3 || J == 4) {
    const float4 v = *reinterpret_cast<const float4*>(p);
    out[0] = v.x; out[1] = v.y; out[2] = v.z;
    if constexpr (J == 4) out[3] = v.w;
  } else if constexpr (J == 2) {
    const float2 v = *reinterpret_cast<const float2*>(p);
    out[0] = v.x; out[1] = v.y;
  } else {
    out[0] = p[0];
  }
}

// Folded per-lane coefficients for this lane's J columns (LDS position p0).
template <int BASIS, int J>
struct SplitFold {
  static constexpr int NS = Dims<BASIS>::N;
  float cu[J], L[NS][J], Ts[J], Tc[J];
  __device__ __forceinline__ void fold(const float* sK8, int p0, const float* uu) {
    float sd = 0.0f, cd = 1.0f;
    if (BASIS == MPMI_BASIS_RACE_CAR) sincosf(uu[0], &sd, &cd);
#pragma unroll
    for (int jj = 0; jj < J; ++jj) {
      const float* Kc = sK8 + p0 + jj;  // column jj of this lane: Kc[f * 8]
      if (BASIS == MPMI_BASIS_RACE_CAR) {
        const float d = uu[0], a = uu[1];
        float v = Kc[0];
        v = fmaf(d, Kc[7 * 8], v);
        v = fmaf(a, Kc[8 * 8], v);
        v = fmaf(d * d, Kc[quad_index(6, 6, 8) * 8], v);
        v = fmaf(d * a, Kc[quad_index(6, 7, 8) * 8], v);
        v = fmaf(a * a, Kc[quad_index(7, 7, 8) * 8], v);
        v = fmaf(sd, Kc[47 * 8], v);
        v = fmaf(cd, Kc[48 * 8], v);
        v = fmaf(a * sd, Kc[63 * 8], v);
        cu[jj] = v;
#pragma unroll
        for (int k = 0; k < 6; ++k)
          L[k][jj] = fmaf(a, Kc[quad_index(k, 7, 8) * 8], fmaf(d, Kc[quad_index(k, 6, 8) * 8], Kc[(1 + k) * 8]));
        L[3][jj] = fmaf(cd, Kc[60 * 8], fmaf(sd, Kc[57 * 8], L[3][jj]));
        L[4][jj] = fmaf(cd, Kc[61 * 8], fmaf(sd, Kc[58 * 8], L[4][jj]));
        L[5][jj] = fmaf(cd, Kc[62 * 8], fmaf(sd, Kc[59 * 8], L[5][jj]));
        Ts[jj] = fmaf(a, Kc[52 * 8], Kc[45 * 8]);
        Tc[jj] = fmaf(a, Kc[56 * 8], Kc[46 * 8]);
      } else {
        const float uv = uu[0];
        cu[jj] = fmaf(uv * uv, Kc[quad_index(4, 4, 5) * 8], fmaf(uv, Kc[5 * 8], Kc[0]));
#pragma unroll
        for (int k = 0; k < NS; ++k) L[k][jj] = fmaf(uv, Kc[quad_index(k, 4, 5) * 8], Kc[(1 + k) * 8]);
        Ts[jj] = Tc[jj] = 0.0f;
      }
    }
  }
};

// This lane's columns of the per-step rows (quadratic state features, and for
// the race car the six heading cross terms), held in registers for the whole
// horizon: at one or two waves per SIMD nothing hides LDS latency, and a wave
// of this kernel has the register file to itself.  LAST: the last rows that an
// instance with less room reads from LDS at every step instead; the step takes
// them last, so the reads, issued at its start, are back by then.
template <int BASIS, int J, int LAST = 0>
struct SplitRows {
  static constexpr int NQ = (BASIS == MPMI_BASIS_RACE_CAR) ? 21 : 10;
  static constexpr int NT = (BASIS == MPMI_BASIS_RACE_CAR) ? 6 : 0;
  static constexpr int NR = NQ + NT, HELD = NR - LAST;
  float k[NR][J];
  const float* last;  // LDS, row HELD
  __device__ __forceinline__ void load(const float* sK8, int D, int colpos) {
#pragma unroll
    for (int r = 0; r < HELD; ++r) ldsJ<J>(&sK8[(D + r) * 8 + colpos], k[r]);
    last = &sK8[(D + HELD) * 8 + colpos];
  }
  // At the start of every step.
  __device__ __forceinline__ void load_last() {
    if constexpr (LAST > 0) {
      int off = 0;
      asm volatile("" : "+v"(off));  // or the reads would be hoisted out of the horizon loop
#pragma unroll
      for (int r = 0; r < LAST; ++r) ldsJ<J>(last + off + r * 8, k[HELD + r]);
    }
  }
};

// This lane's columns of the next state, in the one-lane kernel's operation
// order, so the two give bit-identical states: race car as the feature sum,
// balance bot nested.
template <int BASIS, int J, int LAST>
__device__ __forceinline__ void split_step(const SplitFold<BASIS, J>& F, SplitRows<BASIS, J, LAST>& Kr, const float* x,
                                           float (&y)[J]) {
  constexpr int NS = Dims<BASIS>::N;
  Kr.load_last();
  if constexpr (BASIS == MPMI_BASIS_RACE_CAR) {
    const float sp = __sinf(x[2]), cp = __cosf(x[2]);
#pragma unroll
    for (int jj = 0; jj < J; ++jj) {
      float v = fmaf(F.Tc[jj], cp, fmaf(F.Ts[jj], sp, F.cu[jj]));
#pragma unroll
      for (int k = 0; k < NS; ++k) v = fmaf(F.L[k][jj], x[k], v);
      y[jj] = v;
    }
    int q = 0;
#pragma unroll
    for (int k = 0; k < NS; ++k)
#pragma unroll
      for (int l = k; l < NS; ++l, ++q) {
        const float p = x[k] * x[l];
#pragma unroll
        for (int jj = 0; jj < J; ++jj) y[jj] = fmaf(p, Kr.k[q][jj], y[jj]);
      }
    const float tp[6] = {sp * x[3], sp * x[4], sp * x[5], cp * x[3], cp * x[4], cp * x[5]};
#pragma unroll
    for (int r = 0; r < 6; ++r)
#pragma unroll
      for (int jj = 0; jj < J; ++jj) y[jj] = fmaf(tp[r], Kr.k[q + r][jj], y[jj]);
  } else {
    // y = c + sum_k x_k (L_k + sum_{l >= k} Q_kl x_l) per output column.
#pragma unroll
    for (int jj = 0; jj < J; ++jj) y[jj] = F.cu[jj];
    int q = 0;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      float t[J];
#pragma unroll
      for (int jj = 0; jj < J; ++jj) t[jj] = F.L[k][jj];
#pragma unroll
      for (int l = k; l < NS; ++l, ++q)
#pragma unroll
        for (int jj = 0; jj < J; ++jj) t[jj] = fmaf(Kr.k[q][jj], x[l], t[jj]);
#pragma unroll
      for (int jj = 0; jj < J; ++jj) y[jj] = fmaf(x[k], t[jj], y[jj]);
    }
  }
}

// The constraint constants in registers, loaded once per launch, and the
// track's verdict of a state (the boxes are tested by the lane that holds the
// component).  A verdict is step_safe's: every margin lim - |v| is positive and
// none is NaN exactly when |v| < lim holds for each (with denormals kept, the
// difference of two distinct finite floats is never rounded to zero, and a NaN
// fails either comparison).  The track's
// centreline radius takes track_centre's operations in its order.  TRACK is
// the model's has_track flag, fixed per kernel instance; the float constants
// are pinned to vector registers (the scalar file is too small to hold them
// beside the loop's own state).
//
// NEAR (FP32_RECHECK64): track() also ORs into *near whether its margin lies
// within the track's FP32 band.
template <int NS, int DEG, bool TRACK, bool NEAR = false>
struct SafetyRegs {
  float lim[NS], p[DEG + 1], q[DEG], trk_lim;
  float eps[NEAR ? NS : 1], trk_eps;
  bool chk[NS];
  __device__ __forceinline__ void load(const ModelDev* __restrict__ md) {
    // Every constant is loaded before the first is pinned: a pin waits.
    const ConstSafety* sc = (const ConstSafety*)(uintptr_t)&md->safe;
    const int mask = sc->comp_mask;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      chk[k] = (mask >> k) & 1;
      lim[k] = sc->comp_lim[k];
      if constexpr (NEAR) eps[k] = sc->comp_eps[k];
    }
    if constexpr (TRACK) {
      trk_lim = sc->trk_lim;
      if constexpr (NEAR) trk_eps = sc->trk_eps;
#pragma unroll
      for (int k = 0; k <= DEG; ++k) p[k] = sc->trk_p[k];
#pragma unroll
      for (int k = 0; k < DEG; ++k) q[k] = sc->trk_q[k];
    }
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      asm volatile("" : "+v"(lim[k]));
      if constexpr (NEAR) {
        eps[k] = chk[k] ? eps[k] : 0.0f;  // |margin| < 0 is never true
        asm volatile("" : "+v"(eps[k]));
      }
    }
    if constexpr (TRACK) {
      asm volatile("" : "+v"(trk_lim));
      if constexpr (NEAR) asm volatile("" : "+v"(trk_eps));
#pragma unroll
      for (int k = 0; k <= DEG; ++k) asm volatile("" : "+v"(p[k]));
#pragma unroll
      for (int k = 0; k < DEG; ++k) asm volatile("" : "+v"(q[k]));
    }
  }
  // Bitwise, not short-circuit, combination: each test is one compare into a
  // lane mask, with no branch.
  __device__ __forceinline__ bool track(float x0, float x1, bool* near) const {
    if constexpr (!TRACK) return true;
    const float r2 = fmaf(x0, x0, x1 * x1);
    const float inv = __builtin_amdgcn_rsqf(r2);
    const float rho = r2 * inv;
    const float c1 = x0 * inv, s1 = x1 * inv;
    float P = p[DEG];
#pragma unroll
    for (int k = DEG - 1; k >= 0; --k) P = fmaf(P, c1, p[k]);
    float Q = q[DEG - 1];
#pragma unroll
    for (int k = DEG - 2; k >= 0; --k) Q = fmaf(Q, c1, q[k]);
    const float off = fabsf(rho - fmaf(s1, Q, P));
    if constexpr (NEAR) *near |= fabsf(trk_lim - off) < trk_eps;
    return off < trk_lim;
  }
};

// Value of v in lane `SRC` of this lane's group, with DPP permutes (no LDS
// round trip).  Groups of 2 or 4 lanes sit inside one quad: one quad_perm.
// A group of 8 is two quads of one row half: a quad_perm broadcasts lane
// SRC % 4 of every quad, then the quad that does not hold SRC takes the value
// of the quad beside it (row_shr:4 into banks 1 and 3, or row_shl:4 into
// banks 0 and 2; the other banks keep the broadcast).
template <int SPLIT, int SRC>
__device__ __forceinline__ float group_lane(float v) {
  const int iv = __builtin_bit_cast(int, v);
  if constexpr (SPLIT == 8) {
    const int b = __builtin_amdgcn_mov_dpp(iv, (SRC & 3) * 0x55, 0xF, 0xF, true);
    constexpr int shift = SRC < 4 ? 0x114 : 0x104;      // row_shr:4 / row_shl:4
    constexpr int banks = SRC < 4 ? 0xA : 0x5;          // the quads that take the neighbour's value
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(b, b, shift, 0xF, banks, false));
  } else {
    constexpr int ctrl = (SPLIT == 4) ? SRC * 0x55 : (SRC == 0 ? 0xA0 : 0xF5);  // quad_perm selectors
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(iv, ctrl, 0xF, 0xF, true));
  }
}

template <int NS, int J, int SPLIT, int JJ = 0>
__device__ __forceinline__ void rebuild_state(const float* y, float* x) {
  if constexpr (JJ < NS) {
    x[JJ] = group_lane<SPLIT, JJ / J>(y[JJ % J]);
    rebuild_state<NS, J, SPLIT, JJ + 1>(y, x);
  }
}

// The end of a latency-form tick, every thread of the workgroup calling it:
// lead lanes (one per candidate) hold fv and the cost.  RECHECK: near-band
// candidates go to the list with their FP32 verdict instead of publishing, as
// in tick_fp32_kernel, and the launches that follow complete the slot.
template <int MS, bool RECHECK>
__device__ __forceinline__ void split_finish(const ModelDev* __restrict__ md, const GenParams& gp, int H,
                                             const float* __restrict__ u_user, const float* __restrict__ cand,
                                             Slot* __restrict__ slot, mpmi_selection* __restrict__ out,
                                             RecheckList* __restrict__ rl, bool lead, bool near, int c, int fv,
                                             float cst) {
  const bool listed = RECHECK && lead && near;
  const bool pub = lead && !listed;
  const bool safe = pub && fv == H + 1;
  const unsigned long long ks = safe ? safe_key(cst, c) : kKeyNone;
  const unsigned long long kf = (pub && !safe) ? fallback_key(fv, cst, c) : kKeyNone;
  if constexpr (RECHECK) {
    wave_append(&rl->count, rl->idx, listed, (c << 1) | (fv == H + 1 ? 1 : 0));
    publish_partial(ks, kf, (unsigned int)__popcll(__ballot(safe && c > 0)), (unsigned int)__popcll(__ballot(listed)),
                    slot, blockIdx.x);
  } else {
    if (reduce_and_publish(ks, kf, safe && c > 0, slot, gridDim.x, blockIdx.x) && threadIdx.x == 0)
      finalize<MS>(md, gp, cand, u_user, H, slot, out);
  }
}

// Bound: the wave's instructions and the chain of a column's terms, taken in the
// one-lane form's order.  A lane tests its own columns' boxes only, the verdict
// fills the gaps of the next step's chain, and the exit is one scalar test for
// the wave; every lane testing every box after the step, with an exit per
// candidate, took, for the race car at 60 steps, 2,048 candidates (8 lanes) 26.4
// us against 22.0, 16,385 (4 lanes) 33.5 against 30.7, and for the balance bot at
// 50, 4,097 (4 lanes) 14.6 against 11.5.
//
// GATED (the fallback after a proposal tick): nothing to do if the gate
// selection already found a safe candidate; an instance of its own, since the
// test would hold up the other loads of every launch.
//
// WAVES: waves per SIMD to leave room for.  The race car's two-lane form holds
// three columns of K and takes more than half the registers; an instance with
// room for two waves serves ticks of more than one: 32,769 candidates 37.5 us
// against 53 in two turns, 65,536 47.4 against 64; 32,768, one wave each, 40 against
// 34.6.  It reads its last kLastRows rows from LDS at every step (SplitRows); held,
// they put 19 to 33 values in scratch (39.6 and 51.3 us; FP32_RECHECK64, 65,536, 62.5
// against 53.4), which ticks that may not allocate must not need.  With eight the
// degree-8 instances still spill.
constexpr int kLastRows = 10;
template <int BASIS, int SPLIT, int DEG, bool TRACK, bool RECHECK, bool GATED, int WAVES>
__global__ void __launch_bounds__(SPLIT == 2 && BASIS != MPMI_BASIS_RACE_CAR ? 512 : 256, WAVES)
tick_split_kernel(const ModelDev* __restrict__ md, GenParams gp, int H, const float* __restrict__ x_t,
                  const float* __restrict__ u_user, const float* __restrict__ cand, Slot* __restrict__ slot,
                  mpmi_selection* __restrict__ out, int16_t* __restrict__ fv_out, RecheckList* __restrict__ rl,
                  const mpmi_selection* __restrict__ gate) {
  constexpr int NS = Dims<BASIS>::N, MS = Dims<BASIS>::M;
  constexpr int J = (NS + SPLIT - 1) / SPLIT;
  constexpr int D = (BASIS == MPMI_BASIS_RACE_CAR) ? 64 : 21;
  static_assert(SPLIT == 2 || SPLIT == 4 || SPLIT == 8, "groups of 2, 4 or 8 lanes (one row half)");
  if (GATED && gate->status == MPMI_OK) return;
  __shared__ __attribute__((aligned(16))) float sK8[kSplitRows * 8];
  // A group never straddles a quad (2, 4) or a row half (8): the launch
  // uses a block that is a multiple of 64, so lane l of a wave holds gid with
  // gid % 64 == l.
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int c = gid / SPLIT, h = gid % SPLIT;
  const int Nc = gp.n_cand + 1;
  const bool valid = c < Nc;
  const int colpos = h * SplitLayout<J>::A;

  // State and candidate loads first: their latency overlaps the staging of K.
  float x[NS], u[MS], u0[MS];
#pragma unroll
  for (int j = 0; j < NS; ++j) x[j] = x_t[j];
#pragma unroll
  for (int j = 0; j < MS; ++j) {
    u0[j] = valid ? cand_value(gp, md, cand, u_user, c, 0, j) : 0.0f;
    u[j] = u0[j];
  }
  stage_K_split<BASIS, J>(md, sK8);
  SplitFold<BASIS, J> F;
  F.fold(sK8, colpos, u);
  SplitRows<BASIS, J, (WAVES > 1) ? kLastRows : 0> Kr;
  Kr.load(sK8, D, colpos);
  SafetyRegs<NS, DEG, TRACK, RECHECK> sr;
  sr.load(md);
  // This lane's columns' boxes (the other components' limits are dead after
  // this), and the lanes that hold a boxed column jj.
  float lim[J], eps[J];
  unsigned long long boxed[J];
#pragma unroll
  for (int jj = 0; jj < J; ++jj) {
    bool b = false;
    lim[jj] = eps[jj] = 0.0f;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      const bool mine = h * J + jj == k;
      b = mine ? sr.chk[k] : b;
      lim[jj] = mine ? sr.lim[k] : lim[jj];
      if constexpr (RECHECK) eps[jj] = mine ? sr.eps[k] : eps[jj];
    }
    boxed[jj] = __builtin_amdgcn_ballot_w64(b);
  }
  // The cost needs only the first segment's input: taken now, so its loads
  // are not on the path after the horizon.
  const bool lead = valid && h == 0;
  const float cst = lead ? cost_of<MS>(md, u0, u_user) : 0.0f;
  // Every register above is loaded before the horizon starts, so the loop
  // carries no wait for them.
  __syncthreads();
  // The wave goes through the horizon as one: lanes of a candidate that has
  // ended (not in `live`) run along, their values unused, so a step costs one
  // scalar test and no change of the execution mask.  `on`: the lanes whose
  // verdict counts, none at x_0, the current state.
  const int lane = threadIdx.x & 63, base = lane & ~(SPLIT - 1);
  constexpr unsigned long long kGroup = (1ull << SPLIT) - 1;
  unsigned long long live = __builtin_amdgcn_ballot_w64(valid), on = 0, nears = 0;
  int fv = H + 1;
  float own[J];  // this lane's columns of the state being checked
#pragma unroll
  for (int jj = 0; jj < J; ++jj) own[jj] = 0.0f;
  // Lanes that find x outside the safe set, each testing its own columns' boxes
  // and the track; those within the rounding band are added to `nears`.
  auto failing = [&]() {
    bool nr = false;
    unsigned long long bad = 0;
    if constexpr (TRACK) bad = __builtin_amdgcn_ballot_w64(!sr.track(x[0], x[1], &nr));
    if constexpr (RECHECK && TRACK) nears |= __builtin_amdgcn_ballot_w64(nr) & on;
#pragma unroll
    for (int jj = 0; jj < J; ++jj) {
      bad |= __builtin_amdgcn_ballot_w64(!(fabsf(own[jj]) < lim[jj])) & boxed[jj];
      if constexpr (RECHECK) nears |= __builtin_amdgcn_ballot_w64(fabsf(lim[jj] - fabsf(own[jj])) < eps[jj]) & on;
    }
    return bad & on;
  };
  const int S = gp.n_seg;
  // Segment g covers steps s with floor((s - 1) S / H) == g; the next
  // boundary is the least s - 1 >= ceil((g + 1) H / S).
  int gcur = 0;
  int nxt = (H + S - 1) / S;
  for (int s = 1; s <= H && live != 0ull; ++s) {
    if (s - 1 >= nxt) {
      gcur = ((s - 1) * S) / H;
      nxt = ((gcur + 1) * H + S - 1) / S;
#pragma unroll
      for (int j = 0; j < MS; ++j) u[j] = valid ? cand_value(gp, md, cand, u_user, c, gcur, j) : 0.0f;
      F.fold(sK8, colpos, u);
    }
    float y[J];
    split_step(F, Kr, x, y);
    // The verdict of x_{s-1}, beside the step that forms x_s (the two chains
    // overlap; an unsafe x_{s-1} ends the rollout and x_s is dropped).  The
    // group's lanes hold identical states (same values, same operations).
    const unsigned long long bad = failing();
#pragma unroll
    for (int jj = 0; jj < J; ++jj) asm volatile("" : "+v"(y[jj]));  // formed above the exit
    if (bad != 0ull) {
      const bool ends = ((bad >> base) & kGroup) != 0ull;
      if (ends) fv = s - 1;
      live &= ~__builtin_amdgcn_ballot_w64(ends);
    }
    on = live;
    rebuild_state<NS, J, SPLIT>(y, x);
    settle_state<NS>(x);
#pragma unroll
    for (int jj = 0; jj < J; ++jj) own[jj] = y[jj];
  }
  if (((failing() >> base) & kGroup) != 0ull) fv = H;  // the last state
  const bool near = RECHECK && ((nears >> base) & kGroup) != 0ull;
  if (fv_out && lead) fv_out[c] = (int16_t)fv;
  split_finish<MS, RECHECK>(md, gp, H, u_user, cand, slot, out, rl, lead, near, c, fv, cst);
}

// The full-horizon rollout of given candidates in the latency form: a lane
// stores its own columns.  Race car, 60 steps, 8,192 candidates: 18 us against 73
// with one lane per candidate.
template <int BASIS, int SPLIT>
__global__ void __launch_bounds__(256)
rollout_split_kernel(const ModelDev* __restrict__ md, int Nc, int S, int H, const float* __restrict__ x0,
                     const float* __restrict__ cand, float* __restrict__ traj, long long traj_ld) {
  constexpr int NS = Dims<BASIS>::N, MS = Dims<BASIS>::M;
  constexpr int J = (NS + SPLIT - 1) / SPLIT;
  constexpr int D = (BASIS == MPMI_BASIS_RACE_CAR) ? 64 : 21;
  __shared__ __attribute__((aligned(16))) float sK8[kSplitRows * 8];
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int h = gid % SPLIT;
  const bool valid = gid / SPLIT < Nc;
  const int c = valid ? gid / SPLIT : Nc - 1;  // lanes past the end run along and store nothing
  const int colpos = h * SplitLayout<J>::A;
  float x[NS], u[MS];
#pragma unroll
  for (int j = 0; j < NS; ++j) x[j] = x0[j];
  auto inputs = [&](int g) {
#pragma unroll
    for (int j = 0; j < MS; ++j) u[j] = cand[((size_t)g * MS + j) * (size_t)Nc + c];
  };
  inputs(0);
  stage_K_split<BASIS, J>(md, sK8);
  SplitFold<BASIS, J> F;
  F.fold(sK8, colpos, u);
  SplitRows<BASIS, J> Kr;
  Kr.load(sK8, D, colpos);
  __syncthreads();
  int nxt = (H + S - 1) / S;  // as in tick_split_kernel
  for (int s = 1; s <= H; ++s) {
    if (s - 1 >= nxt) {
      const int g = ((s - 1) * S) / H;
      nxt = ((g + 1) * H + S - 1) / S;
      inputs(g);
      F.fold(sK8, colpos, u);
    }
    float y[J];
    split_step(F, Kr, x, y);
    rebuild_state<NS, J, SPLIT>(y, x);
    settle_state<NS>(x);
#pragma unroll
    for (int jj = 0; jj < J; ++jj) {
      const int j = h * J + jj;
      if (valid && j < NS) __builtin_nontemporal_store(y[jj], &traj[((size_t)(s - 1) * NS + j) * (size_t)traj_ld + c]);
    }
  }
}

template <int BASIS>
static void rollout_split(int split, const ModelDev* md, int Nc, int S, int H, const float* x0, const float* cand,
                          float* traj, long long traj_ld, hipStream_t st) {
  const unsigned grid = (unsigned)(((long long)Nc * split + 255) / 256);
  if (split == 2) rollout_split_kernel<BASIS, 2><<<grid, 256, 0, st>>>(md, Nc, S, H, x0, cand, traj, traj_ld);
  else if (split == 4) rollout_split_kernel<BASIS, 4><<<grid, 256, 0, st>>>(md, Nc, S, H, x0, cand, traj, traj_ld);
  else rollout_split_kernel<BASIS, 8><<<grid, 256, 0, st>>>(md, Nc, S, H, x0, cand, traj, traj_ld);
}

hipError_t launch_rollout_split(int basis, int split, const void* model, int Nc, int S, int H, const float* x0,
                                const float* cand, float* traj, long long traj_ld, hipStream_t st) {
  const ModelDev* md = (const ModelDev*)model;
  if (basis == MPMI_BASIS_RACE_CAR)
    rollout_split<MPMI_BASIS_RACE_CAR>(split, md, Nc, S, H, x0, cand, traj, traj_ld, st);
  else
    rollout_split<MPMI_BASIS_BALANCE_BOT>(split, md, Nc, S, H, x0, cand, traj, traj_ld, st);
  return hipGetLastError();
}

// Latency form for a basis given as data: one candidate over the 8 lanes of an
// aligned lane group.  Per step the group evaluates its atoms (lane h atoms h,
// h + 8, ...) into its row of an LDS table, lane h forms the products of
// features 8 h .. 8 h + 7 (their two row offsets in registers), and every
// lane sums all the products, taken from the lanes that hold them by DPP, times
// column h of K, which it holds in registers for the whole horizon.  A wave's
// LDS operations execute in order, so the exchanges need no wait or barrier,
// only the compiler kept from moving them.  Atoms, products and the sum over
// features take the one-lane step's operations in its order: the same bits.
// The one-lane step reads every feature's two atom numbers by dependent scalar
// loads and runs a latency-bound wave at 6.3 us per step (three-input car, 64
// features, 10,121 candidates, 25 steps: 159 us); here 0.7
// us per step, 28.6 us.  Exchanging the products through LDS instead of DPP took
// 38 us, as did the same with the verdict after the step instead of beside the
// next one.
constexpr int kCustomGroup = 8;
constexpr int kCustomW = 12;                    // x (8), u (4)
constexpr int kCustomAt = MPMI_MAX_ATOMS + 1;   // row strides that spread the groups over the banks
static_assert(MPMI_MAX_STATE == kCustomGroup && MPMI_MAX_DIM == 8 * kCustomGroup, "one column and eight features per lane");

// The eight products v[] of lane L of each quad, in order, times k[], added to
// y: v_fmac_f32 with its first operand taken from that lane by DPP (one rounding
// per feature, as fmaf).  In one statement, with the two wait states a DPP read
// needs after the instruction that wrote its operand.
template <int L>
__device__ __forceinline__ float add_eight(const float (&v)[8], const float* k, float y) {
#define MPMI_FMAC(i, j) "v_fmac_f32_dpp %0, %" #i ", %" #j " quad_perm:[%c17,%c17,%c17,%c17] row_mask:0xf bank_mask:0xf\n\t"
  asm("s_nop 1\n\t" MPMI_FMAC(1, 9) MPMI_FMAC(2, 10) MPMI_FMAC(3, 11) MPMI_FMAC(4, 12) MPMI_FMAC(5, 13)
          MPMI_FMAC(6, 14) MPMI_FMAC(7, 15) MPMI_FMAC(8, 16) "s_nop 0"
      : "+v"(y)
      : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]), "v"(k[0]), "v"(k[1]),
        "v"(k[2]), "v"(k[3]), "v"(k[4]), "v"(k[5]), "v"(k[6]), "v"(k[7]), "i"(L));
#undef MPMI_FMAC
  return y;
}

template <bool TRACK, bool RECHECK>
__global__ void __launch_bounds__(256)
tick_custom_split_kernel(const ModelDev* __restrict__ md, GenParams gp, int H, const float* __restrict__ x_t,
                         const float* __restrict__ u_user, const float* __restrict__ cand, Slot* __restrict__ slot,
                         mpmi_selection* __restrict__ out, int16_t* __restrict__ fv_out,
                         RecheckList* __restrict__ rl) {
  constexpr int NS = MPMI_MAX_STATE, MS = MPMI_MAX_INPUT, kGroups = 256 / kCustomGroup;
  __shared__ float sW[kGroups][kCustomW];
  __shared__ float sAt[kGroups][kCustomAt];
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int c = gid / kCustomGroup, h = gid % kCustomGroup, row = threadIdx.x / kCustomGroup;
  const bool valid = c < gp.n_cand + 1;
  const int n = md->n, m = md->m, D = md->dim, na = md->sys.n_atoms;
  float u0[MS];
#pragma unroll
  for (int j = 0; j < MS; ++j) u0[j] = (valid && j < m) ? cand_value(gp, md, cand, u_user, c, 0, j) : 0.0f;
  sW[row][h] = h < n ? x_t[h] : 0.0f;
  if (h < MS) {
    float v = u0[0];
#pragma unroll
    for (int j = 1; j < MS; ++j) v = h == j ? u0[j] : v;
    sW[row][NS + h] = v;
  }
  float kcol[MPMI_MAX_DIM];
#pragma unroll
  for (int f = 0; f < MPMI_MAX_DIM; ++f) kcol[f] = md->K[f][h];
  // Atom rows of this lane's features (one past the last feature: the row's
  // zero entry, so its product adds 0 * 0) and its atoms' kinds and variables.
  int fa[8], fb[8], kind[4], var[4];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    fa[i] = 8 * h + i < D ? md->sys.feat_a[8 * h + i] : MPMI_MAX_ATOMS;
    fb[i] = 8 * h + i < D ? md->sys.feat_b[8 * h + i] : MPMI_MAX_ATOMS;
  }
  if (h == 0) sAt[row][MPMI_MAX_ATOMS] = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int q = h + 8 * i;
    kind[i] = q < na ? md->sys.atom_kind[q] : MPMI_ATOM_ONE;
    const int v = q < na ? md->sys.atom_var[q] : 0;
    var[i] = v < n ? v : NS + (v - n);
  }
  SafetyRegs<NS, kMaxHarm, TRACK, RECHECK> sr;
  sr.load(md);
  // This lane's own box (the others' limits are dead after this).
  float lim = sr.lim[0], eps = RECHECK ? sr.eps[0] : 0.0f;
  bool boxed = sr.chk[0];
#pragma unroll
  for (int k = 1; k < NS; ++k) {
    lim = h == k ? sr.lim[k] : lim;
    boxed = h == k ? sr.chk[k] : boxed;
    if (RECHECK) eps = h == k ? sr.eps[k] : eps;
  }
  const bool lead = valid && h == 0;
  const float cst = lead ? cost_of<MS>(md, u0, u_user) : 0.0f;
  const int base = threadIdx.x & 63 & ~(kCustomGroup - 1);
  __syncthreads();
  int fv = H + 1;
  bool near = false;
  if (valid) {
    const int S = gp.n_seg;
    int nxt = (H + S - 1) / S;
    float own = 0.0f;  // component h of the state being checked
    for (int s = 1; s <= H; ++s) {
      if (s - 1 >= nxt) {
        const int g = ((s - 1) * S) / H;
        nxt = ((g + 1) * H + S - 1) / S;
        if (h < m) sW[row][NS + h] = cand_value(gp, md, cand, u_user, c, g, h);
        asm volatile("" ::: "memory");
      }
      // This lane's atoms, all read before the first is evaluated; the second
      // half only for more than 16 atoms (entries past the last are not read).
      auto atoms = [&](auto first) {
        constexpr int i0 = decltype(first)::value;
        const float w0 = sW[row][var[i0]], w1 = sW[row][var[i0 + 1]];
        const float w[2] = {w0, w1};
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float sn = __sinf(w[i]), cs = __cosf(w[i]);
          float a = 1.0f;
          a = kind[i0 + i] == MPMI_ATOM_VAR ? w[i] : a;
          a = kind[i0 + i] == MPMI_ATOM_SIN ? sn : a;
          a = kind[i0 + i] == MPMI_ATOM_COS ? cs : a;
          sAt[row][h + 8 * (i0 + i)] = a;
        }
      };
      atoms(std::integral_constant<int, 0>{});
      if (na > 16) atoms(std::integral_constant<int, 2>{});  // uniform
      asm volatile("" ::: "memory");
      float p[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) p[i] = sAt[row][fa[i]] * sAt[row][fb[i]];
      // The verdict of x_{s-1}, beside the step that forms x_s (the two chains
      // overlap; an unsafe x_{s-1} ends the rollout and x_s is dropped): lane h
      // tests component h's box, every lane the track, and one ballot combines
      // the group's tests (its lanes are all active: they leave the loop
      // together).  x_0, the current state, is not checked.
      bool nr = false;
      if (RECHECK) nr = fabsf(lim - fabsf(own)) < eps;
      bool ok = (fabsf(own) < lim) | !boxed;
      ok &= sr.track(group_lane<8, 0>(own), group_lane<8, 1>(own), &nr);
      // The products of lanes 0 .. 3 of the group in both quads, and those of
      // lanes 4 .. 7: one DPP move each (row_shr:4 into banks 1 and 3,
      // row_shl:4 into banks 0 and 2; the other banks keep their own).
      float pa[8], pb[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int v = __builtin_bit_cast(int, p[i]);
        pa[i] = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xF, 0xA, false));
        pb[i] = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(v, v, 0x104, 0xF, 0x5, false));
      }
      float y = 0.0f;
      y = add_eight<0>(pa, kcol, y);
      y = add_eight<1>(pa, kcol + 8, y);
      y = add_eight<2>(pa, kcol + 16, y);
      y = add_eight<3>(pa, kcol + 24, y);
      if (D > 32) {  // uniform
        y = add_eight<0>(pb, kcol + 32, y);
        y = add_eight<1>(pb, kcol + 40, y);
        y = add_eight<2>(pb, kcol + 48, y);
        y = add_eight<3>(pb, kcol + 56, y);
      }
      y = h < n ? y : 0.0f;
      sW[row][h] = y;
      asm volatile("" ::: "memory");
      const unsigned long long okm = __ballot(ok);
      if (s > 1) {
        near |= nr;
        if (((okm >> base) & 0xFFull) != 0xFFull) {
          fv = s - 1;
          break;
        }
      }
      own = y;
    }
    if (fv > H) {  // the last state
      bool nr = false;
      if (RECHECK) nr = fabsf(lim - fabsf(own)) < eps;
      bool ok = (fabsf(own) < lim) | !boxed;
      ok &= sr.track(group_lane<8, 0>(own), group_lane<8, 1>(own), &nr);
      near |= nr;
      const unsigned long long okm = __ballot(ok);
      if (((okm >> base) & 0xFFull) != 0xFFull) fv = H;
    }
    if (fv_out && h == 0) fv_out[c] = (int16_t)fv;
  }
  // Some lane of the group saw a near margin.
  const unsigned long long nm = __ballot(near);
  near = ((nm >> base) & 0xFFull) != 0;
  split_finish<MS, RECHECK>(md, gp, H, u_user, cand, slot, out, rl, lead, near, c, fv, cst);
}

// What every instance takes, in one place.
struct SplitLaunch {
  unsigned grid;
  int block, split;
  bool open_block;  // the descriptor leaves the workgroup's size to the library
  hipStream_t st;
  const ModelDev* md;
  GenParams gp;
  int H;
  const float *x_t, *u_user, *cand;
  Slot* slot;
  mpmi_selection* out;
  int16_t* fv;
  RecheckList* rl;
  const mpmi_selection* gate;
};

template <int BASIS, int SPLIT, int DEG, bool TRACK, bool RECHECK, bool GATED, int WAVES = 1>
static void split_launch(const SplitLaunch& a) {
  tick_split_kernel<BASIS, SPLIT, DEG, TRACK, RECHECK, GATED, WAVES><<<a.grid, a.block, 0, a.st>>>(
      a.md, a.gp, a.H, a.x_t, a.u_user, a.cand, a.slot, a.out, a.fv, a.rl, a.gate);
}
template <int BASIS, int DEG, bool TRACK, bool RECHECK, bool GATED>
static void split_lanes(const SplitLaunch& a) {
  if (a.split == 2 && (long long)a.grid * a.block > 64ll * 4 * device_cu_count()) {
    if constexpr (BASIS == MPMI_BASIS_RACE_CAR) return split_launch<BASIS, 2, DEG, TRACK, RECHECK, GATED, 2>(a);
    // More than a wave per SIMD, and a short step: as many candidates to a
    // workgroup, and so as few publications, as in the one-lane form.  Balance bot,
    // H = 50, workgroups of 512 against 256: 65,536 candidates 17.3 and 18.9 us, 131,072
    // 21.7 and 24; all ending in the first step, 9.1 and 10.8, 12.2 and 15.4 (one lane 9.1
    // and 10.9).  The race car's own 65,536 took 51 and 48.
    if (a.open_block) {
      SplitLaunch w = a;
      w.block = 512;
      w.grid = (a.grid + 1) / 2;
      return split_launch<BASIS, 2, DEG, TRACK, RECHECK, GATED>(w);
    }
  }
  if (a.split == 2) split_launch<BASIS, 2, DEG, TRACK, RECHECK, GATED>(a);
  else if (a.split == 4) split_launch<BASIS, 4, DEG, TRACK, RECHECK, GATED>(a);
  else split_launch<BASIS, 8, DEG, TRACK, RECHECK, GATED>(a);
}
template <bool RECHECK, bool GATED>
static void split_race_car(const mpmi_system& sys, const SplitLaunch& a) {
  if (!sys.has_track) split_lanes<MPMI_BASIS_RACE_CAR, 1, false, RECHECK, GATED>(a);
  else if (track_degree(sys) <= kSmallTrackDeg)
    split_lanes<MPMI_BASIS_RACE_CAR, kSmallTrackDeg, true, RECHECK, GATED>(a);
  else split_lanes<MPMI_BASIS_RACE_CAR, kMaxHarm, true, RECHECK, GATED>(a);
}
template <bool TRACK, bool RECHECK>
static void split_custom(const SplitLaunch& a) {
  tick_custom_split_kernel<TRACK, RECHECK><<<a.grid, a.block, 0, a.st>>>(a.md, a.gp, a.H, a.x_t, a.u_user, a.cand,
                                                                        a.slot, a.out, a.fv, a.rl);
}
template <bool RECHECK>
static void split_basis(const mpmi_system& sys, const SplitLaunch& a) {
  if (sys.basis == MPMI_BASIS_CUSTOM) {
    if (sys.has_track) split_custom<true, RECHECK>(a);
    else split_custom<false, RECHECK>(a);
  } else if (sys.basis == MPMI_BASIS_RACE_CAR) {
    if (a.gate) split_race_car<RECHECK, true>(sys, a);
    else split_race_car<RECHECK, false>(sys, a);
  } else {
    if (sys.has_track) split_lanes<MPMI_BASIS_BALANCE_BOT, kMaxHarm, true, RECHECK, false>(a);
    else split_lanes<MPMI_BASIS_BALANCE_BOT, 1, false, RECHECK, false>(a);
  }
}

hipError_t launch_tick_split(const mpmi_system& sys, int split, const void* model, const mpmi_tick_desc& d,
                             const float* x_t, const float* u_user, const float* cand, void* slot,
                             mpmi_selection* out, int16_t* fv, hipStream_t st, const mpmi_selection* gate,
                             void* recheck, int recheck_capacity, int recheck_grid) {
  if (gate && sys.basis != MPMI_BASIS_RACE_CAR) return hipErrorInvalidValue;  // only race-car ticks are gated
  SplitLaunch a;
  a.gp.seed = d.seed;
  a.gp.tick = d.tick;
  a.gp.loop = d.loop;
  a.gp.gen = d.gen;
  a.gp.n_cand = d.n_cand;
  a.gp.n_seg = d.n_seg;
  for (int j = 0; j < MPMI_MAX_INPUT; ++j) a.gp.grid[j] = d.grid[j] > 0 ? d.grid[j] : 1;
  a.block = d.block > 0 ? d.block : 256;
  a.open_block = d.block == 0;
  a.split = split;
  a.grid = (unsigned)((((long long)d.n_cand + 1) * split + a.block - 1) / a.block);
  a.st = st;
  a.md = (const ModelDev*)model;
  a.H = d.horizon;
  a.x_t = x_t;
  a.u_user = u_user;
  a.cand = cand;
  a.slot = (Slot*)slot;
  a.out = out;
  a.fv = fv;
  a.rl = (RecheckList*)recheck;
  a.gate = gate;
  if (recheck) split_basis<true>(sys, a);
  else split_basis<false>(sys, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !recheck) return e;
  return launch_recheck64(sys, model, d, x_t, u_user, cand, slot, out, fv, recheck, recheck_capacity, recheck_grid,
                          st, gate);
}

}  // namespace mpmi
