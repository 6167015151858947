// belief.hpp -- device side of the (beta, g) belief update, Eq. (beta_update)
// in the log form of Sec. III-B, for one human per thread block.
#pragma once

#include "dfloat.hpp"
#include "model.hpp"

namespace capred {

constexpr int kBeliefThreads = 256;       // threads of an update block of a plan
constexpr int kBeliefThreadsWide = 1024;  // threads of the single-human entry point's blocks
constexpr int kMaxChunkT = 64;     // transitions per chunk

// NT threads per block.  The Delta buffer holds four values per thread: 8 KiB
// in a plan, where the update fits beside the rollout blocks of a busy CU.
template <int NT>
struct BeliefShared {
  static constexpr int kDeltas = 4 * NT;
  static constexpr int kTerms = NT > CAP_MAX_J ? NT : CAP_MAX_J;
  BeliefModel m;           // staged: lanes read its tables by their own index
  double dl[kDeltas];      // Delta of a chunk of transitions x goals x controls
  double term[kTerms];     // policy terms of the chunk, [transition][pair]
  int ks[kMaxChunkT];
};

// Control recovered from one observed transition (the nearest control):
// heading k* = argmax_k <dz, (cos, sin)theta_k> with the lowest k on ties, then
// the speed whose step v_s dt is nearest to that projection (lowest s on
// ties); returns u* = s* K + k*, or -1 when the displacement is below 1e-9 m.
__device__ __forceinline__ int recover_control(const BeliefModel& m, float dx, float dy) {
  if (fmaf(dx, dx, dy * dy) < 1e-18f) return -1;
  int ks = 0;
  float best = -INFINITY;
  for (int k = 0; k < m.K; ++k) {
    const float v = fmaf(dx, m.cth[k], dy * m.sth[k]);
    if (v > best) {
      best = v;
      ks = k;
    }
  }
  int ss = 0;
  float err = INFINITY;
  for (int s = 0; s < m.S; ++s) {
    const float e = fabsf(m.vdt[s] - best);
    if (e < err) {
      err = e;
      ss = s;
    }
  }
  return ss * m.K + ks;
}

// log pi(u* | z; beta_b, g) for every b over the U controls in plain FP32 (the
// trajectory log-likelihood's terms: its bar is relative to |LL|, a sum of
// hundreds of terms, so FP32 logits meet it; the posterior update uses the
// compensated policy_delta and policy_term_lanes below).
// Delta_u = |a + s_u| - |a| with a = z - g carried as an unevaluated sum
// (hi + lo, exact subtraction), from the cancellation-free quotient
// (2 a.s_u + |s_u|^2) / (|a + s_u| + |a|); then l_u = -beta Delta_u and
// log pi = l_{u*} - max l - log sum exp(l - max l).  NMAX bounds U.
// exp(x) for the policy's shifted logits (x <= 0) through the hardware base-2
// exponential: one multiply by log2(e) and V_EXP_F32.  Relative error below
// 2e-7 + |x| 6e-8, against 1e-5 for the posterior and log-likelihood bars.
__device__ __forceinline__ float exp_nonpos(float x) { return fast_exp2(x * kLog2e); }

// Hardware base-2 logarithm (within 1 ulp for the normal arguments it gets
// here: sums of K weights whose largest is 1).
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }
constexpr float kLn2 = 0.6931471805599453f;

template <int NMAX>
__device__ __forceinline__ void policy_terms(const BeliefModel& m, float zx, float zy, int ks,
                                             float gx, float gy, const float* beta, int B,
                                             float* out) {
  if (ks < 0) {
    for (int b = 0; b < B; ++b) out[b] = 0.f;
    return;
  }
  const int U = m.U;
  const float ax = zx - gx, bx = ax - zx;
  const float ax_lo = (zx - (ax - bx)) + (-gx - bx);
  const float ay = zy - gy, by = ay - zy;
  const float ay_lo = (zy - (ay - by)) + (-gy - by);
  const float D2 = fmaf(ax, ax, ay * ay);
  const float D = sqrtf(D2);
  const float ax2 = ax + ax, ay2 = ay + ay;
  float dl[NMAX];
  float dmin = INFINITY;
  for (int k = 0; k < U; ++k) {
    const float corr = fmaf(2.f * ax_lo, m.sx[k], fmaf(2.f * ay_lo, m.sy[k], m.s2[k]));
    const float n = fmaf(ax2, m.sx[k], fmaf(ay2, m.sy[k], corr));
    const float d = sqrtf(fmaxf(D2 + n, 0.f));
    dl[k] = n / (d + D);
    dmin = fminf(dmin, dl[k]);
  }
  for (int b = 0; b < B; ++b) {
    const float nbt = -beta[b];
    // max_k (nbt dl_k) for nbt <= 0: the rounded product is monotone in dl_k
    const float mx = nbt * dmin;
    float s = 0.f;
    for (int k = 0; k < U; ++k) s += exp_nonpos(nbt * dl[k] - mx);
    out[b] = (nbt * dl[ks] - mx) - logf(s);
  }
}

// policy_terms for a model of exactly KT controls (KT > 0), for the batched
// log-likelihood: the loops over the controls are unrolled (the KT distance
// chains are independent, which the runtime-length loops above hide from the
// scheduler), the chosen control's Delta is evaluated from its own step by the
// same operations (st: (sx, sy, s2) per control in LDS), each beta's term goes to
// out(b, term) at once, and the distances take the hardware square root
// and reciprocal (within 1 ulp) in place of the IEEE ones: the log-likelihood's
// error bar is 1e-5 of its magnitude, not the posterior's absolute 1e-5.
template <int KT, class Out>
__device__ __forceinline__ void policy_terms_fixed(const float4* st, float zx, float zy,
                                                   int ks, float gx, float gy,
                                                   const float* beta, int B, Out out) {
  const float ax = zx - gx, bx = ax - zx;
  const float ax_lo = (zx - (ax - bx)) + (-gx - bx);
  const float ay = zy - gy, by = ay - zy;
  const float ay_lo = (zy - (ay - by)) + (-gy - by);
  const float D2 = fmaf(ax, ax, ay * ay);
  const float D = fast_sqrt(D2);
  const float ax2 = ax + ax, ay2 = ay + ay;
  auto delta = [&](float4 c) {
    const float corr = fmaf(2.f * ax_lo, c.x, fmaf(2.f * ay_lo, c.y, c.z));
    const float n = fmaf(ax2, c.x, fmaf(ay2, c.y, corr));
    const float d = fast_sqrt(fmaxf(D2 + n, 0.f));
    return n * fast_rcp(d + D);
  };
  const float dks = delta(st[ks]);
  float dl[KT];
  float dmin = INFINITY;
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    dl[k] = delta(st[k]);
    dmin = fminf(dmin, dl[k]);
  }
  // logits in base 2: a_k = -beta log2(e) Delta_k - c with the shift c = -beta
  // log2(e) min_k Delta_k (rounded), so pi_k = 2^a_k / sum_j 2^a_j for any c
  // and the term is (a_k* - log2 sum_j 2^a_j) ln 2; each exponent is one FMA
  for (int b = 0; b < B; ++b) {
    const float nb2 = -beta[b] * kLog2e;
    const float mx2 = nb2 * dmin;
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < KT; ++k) s += fast_exp2(fmaf(nb2, dl[k], -mx2));
    out(b, (fmaf(nb2, dks, -mx2) - fast_log2(s)) * kLn2);
  }
}

// Delta_u = |a + s_u| - |a| for a = z - g, the distance change of control u
// that the policy's logits -beta Delta_u are built from (the shift-invariant
// form of beta Q).  The posterior multiplies up to thousands of these terms
// into a log that must stay within 1e-5 of the exact one, and a logit's
// rounding error scales with beta |s| (about 15 at beta = 100 and a 0.15 m
// step): plain FP32 Delta errs by a few 1e-6 per transition.  So Delta is
// evaluated in compensated FP32 (hi + lo pairs, about 46 bits): a = z - g
// exactly, |a|^2, n_u = 2 a.s_u + |s_u|^2 and the cancellation-free quotient
// n_u / (|a + s_u| + |a|), rounded once to FP64, where the rest of the term
// (the product with beta and the log-sum-exp over the controls) runs.
struct GoalOffset {
  dfl ax, ay, D2, D;
};

__device__ __forceinline__ GoalOffset goal_offset(float zx, float zy, float gx, float gy) {
  GoalOffset o;
  o.ax = two_sum(zx, -gx);
  o.ay = two_sum(zy, -gy);
  o.D2 = df_add(df_mul(o.ax, o.ax), df_mul(o.ay, o.ay));
  o.D = df_sqrt(o.D2);
  return o;
}

__device__ __forceinline__ double policy_delta(const GoalOffset& o, float sx, float sy) {
  const dfl s2 = df_add(two_prod(sx, sx), two_prod(sy, sy));
  const dfl dot = df_add(df_mul_f(o.ax, sx), df_mul_f(o.ay, sy));
  const dfl n = df_add(dfl{2.f * dot.hi, 2.f * dot.lo}, s2);
  const dfl d = df_sqrt(df_add(o.D2, n));
  return df_to_double(df_div(n, df_add(d, o.D)));
}

// Sum and minimum over the L = 8 or 16 lanes of a group (aligned), in every
// lane, by DPP moves: neighbours, pairs, then mirrored halves of 8 and of 16.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;

template <int L>
__device__ __forceinline__ double lanes_sum(double v) {
  v += dpp_move<kDppXor1>(v);
  v += dpp_move<kDppXor2>(v);
  v += dpp_move<kDppHalfMirror>(v);
  if constexpr (L == 16) v += dpp_move<kDppMirror>(v);
  return v;
}
template <int L>
__device__ __forceinline__ double lanes_min(double v) {
  v = fmin(v, dpp_move<kDppXor1>(v));
  v = fmin(v, dpp_move<kDppXor2>(v));
  v = fmin(v, dpp_move<kDppHalfMirror>(v));
  if constexpr (L == 16) v = fmin(v, dpp_move<kDppMirror>(v));
  return v;
}

// log pi(u* | z; beta, g) from the U values Delta_u, by L lanes together (lane
// `sub` takes every L-th control): l_u = -beta Delta_u and
// log pi = (l_{u*} - max l) - log sum exp(l - max l), FP64.  The largest logit
// belongs to the smallest Delta (beta > 0, rounding is monotone).
template <int L>
__device__ __forceinline__ double policy_term_lanes(const double* dl, int U, int ks, double beta,
                                                    int sub) {
  double dmin = INFINITY;
  for (int u = sub; u < U; u += L) dmin = fmin(dmin, dl[u]);
  const double mx = -beta * lanes_min<L>(dmin);
  double s = 0.0;
  for (int u = sub; u < U; u += L) s += exp(-beta * dl[u] - mx);
  return (-beta * dl[ks] - mx) - log(lanes_sum<L>(s));
}

// Adds sum_t ell_t(g, b) of the goals [g0, g1) and betas [b0, b1) to
// log_belief (not yet normalised).  Every Delta of a chunk of transitions x
// goals x controls is evaluated once, in parallel, into LDS; groups of L lanes
// then take the policy terms of the chunk's (transition, pair)s one at a time,
// and one thread per pair adds that pair's terms in transition order.  So a
// pair's sum does not depend on the chunks, the block size or the share of the
// pairs that the block has: the single-human call, a plan's shared update and
// its per-human form give the same bits.  What bounds it is the latency of
// dependent FP64 work, so every level (transitions, goals, pairs, controls) is
// spread over the lanes: with one thread per pair running its controls'
// exponentials one after another and the transitions in series, 40 observations
// of a 96-control model over 21 goals x 5 betas took 2524 us.  Now 13.0 us for
// that history (one block per pair) and 8.4 us for 10 observations of 8 controls
// over 2 goals x 4 betas (38.7 us before), most of it the round trips and chains
// of one term.
template <int NT, int L>
__device__ __forceinline__ void belief_terms(const float* __restrict__ obs,
                                             int n_obs, double* log_belief, int g0,
                                             int g1, int b0, int b1, BeliefShared<NT>& sh) {
  const BeliefModel& m = sh.m;
  const int tid = threadIdx.x;
  const int B = m.B, U = m.U, nb = b1 - b0;
  constexpr int kGroups = NT / L;
  constexpr int kPer = (CAP_MAX_J + NT - 1) / NT;   // pairs of a thread
  const int grp = tid / L, sub = tid % L;
  const int gstep = max(1, min(g1 - g0, sh.kDeltas / U));
  for (int gb = g0; gb < g1; gb += gstep) {
    const int gn = min(gstep, g1 - gb), pairs = gn * nb;   // pairs <= CAP_MAX_J <= kTerms
    const int tstep = min(kMaxChunkT, min(sh.kDeltas / (gn * U), sh.kTerms / pairs));
    double sum[kPer];
#pragma unroll
    for (int r = 0; r < kPer; ++r) sum[r] = 0.0;
    for (int t0 = 0; t0 < n_obs; t0 += tstep) {
      const int tn = min(tstep, n_obs - t0);
      for (int i = tid; i < tn; i += NT) {
        const float* z = obs + 2 * (t0 + i);
        sh.ks[i] = recover_control(m, z[2] - z[0], z[3] - z[1]);
      }
      for (int item = tid; item < tn * gn * U; item += NT) {
        const int tg = item / U, u = item - tg * U;
        const int tl = tg / gn, gl = tg - tl * gn;
        const float zx = obs[2 * (t0 + tl)], zy = obs[2 * (t0 + tl) + 1];
        const GoalOffset o = goal_offset(zx, zy, m.gx[gb + gl], m.gy[gb + gl]);
        sh.dl[item] = policy_delta(o, m.sx[u], m.sy[u]);
      }
      __syncthreads();
      for (int k = grp; k < tn * pairs; k += kGroups) {
        const int tl = k / pairs, p = k - tl * pairs, gl = p / nb;
        const double beta = (double)m.beta[b0 + p - gl * nb];
        const int ks = sh.ks[tl];
        double ell = 0.0;   // below 1e-9 m: no information
        if (ks >= 0) ell = policy_term_lanes<L>(sh.dl + (tl * gn + gl) * U, U, ks, beta, sub);
        if (sub == 0) sh.term[k] = ell;
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < kPer; ++r) {
        const int p = tid + r * NT;
        if (p < pairs) {
#pragma unroll 8
          for (int tl = 0; tl < tn; ++tl) sum[r] += sh.term[tl * pairs + p];
        }
      }
      // (the next chunk's terms come after another barrier)
    }
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
      const int p = tid + r * NT, gl = p / nb;
      if (p < pairs) log_belief[(gb + gl) * B + b0 + p - gl * nb] += sum[r];
    }
  }
  __syncthreads();
}

template <int NT>
__device__ __forceinline__ void belief_terms_any(const BeliefModel& m, const float* obs, int n_obs,
                                                 double* log_belief, int g0, int g1, int b0,
                                                 int b1, BeliefShared<NT>& sh) {
  // stage the model first: its tables lie in the kernel's arguments or in a
  // slot's descriptor, and each dependent read of those costs a round trip
  static_assert(sizeof(BeliefModel) % 4 == 0, "copied as words");
  for (int i = threadIdx.x; i < (int)(sizeof(BeliefModel) / 4); i += NT)
    reinterpret_cast<uint32_t*>(&sh.m)[i] = reinterpret_cast<const uint32_t*>(&m)[i];
  __syncthreads();
  if (m.U <= 8) belief_terms<NT, 8>(obs, n_obs, log_belief, g0, g1, b0, b1, sh);
  else belief_terms<NT, 16>(obs, n_obs, log_belief, g0, g1, b0, b1, sh);
}

// Renormalises the J entries of log_belief by one FP64 log-sum-exp and writes
// belief_out = exp(log_belief) (nullable).  One wavefront (the caller's first;
// the others return): at most eight pairs per lane, and no barrier between the
// steps of a chain whose latency is all there is to pay.
__device__ __forceinline__ void belief_normalize(int J, double* log_belief, double* belief_out) {
  constexpr int kPerLane = CAP_MAX_J / 64;
  if (threadIdx.x >= 64) return;
  const int lane = threadIdx.x;
  double v[kPerLane];
  double mx = -INFINITY;
#pragma unroll
  for (int r = 0; r < kPerLane; ++r) {
    const int j = lane + r * 64;
    v[r] = j < J ? log_belief[j] : -INFINITY;
    mx = fmax(mx, v[r]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
  double s = 0.0;
#pragma unroll
  for (int r = 0; r < kPerLane; ++r)
    if (lane + r * 64 < J) s += exp(v[r] - mx);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  const double lse = mx + log(s);
#pragma unroll
  for (int r = 0; r < kPerLane; ++r) {
    const int j = lane + r * 64;
    if (j < J) {
      const double lb = v[r] - lse;
      log_belief[j] = lb;
      if (belief_out) belief_out[j] = exp(lb);
    }
  }
}

}  // namespace capred
