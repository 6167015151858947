// loglik.hip -- batched trajectory log-likelihood (product form of
// Eq. beta_update over each track) and its adjoint with respect to the goal
// positions and log beta.  A block takes one track (and, beyond 21 goals, a
// slice of the goals): the controls of its steps are recovered once into LDS,
// each lane keeps one goal, and a wave takes chunks of 64 / goals consecutive
// steps, the block's waves in turn.  So a track leaves idle lanes only in its
// last chunk, and the waves that have no chunk left end.  Both kernels are bound
// by the issue of their (beta, heading) terms.  FP32 policy terms are
// accumulated per lane in FP64 and reduced over lanes and waves in a fixed
// order, so for a given launch shape results are bitwise reproducible.  The
// adjoint writes per-track partials to the workspace and a second kernel sums
// them in a fixed order (no atomics).
#include <algorithm>
#include <mutex>

#include "belief.hpp"

namespace capred {

constexpr int kStepBuf = 1024;    // recovered controls of a block held in LDS

struct LLArgs {
  BeliefModel m;           // K, continuous steps and heading unit vectors
  const float* tracks;     // [N][Tmax+1][2]
  const int32_t* lengths;  // [N]
  int32_t N, Tmax, G, B, per_track;
  const float* goals;      // [G][2]
  const float* log_beta;   // [B] or [N][B]
};

// A block's share of the work: L lanes per goal, goals [g0, g0 + gn) of a track.
struct LLShape {
  int L, slice;   // lanes per goal, goals per slice (L * slice <= 64)
};

// The step table in LDS, (sx, sy, s2) of a control in one read.  (3 KT scalars do
// not fit the scalar registers at KT = 32; spilled, each use is a VALU access.)
__device__ __forceinline__ void load_steps(const BeliefModel& m, float4* st) {
  for (int k = threadIdx.x; k < m.K; k += blockDim.x)
    st[k] = make_float4(m.sx[k], m.sy[k], m.s2[k], 0.f);
}

// Recovers the controls of steps [t0, t0 + n) of a track into ks (255: none).
__device__ __forceinline__ void recover_steps(const BeliefModel& m, const float* z, int t0, int n,
                                              uint8_t* ks) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const float* p = z + 2 * (t0 + i);
    ks[i] = (uint8_t)recover_control(m, p[2] - p[0], p[3] - p[1]);
  }
}

// Sum over the L lanes of this lane's goal, complete in its first lane (sub 0).
__device__ __forceinline__ double goal_sum(double v, int sub, int L) {
  for (int o = 1; o < L; o <<= 1) {
    const double x = __shfl_down(v, o, 64);
    if (sub + o < L) v += x;
  }
  return v;
}

template <int KT>
__global__ void __launch_bounds__(1024)
    loglik_kernel(const LLArgs a, const LLShape sh, double* __restrict__ LL) {
  __shared__ uint8_t ks[kStepBuf];
  __shared__ float4 st[CAP_MAX_K];
  __shared__ float beta[CAP_MAX_B];
  extern __shared__ double dyn[];    // sums [B][threads], then [waves][goals of the slice][B]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, W = blockDim.x >> 6;
  const int n = blockIdx.x, g0 = (int)blockIdx.y * sh.slice, gn = min(sh.slice, a.G - g0);
  const int gl = lane / sh.L, sub = lane - gl * sh.L, B = a.B;
  const bool on = gl < gn;
  const int g = g0 + (on ? gl : 0);
  const int len = a.lengths[n];
  const float* z = a.tracks + (size_t)n * (a.Tmax + 1) * 2;
  const float* lb = a.per_track ? a.log_beta + (size_t)n * B : a.log_beta;
  const float gx = a.goals[2 * g], gy = a.goals[2 * g + 1];
  const int nthr = blockDim.x;
  double* acc = dyn + threadIdx.x;
  double* part = dyn + (size_t)B * nthr;
  for (int b = threadIdx.x; b < B; b += nthr) beta[b] = expf(lb[b]);
  for (int b = 0; b < B; ++b) acc[b * nthr] = 0.0;
  if constexpr (KT > 0) load_steps(a.m, st);   // (the general form reads the arguments)
  for (int t0 = 0; t0 < len; t0 += kStepBuf) {
    const int tn = min(kStepBuf, len - t0);
    __syncthreads();
    recover_steps(a.m, z, t0, tn, ks);
    __syncthreads();
    for (int i = wave * sh.L + sub; i < tn; i += W * sh.L) {
      const int k = ks[i];
      if (!on || k == 255) continue;
      asm volatile("" ::: "memory");   // the table stays in LDS: held, it takes 3 KT registers
      const float zx = z[2 * (t0 + i)], zy = z[2 * (t0 + i) + 1];
      if constexpr (KT > 0) {
        policy_terms_fixed<KT>(st, zx, zy, k, gx, gy, beta, B,
                               [&](int b, float v) { acc[b * nthr] += (double)v; });
      } else {
        float terms[CAP_MAX_B];
        policy_terms<CAP_MAX_K>(a.m, zx, zy, k, gx, gy, beta, B, terms);
        for (int b = 0; b < B; ++b) acc[b * nthr] += (double)terms[b];
      }
    }
  }
  for (int b = 0; b < B; ++b) {
    const double s = goal_sum(acc[b * nthr], sub, sh.L);
    if (on && sub == 0) part[(wave * gn + gl) * B + b] = s;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < gn * B; i += blockDim.x) {
    double s = part[i];
    for (int w = 1; w < W; ++w) s += part[w * gn * B + i];
    const int q = i / B, b = i - q * B;
    LL[((size_t)n * B + b) * a.G + g0 + q] = s;
  }
}

// Per-step adjoint terms for one (z, goal) and every beta:
//   d ell/d g        = -beta (E_p[yhat] - yhat_{k*}),
//   d ell/d log beta = -beta (Delta_{k*} - E_p[Delta]),
// with yhat_k = (a + s_k)/d_k and, to avoid cancellation between unit vectors,
//   yhat_k - yhat_* = a (Delta_* - Delta_k)/(d_k d_*) + s_k/d_k - s_*/d_*.
//
//
// KT > 0 (the model has KT headings, every loop over them unrolled): the unit
// vectors' differences are formed once per heading (from each distance's own
// square root; the chosen heading's is exactly zero).  Per beta the KT
// probabilities give four moments, of even and odd headings apart and Delta
// relative to its minimum (shorter FP32 sums; where the chosen heading is the
// unlikely one its part is not rounded with the sum), which are added over betas
// and steps in FP64; the per-lane sums of d log beta are kept in LDS.  Four arrays of KT
// values live over the betas: at K = 32, 160 registers and three waves per SIMD,
// so blocks of at most 768 threads (1024 tracks x 200 steps x 8 goals x 9 betas:
// 150 us; at 128 registers, the differences of Delta formed anew for every beta,
// 160).  One coefficient per heading in place of the two goal moments takes 135,
// but adds the betas in FP32.
template <int KT>
__global__ void __launch_bounds__(KT > 16 ? 768 : 1024)
    loglik_backward_kernel(const LLArgs a, const LLShape sh, const double* __restrict__ dLL,
                           double* __restrict__ ws_g, double* __restrict__ ws_b) {
  constexpr int KM = KT > 0 ? KT : CAP_MAX_K;
  __shared__ uint8_t ks[kStepBuf];
  __shared__ float4 st[CAP_MAX_K];
  __shared__ float beta[CAP_MAX_B];
  // sums [waves][2 x 64], then ab [B][threads], then w [B][64] (FP32)
  extern __shared__ double lds[];
  const int nthr = blockDim.x, W = nthr >> 6;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = blockIdx.x, g0 = (int)blockIdx.y * sh.slice, gn = min(sh.slice, a.G - g0);
  const int gl = lane / sh.L, sub = lane - gl * sh.L, B = a.B;
  const bool on = gl < gn;
  const int g = g0 + (on ? gl : 0);
  const int K = KT > 0 ? KT : a.m.K;
  double* red = lds;
  double* dyn = lds + 2 * nthr;
  const int len = a.lengths[n];
  const float* z = a.tracks + (size_t)n * (a.Tmax + 1) * 2;
  const float* lb = a.per_track ? a.log_beta + (size_t)n * B : a.log_beta;
  const float gx = a.goals[2 * g], gy = a.goals[2 * g + 1];
  double* ab = dyn + tid;
  float* wl = reinterpret_cast<float*>(dyn + (size_t)B * nthr) + gl;
  for (int b = tid; b < B; b += nthr) beta[b] = expf(lb[b]);
  for (int i = tid; i < B * gn; i += nthr) {
    const int b = i / gn, q = i - b * gn;
    reinterpret_cast<float*>(dyn + (size_t)B * nthr)[b * 64 + q] =
        (float)dLL[((size_t)n * B + b) * a.G + g0 + q];
  }
  for (int b = 0; b < B; ++b) ab[b * nthr] = 0.0;
  load_steps(a.m, st);
  double agx = 0.0, agy = 0.0;
  for (int t0 = 0; t0 < len; t0 += kStepBuf) {
    const int tn = min(kStepBuf, len - t0);
    __syncthreads();
    recover_steps(a.m, z, t0, tn, ks);
    __syncthreads();
    for (int i = wave * sh.L + sub; i < tn; i += W * sh.L) {
      const int kc = ks[i];
      if (!on || kc == 255) continue;
      asm volatile("" ::: "memory");   // the table stays in LDS, as in the forward
      const float zx = z[2 * (t0 + i)], zy = z[2 * (t0 + i) + 1];
      const float ax = zx - gx, bx = ax - zx;
      const float ax_lo = (zx - (ax - bx)) + (-gx - bx);
      const float ay = zy - gy, by = ay - zy;
      const float ay_lo = (zy - (ay - by)) + (-gy - by);
      const float D2 = fmaf(ax, ax, ay * ay);
      const float D = fast_sqrt(D2);
      const float4 own = st[kc];
      const float sxs = own.x, sys = own.y;
      // hardware square root and reciprocal, as in the forward's fixed-K path
      auto delta = [&](float sx, float sy, float s2, float* d) {
        const float corr = fmaf(2.f * ax_lo, sx, fmaf(2.f * ay_lo, sy, s2));
        const float nk = fmaf(ax + ax, sx, fmaf(ay + ay, sy, corr));
        *d = fast_sqrt(fmaxf(D2 + nk, 0.f));
        return nk * fast_rcp(*d + D);
      };
      float ds;
      const float dls = delta(sxs, sys, own.z, &ds);
      if constexpr (KT > 0) {
        float dl[KM], ux[KM], uy[KM];
        float dmin = INFINITY;
        // yhat_k - yhat_*  (yhat := 0 where the distance is 0)
        const float rds = ds > 0.f ? fast_rcp(ds) : 0.f;
        // s_*/d_* with its rounding error, so that k = * leaves exactly zero
        const float qx = sxs * rds, qy = sys * rds;
        const float qx_lo = fmaf(sxs, rds, -qx), qy_lo = fmaf(sys, rds, -qy);
#pragma unroll
        for (int k = 0; k < KM; ++k) {
          float d;
          const float4 c = st[k];
          dl[k] = delta(c.x, c.y, c.z, &d);
          dmin = fminf(dmin, dl[k]);
          const float rk = d > 0.f ? fast_rcp(d) : 0.f;
          if (d > 0.f && ds > 0.f) {
            const float v = (dls - dl[k]) * (rk * rds);
            ux[k] = fmaf(ax, v, fmaf(c.x, rk, -qx) - qx_lo);
            uy[k] = fmaf(ay, v, fmaf(c.y, rk, -qy) - qy_lo);
          } else {
            ux[k] = (ax + c.x) * rk - (ax + sxs) * rds;
            uy[k] = (ay + c.y) * rk - (ay + sys) * rds;
          }
        }
        for (int b = 0; b < B; ++b) {
          // base-2 exponents with the shift folded into one FMA (p is a ratio,
          // so the shift's rounding cancels)
          const float be = beta[b], nb2 = -be * kLog2e, mx2 = nb2 * dmin, w = wl[b * 64];
          float s2[2] = {}, ex2[2] = {}, ey2[2] = {}, ed2[2] = {};   // even and odd headings
#pragma unroll
          for (int k = 0; k < KM; ++k) {
            const float p = fast_exp2(fmaf(nb2, dl[k], -mx2));
            s2[k & 1] += p;
            ex2[k & 1] = fmaf(p, ux[k], ex2[k & 1]);
            ey2[k & 1] = fmaf(p, uy[k], ey2[k & 1]);
            ed2[k & 1] = fmaf(p, dl[k] - dmin, ed2[k & 1]);
          }
          const float inv = 1.f / (s2[0] + s2[1]);
          // E[yhat] - yhat_* = ex/s ; E[Delta - min] - (Delta_* - min) = ed/s - ...
          agx -= (double)(w * (be * ((ex2[0] + ex2[1]) * inv)));
          agy -= (double)(w * (be * ((ey2[0] + ey2[1]) * inv)));
          ab[b * nthr] += (double)(w * (be * fmaf(ed2[0] + ed2[1], inv, dmin - dls)));
        }
      } else {
        // any K: per (beta, heading), without per-heading arrays beyond dl and dk
        float dl[KM], dk[KM];
        for (int k = 0; k < K; ++k) dl[k] = delta(a.m.sx[k], a.m.sy[k], a.m.s2[k], dk + k);
        for (int b = 0; b < B; ++b) {
          const float be = beta[b], nbt = -be, w = wl[b * 64];
          float mx = -INFINITY;
          for (int k = 0; k < K; ++k) mx = fmaxf(mx, nbt * dl[k]);
          float s = 0.f, ex = 0.f, ey = 0.f, ed = 0.f;
          for (int k = 0; k < K; ++k) {
            const float p = exp_nonpos(nbt * dl[k] - mx);
            s += p;
            // yhat_k - yhat_*  (yhat := 0 where the distance is 0)
            float ux, uy;
            if (dk[k] > 0.f && ds > 0.f) {
              const float v = (dls - dl[k]) / (dk[k] * ds);
              ux = fmaf(ax, v, a.m.sx[k] / dk[k] - sxs / ds);
              uy = fmaf(ay, v, a.m.sy[k] / dk[k] - sys / ds);
            } else if (dk[k] > 0.f) {
              ux = (ax + a.m.sx[k]) / dk[k];
              uy = (ay + a.m.sy[k]) / dk[k];
            } else if (ds > 0.f) {
              ux = -(ax + sxs) / ds;
              uy = -(ay + sys) / ds;
            } else {
              ux = 0.f;
              uy = 0.f;
            }
            ex = fmaf(p, ux, ex);
            ey = fmaf(p, uy, ey);
            ed = fmaf(p, dl[k] - dls, ed);
          }
          const float inv = 1.f / s;
          // E[yhat] - yhat_* = ex/s ; E[Delta] - Delta_* = ed/s
          agx += (double)(w * (nbt * (ex * inv)));
          agy += (double)(w * (nbt * (ey * inv)));
          ab[b * nthr] += (double)(w * (be * (ed * inv)));
        }
      }
    }
  }
  const double sgx = goal_sum(agx, sub, sh.L), sgy = goal_sum(agy, sub, sh.L);
  if (on && sub == 0) {
    red[wave * 128 + 2 * gl] = sgx;
    red[wave * 128 + 2 * gl + 1] = sgy;
  }
  __syncthreads();
  for (int i = tid; i < 2 * gn; i += nthr) {
    double s = red[i];
    for (int w = 1; w < W; ++w) s += red[w * 128 + i];
    ws_g[((size_t)n * a.G + g0) * 2 + i] = s;
  }
  // d log beta of the slice: a wave per beta sums the threads' entries
  for (int b = wave; b < B; b += W) {
    double s = 0.0;
    for (int i = lane; i < nthr; i += 64) s += dyn[(size_t)b * nthr + i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) ws_b[((size_t)n * gridDim.y + blockIdx.y) * B + b] = s;
  }
}

// Fixed-order second stage.  Long sums -- the goals over tracks, a shared log
// beta over (track, slice) -- take one block per output: thread t adds terms
// t, t + 256, ... in ascending order, then a fixed tree combines the 256
// partials.  Per-track log beta (a sum over the slices only) takes one thread
// per output.  Every order is fixed, so results are bitwise reproducible.
constexpr int kSumThreads = 256;

__global__ void __launch_bounds__(kSumThreads)
    loglik_sum_kernel(int N, int G, int B, int slices, const double* __restrict__ ws_g,
                      const double* __restrict__ ws_b, double* __restrict__ dgoals,
                      double* __restrict__ dlog_beta) {
  __shared__ double red[kSumThreads / 64];
  const int o = blockIdx.x;
  const bool goal = o < 2 * G;
  const double* src = goal ? ws_g + o : ws_b + (o - 2 * G);
  const size_t stride = goal ? (size_t)2 * G : (size_t)B;
  const int total = goal ? N : N * slices;
  double s = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < total; i += kSumThreads) s += src[(size_t)i * stride];
#pragma unroll
  for (int w = 32; w > 0; w >>= 1) s += __shfl_xor(s, w, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    s = red[0];
    for (int w = 1; w < kSumThreads / 64; ++w) s += red[w];
    if (goal) dgoals[o] = s;
    else dlog_beta[o - 2 * G] = s;
  }
}

__global__ void loglik_track_beta_kernel(int N, int B, int slices,
                                         const double* __restrict__ ws_b,
                                         double* __restrict__ dlog_beta) {
  const int jb = blockIdx.x * blockDim.x + threadIdx.x;
  if (jb >= N * B) return;
  const int n = jb / B, b = jb - n * B;
  double s = 0.0;
  for (int q = 0; q < slices; ++q) s += ws_b[((size_t)n * slices + q) * B + b];
  dlog_beta[jb] = s;
}

// Lanes per goal and goals per slice.  At most 21 goals a slice, so that each
// keeps at least three lanes (60 or more of the 64 busy); more slices than that
// only while the tracks leave CUs without a block (each slice recovers the
// track's controls again).
static LLShape ll_shape(int N, int G, int cus) {
  const int fill = std::min(G, (cus + std::max(N, 1) - 1) / std::max(N, 1));
  const int slices = std::max((G + 20) / 21, fill);
  const int per = (G + slices - 1) / slices;
  return LLShape{64 / per, per};
}

// Waves per block.  At most four (one per SIMD), as few as take the chunks in
// that many rounds: a further wave would only idle (100000 tracks x 5 steps, one
// goal, K = 32, forward: 432 us with four waves a block, 139 with one), and an
// uneven split leaves the first waves, which sit on the same SIMDs in every
// block, the longest (800 tracks x 100 steps x 5 goals, K = 32, adjoint: nine
// chunks to four waves 49 us, to three 40).  More only while the blocks do not
// fill the device, in whole fours (a block's waves go to the SIMDs in turn: five
// waves at 1024 tracks 102 us instead of 90 forward and 242 instead of 152 in the
// adjoint): eight while blocks of four leave wave slots empty (`per_cu` of them on
// a CU, two blocks or more), and further only where the blocks still fit the
// device together (300 tracks x 100 steps x 21 goals, K = 32: 65 us with 16
// waves, 59 with 8).
static int ll_waves(int64_t blocks, int Tmax, int L, int cus, int per_cu, int most) {
  const int chunks = std::max(1, (Tmax + L - 1) / L);
  const int rounds = (chunks + 3) / 4;
  int w = (chunks + rounds - 1) / rounds;
  if (chunks >= 16 && per_cu >= 16 && blocks * 4 < (int64_t)cus * per_cu) w = 8;
  for (int c = 8; c <= most; c += 4)
    if (w < c && c - 4 < chunks && blocks <= (int64_t)cus * (per_cu / c)) w = c;
  return w;
}

// Tracks of one launch: a block each, of at most 1024 threads, and a grid
// dimension holds less than 2^32 threads.  More tracks take several launches.
constexpr int kLaunchTracks = 1 << 21;

// The arguments of the tracks from n0 on.
static LLArgs from_track(LLArgs a, int n0) {
  a.tracks += (size_t)n0 * (a.Tmax + 1) * 2;
  a.lengths += n0;
  if (a.per_track) a.log_beta += (size_t)n0 * a.B;
  a.N -= n0;
  return a;
}

static cap_status make_ll_args(int32_t K, double speed, double dt, const float* tracks,
                               const int32_t* lengths, int32_t N, int32_t Tmax,
                               const float* goals, int32_t G, const float* log_beta, int32_t B,
                               int32_t per_track, LLArgs* a) {
  Controls c;
  cap_status st = make_controls(K, speed, dt, 0, nullptr, 0u, &c);
  if (st != CAP_OK) return st;
  if (N < 0 || Tmax < 0) return fail(CAP_E_INVALID, "N and Tmax must be >= 0");
  if (G < 1 || G > CAP_MAX_G || B < 1 || B > CAP_MAX_B)
    return fail(CAP_E_INVALID, "G in [1, 64] and B in [1, 16] required");
  // term counts and the second stage's thread indices stay in int
  if ((int64_t)N * G > ((int64_t)1 << 25)) return fail(CAP_E_INVALID, "N * G above 2^25");
  if (N > 0 && (!tracks || !lengths || !goals || !log_beta))
    return fail(CAP_E_INVALID, "tracks/lengths/goals/log_beta is NULL");
  a->m = make_belief_model(c, dt, 0, nullptr, 0, nullptr);
  a->tracks = tracks;
  a->lengths = lengths;
  a->N = N;
  a->Tmax = Tmax;
  a->G = G;
  a->B = B;
  a->per_track = per_track ? 1 : 0;
  a->goals = goals;
  a->log_beta = log_beta;
  return CAP_OK;
}

}  // namespace capred

using namespace capred;

extern "C" cap_status cap_loglik(int32_t K, double speed, double dt, const float* tracks_dev,
                                 const int32_t* lengths_dev, int32_t N, int32_t Tmax,
                                 const float* goals_dev, int32_t G, const float* log_beta_dev,
                                 int32_t B, int32_t per_track_beta, double* LL_dev, void* stream) {
  LLArgs a;
  cap_status st = make_ll_args(K, speed, dt, tracks_dev, lengths_dev, N, Tmax, goals_dev, G,
                               log_beta_dev, B, per_track_beta, &a);
  if (st != CAP_OK) return st;
  if (N == 0) return CAP_OK;
  if (!LL_dev) return fail(CAP_E_INVALID, "LL is NULL");
  const int cus = std::max(1, cap_device_cu_count());
  const LLShape lg = ll_shape(N, G, cus);
  const int slices = (G + lg.slice - 1) / lg.slice;
  int W = ll_waves((int64_t)N * slices, Tmax, lg.L, cus, 16, 16);
  while (W > 4 && W * B * (64 + lg.slice) > 12288) W -= 4;   // sums within 96 KiB of LDS
  const dim3 block(64 * W);
  const size_t lds = (size_t)W * (64 + lg.slice) * B * sizeof(double);
  hipStream_t s = as_stream(stream);
  for (int n0 = 0; n0 < N; n0 += kLaunchTracks) {
    const LLArgs q = from_track(a, n0);
    const dim3 grid((unsigned)std::min(q.N, kLaunchTracks), (unsigned)slices);
    double* out = LL_dev + (size_t)n0 * B * G;
    switch (q.m.U) {
      case 4: hipLaunchKernelGGL(loglik_kernel<4>, grid, block, lds, s, q, lg, out); break;
      case 8: hipLaunchKernelGGL(loglik_kernel<8>, grid, block, lds, s, q, lg, out); break;
      case 16: hipLaunchKernelGGL(loglik_kernel<16>, grid, block, lds, s, q, lg, out); break;
      case 32: hipLaunchKernelGGL(loglik_kernel<32>, grid, block, lds, s, q, lg, out); break;
      default: hipLaunchKernelGGL(loglik_kernel<0>, grid, block, lds, s, q, lg, out); break;
    }
    CAP_HIP(hipGetLastError());
  }
  return CAP_OK;
}

extern "C" size_t cap_loglik_backward_workspace(int32_t N, int32_t G, int32_t B,
                                                int32_t per_track_beta) {
  (void)per_track_beta;
  if (N < 0 || G < 0 || B < 0) return 0;
  return (size_t)N * G * (2 + B) * sizeof(double);
}

namespace capred {

// The adjoint's launches with the partial sums in ws (cap_loglik_backward_workspace bytes).
static cap_status loglik_backward_launch(const LLArgs& a, int32_t per_track_beta,
                                         const double* dLL_dev, double* dgoals_dev,
                                         double* dlog_beta_dev, void* ws_dev, hipStream_t s) {
  const int32_t N = a.N, G = a.G, B = a.B;
  double* ws_g = static_cast<double*>(ws_dev);
  double* ws_b = ws_g + (size_t)N * G * 2;
  const int cus = std::max(1, cap_device_cu_count());
  const LLShape lg = ll_shape(N, G, cus);
  const int slices = (G + lg.slice - 1) / lg.slice;
  if (N > 0) {
    const int kt = a.m.K == 4 || a.m.K == 8 || a.m.K == 16 || a.m.K == 32 ? a.m.K : 0;
    const int most = kt == 32 ? 12 : 16;   // waves per CU (and of a block)
    int W = ll_waves((int64_t)N * slices, a.Tmax, lg.L, cus, most, most);
    while (W > 4 && W * B > 192) W -= 4;   // sums within 96 KiB of LDS
    const dim3 block(64 * W);
    const size_t lds = (size_t)W * 128 * sizeof(double) +
                       (size_t)B * (64 * W * sizeof(double) + 64 * sizeof(float));
    for (int n0 = 0; n0 < N; n0 += kLaunchTracks) {
      const LLArgs q = from_track(a, n0);
      const dim3 grid((unsigned)std::min(q.N, kLaunchTracks), (unsigned)slices);
      const double* d = dLL_dev + (size_t)n0 * B * G;
      double* wg = ws_g + (size_t)n0 * G * 2;
      double* wb = ws_b + (size_t)n0 * slices * B;
      switch (kt) {
        case 4: hipLaunchKernelGGL(loglik_backward_kernel<4>, grid, block, lds, s, q, lg, d, wg, wb); break;
        case 8: hipLaunchKernelGGL(loglik_backward_kernel<8>, grid, block, lds, s, q, lg, d, wg, wb); break;
        case 16: hipLaunchKernelGGL(loglik_backward_kernel<16>, grid, block, lds, s, q, lg, d, wg, wb); break;
        case 32: hipLaunchKernelGGL(loglik_backward_kernel<32>, grid, block, lds, s, q, lg, d, wg, wb); break;
        default: hipLaunchKernelGGL(loglik_backward_kernel<0>, grid, block, lds, s, q, lg, d, wg, wb); break;
      }
      CAP_HIP(hipGetLastError());
    }
  }
  // with N = 0 the sums are empty: the kernels write zeros
  const int long_sums = 2 * G + (per_track_beta ? 0 : B);
  hipLaunchKernelGGL(loglik_sum_kernel, dim3(long_sums), dim3(kSumThreads), 0, s, N, G, B, slices,
                     ws_g, ws_b, dgoals_dev, dlog_beta_dev);
  if (per_track_beta && N > 0)
    hipLaunchKernelGGL(loglik_track_beta_kernel, dim3((N * B + 255) / 256), dim3(256), 0, s, N, B,
                       slices, ws_b, dlog_beta_dev);
  CAP_HIP(hipGetLastError());
  return CAP_OK;
}

// Device-resident partial sums of the allocation-free adjoint.  Each device
// holds its own copy (until the process ends); host code reaches it only
// through the per-device address from hipGetSymbolAddress, never through the
// array's name, which on the host is a stand-in and not a device address.
__device__ __align__(256) double loglik_scratch[CAP_LOGLIK_SCRATCH_BYTES / sizeof(double)];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};

// loglik_scratch's address on the current device (looked up once per device).
static cap_status scratch_of_current_device(void** out) {
  int dev = 0;
  CAP_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(CAP_E_UNSUPPORTED, "device index above 63");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    CAP_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(loglik_scratch)));
    if (!p) return fail(CAP_E_HIP, "hipGetSymbolAddress returned no address for the scratch");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return CAP_OK;
}

}  // namespace capred

extern "C" cap_status cap_loglik_backward(int32_t K, double speed, double dt,
                                          const float* tracks_dev, const int32_t* lengths_dev,
                                          int32_t N, int32_t Tmax, const float* goals_dev,
                                          int32_t G, const float* log_beta_dev, int32_t B,
                                          int32_t per_track_beta, const double* dLL_dev,
                                          double* dgoals_dev, double* dlog_beta_dev, void* ws_dev,
                                          size_t ws_bytes, void* stream) {
  LLArgs a;
  cap_status st = make_ll_args(K, speed, dt, tracks_dev, lengths_dev, N, Tmax, goals_dev, G,
                               log_beta_dev, B, per_track_beta, &a);
  if (st != CAP_OK) return st;
  if (!dgoals_dev || !dlog_beta_dev) return fail(CAP_E_INVALID, "dgoals/dlog_beta is NULL");
  if (N > 0 && !dLL_dev) return fail(CAP_E_INVALID, "dLL is NULL");
  const size_t need = cap_loglik_backward_workspace(N, G, B, per_track_beta);
  if (need > 0 && (!ws_dev || ws_bytes < need))
    return fail(CAP_E_WORKSPACE, "workspace smaller than cap_loglik_backward_workspace()");
  return loglik_backward_launch(a, per_track_beta, dLL_dev, dgoals_dev, dlog_beta_dev, ws_dev,
                                as_stream(stream));
}

extern "C" cap_status cap_loglik_backward_noalloc(int32_t K, double speed, double dt,
                                                  const float* tracks_dev,
                                                  const int32_t* lengths_dev, int32_t N,
                                                  int32_t Tmax, const float* goals_dev, int32_t G,
                                                  const float* log_beta_dev, int32_t B,
                                                  int32_t per_track_beta, const double* dLL_dev,
                                                  double* dgoals_dev, double* dlog_beta_dev,
                                                  void* stream) {
  LLArgs a;
  cap_status st = make_ll_args(K, speed, dt, tracks_dev, lengths_dev, N, Tmax, goals_dev, G,
                               log_beta_dev, B, per_track_beta, &a);
  if (st != CAP_OK) return st;
  if (!dgoals_dev || !dlog_beta_dev) return fail(CAP_E_INVALID, "dgoals/dlog_beta is NULL");
  if (N > 0 && !dLL_dev) return fail(CAP_E_INVALID, "dLL is NULL");
  if (cap_loglik_backward_workspace(N, G, B, per_track_beta) > CAP_LOGLIK_SCRATCH_BYTES)
    return fail(CAP_E_CAPACITY,
                "N * G * (2 + B) * 8 bytes exceed CAP_LOGLIK_SCRATCH_BYTES; use cap_loglik_backward "
                "with a caller workspace");
  void* scratch = nullptr;
  st = scratch_of_current_device(&scratch);
  if (st != CAP_OK) return st;
  // every partial-sum slot the launches read is written first (one per track
  // and goal or slice), so the previous call's contents need no clearing
  return loglik_backward_launch(a, per_track_beta, dLL_dev, dgoals_dev, dlog_beta_dev, scratch,
                                as_stream(stream));
}
