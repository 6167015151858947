// mppi.hip -- MPPI consumer of the predicted occupancy grids (Sec. III-C,
// local planner): N sampled control sequences for the 4-D Dubins robot of
// Eq. (robot_model), their trajectory costs against the device-resident
// prediction grids, and the exponentially weighted update of the reference
// controls.
//
// Layout on gfx950: one sample per lane, 64 samples per block, and the steps of
// a chunk dealt to the block's waves.  A sample's trajectory is serial only in
// its four running sums (v, theta, then x, y: one add a step each); the work of
// a step -- FP64 sine and cosine, the grid read, the cost -- needs no other
// step's.  So the waves stage the controls, two waves run the sums of v and
// theta through LDS, all waves take their steps' sine and cosine, two waves run
// x and y, and all waves add their steps' costs, always by the step's place among
// 16, which one wave sums in order: a sample's cost depends neither on the batch nor
// on the waves (perturbations laid out [T][N][2]: a wave reads 64 consecutive
// (a, omega) pairs per step).  The robot state and the cost run in FP64: the collision term is a
// step function of the grid cell, and FP64 positions (every product and sum
// rounded on its own) keep the cell decisions of this kernel and of an FP64
// reference identical
// except within ~1e-12 m of a cell edge.  The update runs one block per step
// t; every block recomputes min S and the weight sum with the same fixed-order
// reduction, so the result does not depend on the launch.
#include <algorithm>

#include "common.hpp"

namespace capred {

constexpr int kChunkSteps = 48;        // steps of a chunk (3 per wave at 16 waves)
constexpr int kRuns = 16;              // partial costs of a chunk: steps r, r + 16, r + 32
constexpr int kUpdateThreads = 1024;

struct MppiArgs {
  double z0[4], goal[4];
  double Q[4], Qf[4], R[2];
  double w_coll, p_coll, c_time, tau, dt;
  double x0, y0, cell;
  int32_t T, N, H, nx, ny;
  const double* U;      // [T][2]
  const double* delta;  // [T][N][2]
  const float* occ;     // [H][ny][nx] or null
  double* S;            // [N]
};

// One lane per sample, serial over T: 33 us at 8192 samples x 40 steps (128
// waves on 1024 SIMDs, each step's sine and cosine on the critical path).
// W waves share a chunk's steps instead: 10.2 us.
template <int W>
__global__ void __launch_bounds__(64 * W) mppi_rollout_kernel(const MppiArgs a) {
#pragma clang fp contract(off)
  constexpr int kOwn = kChunkSteps / W;   // steps of a wave per chunk
  static_assert(kChunkSteps % kRuns == 0 && kRuns % W == 0 && W >= 3, "whole runs per wave");
  constexpr int kOwnRuns = kRuns / W;     // runs wave, wave + W, ... of a chunk
  // row t + 1 belongs to step t of the chunk, row 0 to the state before it
  __shared__ double A[kChunkSteps + 1][64], B[kChunkSteps + 1][64];
  __shared__ double part[kRuns][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane;
  const int is = min(i, a.N - 1);   // lanes past the end repeat the last sample
  const double2* dl = reinterpret_cast<const double2*>(a.delta);
  const size_t plane = (size_t)a.nx * a.ny;
  // The last wave carries the cost: it adds a chunk's runs while the first two run
  // the next chunk's sums (part is written again some barriers later).
  double sum = 0.0;
  const auto add_runs = [&] {
#pragma unroll 8
    for (int r = 0; r < kRuns; ++r) sum += part[r][lane];
  };
  double c0 = wave == 0 ? a.z0[2] : a.z0[3];   // wave 0 carries v and x, wave 1 theta and y
  double c1 = wave == 0 ? a.z0[0] : a.z0[1];
  for (int t0 = 0; t0 < a.T; t0 += kChunkSteps) {
    const int tn = min(kChunkSteps, a.T - t0);
    double ua[kOwn], uw[kOwn], v[kOwn], th[kOwn], x[kOwn], y[kOwn];
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
      const int t = wave + k * W;
      if (t < tn) {
        const double2 d = dl[(size_t)(t0 + t) * a.N + is];
        ua[k] = a.U[2 * (t0 + t)] + d.x;
        uw[k] = a.U[2 * (t0 + t) + 1] + d.y;
        A[t + 1][lane] = ua[k] * a.dt;
        B[t + 1][lane] = uw[k] * a.dt;
      }
    }
    __syncthreads();
    if (wave == W - 1 && t0 > 0) add_runs();
    if (wave < 2) {
      double (*R)[64] = wave == 0 ? A : B;
      R[0][lane] = c0;
#pragma unroll 8
      for (int t = 1; t <= tn; ++t) {
        c0 = c0 + R[t][lane];
        R[t][lane] = c0;
      }
    }
    __syncthreads();
    double px[kOwn], py[kOwn];
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
      const int t = wave + k * W;
      if (t < tn) {
        const double vo = A[t][lane], to = B[t][lane];
        v[k] = A[t + 1][lane];
        th[k] = B[t + 1][lane];
        double sn, cs;
        sincos(to, &sn, &cs);
        px[k] = vo * cs * a.dt;
        py[k] = vo * sn * a.dt;
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
      const int t = wave + k * W;
      if (t < tn) {
        A[t + 1][lane] = px[k];
        B[t + 1][lane] = py[k];
      }
    }
    __syncthreads();
    if (wave < 2) {
      double (*R)[64] = wave == 0 ? A : B;
#pragma unroll 8
      for (int t = 1; t <= tn; ++t) {
        c1 = c1 + R[t][lane];
        R[t][lane] = c1;
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
      const int t = wave + k * W;
      if (t < tn) {
        x[k] = A[t + 1][lane];
        y[k] = B[t + 1][lane];
      }
    }
    // (no barrier: the next chunk's rows are written by the waves that read these)
    double s[kOwnRuns] = {};
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
      const int t = t0 + wave + k * W + 1;   // 1 .. T
      if (wave + k * W < tn) {
        const double e0 = x[k] - a.goal[0], e1 = y[k] - a.goal[1], e2 = v[k] - a.goal[2],
                     e3 = th[k] - a.goal[3];
        if (t < a.T) {
          s[k % kOwnRuns] += a.Q[0] * e0 * e0;
          s[k % kOwnRuns] += a.Q[1] * e1 * e1;
          s[k % kOwnRuns] += a.Q[2] * e2 * e2;
          s[k % kOwnRuns] += a.Q[3] * e3 * e3;
          s[k % kOwnRuns] += a.R[0] * ua[k] * ua[k] + a.R[1] * uw[k] * uw[k];
          if (a.occ && t <= a.H) {
            const double cx = floor((x[k] - a.x0) / a.cell), cy = floor((y[k] - a.y0) / a.cell);
            if (cx >= 0.0 && cx < (double)a.nx && cy >= 0.0 && cy < (double)a.ny) {
              const float p = a.occ[(size_t)(t - 1) * plane + (size_t)cy * a.nx + (size_t)cx];
              if ((double)p >= a.p_coll) s[k % kOwnRuns] += a.w_coll;
            }
          }
          s[k % kOwnRuns] += a.c_time;
        } else {
          s[k % kOwnRuns] += a.Qf[0] * e0 * e0;
          s[k % kOwnRuns] += a.Qf[1] * e1 * e1;
          s[k % kOwnRuns] += a.Qf[2] * e2 * e2;
          s[k % kOwnRuns] += a.Qf[3] * e3 * e3;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kOwnRuns; ++j) part[wave + j * W][lane] = s[j];
  }
  __syncthreads();
  if (wave == W - 1) {
    add_runs();
    if (i < a.N) a.S[i] = sum;
  }
}

// Block-wide reduction of M values in a fixed order (a butterfly in each wave,
// then the waves in order); every thread gets the results.
template <bool MIN, int M>
__device__ __forceinline__ void block_fold(double* v, double (*red)[kUpdateThreads / 64]) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int k = 0; k < M; ++k) {
      const double x = __shfl_xor(v[k], o, 64);
      v[k] = MIN ? fmin(v[k], x) : v[k] + x;
    }
  __syncthreads();
  if ((threadIdx.x & 63) == 0)
    for (int k = 0; k < M; ++k) red[k][threadIdx.x >> 6] = v[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < M; ++k) {
    v[k] = red[k][0];
#pragma unroll
    for (int w = 1; w < kUpdateThreads / 64; ++w)
      v[k] = MIN ? fmin(v[k], red[k][w]) : v[k] + red[k][w];
  }
}

// Block t: U[t] += sum_i w_i delta[t][i] / sum_i w_i, w_i = exp(-(S_i - min S) / tau).
// Latency-bound (T blocks, each over all N): 1024 threads a block instead of
// 256 took it from 18 us to 7.5 us at 8192 samples x 40 steps.
__global__ void __launch_bounds__(kUpdateThreads)
    mppi_update_kernel(const double* __restrict__ S, const double* __restrict__ delta, int N,
                       double tau, double* __restrict__ U) {
  __shared__ double red[3][kUpdateThreads / 64];
  const int t = blockIdx.x;
  double m = INFINITY;
#pragma unroll 8
  for (int i = threadIdx.x; i < N; i += kUpdateThreads) m = fmin(m, S[i]);
  block_fold<true, 1>(&m, red);
  double acc[3] = {0.0, 0.0, 0.0};   // sum w, sum w delta
  const double2* dl = reinterpret_cast<const double2*>(delta) + (size_t)t * N;
  // (m - S) / tau as a product with the rounded reciprocal and one correction,
  // which rounds as the division does (Markstein); out of the range of tau where
  // nothing over- or underflows, the division itself.  The bound (its weight is 0
  // already) keeps an infinite cost from a product of infinities; NaN stays NaN.
  const double rate = 1.0 / tau;
  const auto add = [&](auto quotient) {
#pragma unroll 8
    for (int i = threadIdx.x; i < N; i += kUpdateThreads) {
      const double w = exp(quotient(m - S[i]));
      const double2 d = dl[i];
      acc[0] += w;
      acc[1] += w * d.x;
      acc[2] += w * d.y;
    }
  };
  if (tau > 0x1p-500 && tau < 0x1p500)
    add([&](double x) {
      const double q = fmax(x * rate, -4096.0);
      return fma(fma(-q, tau, x), rate, q);
    });
  else
    add([&](double x) { return x / tau; });
  block_fold<false, 3>(acc, red);
  if (threadIdx.x == 0) {
    U[2 * t] += acc[1] / acc[0];
    U[2 * t + 1] += acc[2] / acc[0];
  }
}

}  // namespace capred

using namespace capred;

extern "C" cap_status cap_mppi_step(const double z0[4], const double goal[4], int32_t T,
                                    double dt, int32_t N, double* U_dev,
                                    const double* delta_dev, const float* occ_dev, int32_t H,
                                    const cap_grid* grid, const cap_mppi_cost* cost,
                                    double* S_dev, void* stream) {
  if (!z0 || !goal || !cost) return fail(CAP_E_INVALID, "z0, goal or cost is NULL");
  if (T < 1 || T > 65535 || N < 1 || N > (1 << 24))
    return fail(CAP_E_INVALID, "T must be in [1, 65535] and N in [1, 2^24]");
  if (!(dt > 0.0) || !std::isfinite(dt)) return fail(CAP_E_INVALID, "dt must be > 0");
  if (!(cost->tau > 0.0) || !std::isfinite(cost->tau)) return fail(CAP_E_INVALID, "tau must be > 0");
  if (!U_dev || !delta_dev || !S_dev) return fail(CAP_E_INVALID, "U, delta or S is NULL");
  if (occ_dev) {
    if (!grid || !(grid->cell > 0.0) || grid->nx < 1 || grid->ny < 1 || H < 0 ||
        !std::isfinite(grid->x0) || !std::isfinite(grid->y0))
      return fail(CAP_E_INVALID, "occupancy needs a valid grid and H >= 0");
  }
  if ((reinterpret_cast<uintptr_t>(delta_dev) & 15u) != 0)
    return fail(CAP_E_INVALID, "delta must be 16-byte aligned");
  MppiArgs a{};
  for (int k = 0; k < 4; ++k) {
    a.z0[k] = z0[k];
    a.goal[k] = goal[k];
    a.Q[k] = cost->Q[k];
    a.Qf[k] = cost->Qf[k];
  }
  a.R[0] = cost->R[0];
  a.R[1] = cost->R[1];
  a.w_coll = cost->w_coll;
  a.p_coll = cost->p_coll;
  a.c_time = cost->c_time;
  a.tau = cost->tau;
  a.dt = dt;
  a.T = T;
  a.N = N;
  a.U = U_dev;
  a.delta = delta_dev;
  a.S = S_dev;
  if (occ_dev) {
    a.occ = occ_dev;
    a.H = H;
    a.x0 = grid->x0;
    a.y0 = grid->y0;
    a.cell = grid->cell;
    a.nx = grid->nx;
    a.ny = grid->ny;
  } else {
    a.cell = 1.0;
    a.nx = a.ny = 1;
  }
  hipStream_t s = as_stream(stream);
  // Waves per block by the waves the samples alone bring: 16 (shortest path
  // through a step chunk) while they fit the chip's 4096 wave slots at four per
  // SIMD, fewer beyond, where the serial sums of two waves would idle the rest.
  const unsigned blocks = (unsigned)((N + 63) / 64);
  if (blocks <= 256)
    hipLaunchKernelGGL(mppi_rollout_kernel<16>, dim3(blocks), dim3(64 * 16), 0, s, a);
  else if (blocks <= 1024)
    hipLaunchKernelGGL(mppi_rollout_kernel<8>, dim3(blocks), dim3(64 * 8), 0, s, a);
  else
    hipLaunchKernelGGL(mppi_rollout_kernel<4>, dim3(blocks), dim3(64 * 4), 0, s, a);
  hipLaunchKernelGGL(mppi_update_kernel, dim3((unsigned)T), dim3(kUpdateThreads), 0, s,
                     (const double*)S_dev, delta_dev, (int)N, cost->tau, U_dev);
  CAP_HIP(hipGetLastError());
  return CAP_OK;
}
