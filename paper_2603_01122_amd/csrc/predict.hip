// predict.hip -- single-human Alg. 1 (cap_predict_occupancy), grid clearing,
// normalisation (cap_normalize) and the track simulator (cap_simulate_tracks).
#include <algorithm>

#include "model.hpp"

namespace capred {

// Clears the n counts and the m off-grid counters (nullable).
__global__ void __launch_bounds__(256)
    zero_u32_kernel(uint32_t* __restrict__ p, size_t n, uint32_t* __restrict__ q, size_t m) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q)
    for (size_t v = i; v < m; v += stride) q[v] = 0u;
  const size_t head = (reinterpret_cast<uintptr_t>(p) & 15u) ? 0 : n / 4;
  uint4* p4 = reinterpret_cast<uint4*>(p);
  for (size_t v = i; v < head; v += stride) p4[v] = make_uint4(0u, 0u, 0u, 0u);
  for (size_t v = head * 4 + i; v < n; v += stride) p[v] = 0u;
}

__global__ void __launch_bounds__(256) normalize_kernel(const uint32_t* __restrict__ c,
                                                        float* __restrict__ p, size_t n,
                                                        float inv_n_unused, float N) {
  (void)inv_n_unused;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool aligned = ((reinterpret_cast<uintptr_t>(c) | reinterpret_cast<uintptr_t>(p)) & 15u) == 0;
  const size_t head = aligned ? n / 4 : 0;
  const uint4* c4 = reinterpret_cast<const uint4*>(c);
  float4* p4 = reinterpret_cast<float4*>(p);
  for (size_t v = i; v < head; v += stride) {
    const uint4 x = c4[v];
    p4[v] = make_float4((float)x.x / N, (float)x.y / N, (float)x.z / N, (float)x.w / N);
  }
  for (size_t v = head * 4 + i; v < n; v += stride) p[v] = (float)c[v] / N;
}

// Threads of a block at most.  The shifted draw of several speeds keeps its
// exponents over two passes (239 and 256 registers at K = 16 and 32): with the 128
// of 1024-thread blocks it spills (400000 particles x 20 steps of 6 x 16 controls
// 3.27 ms, with 256 threads 1.22).
template <int KT, bool SHIFT, bool MS>
constexpr int plain_threads() { return SHIFT && MS && KT >= 16 ? 256 : 1024; }

template <int KT, int P, bool SHIFT, bool MS, int L>
__global__ void __launch_bounds__((plain_threads<KT, SHIFT, MS>()))
    rollout_plain_kernel(const RolloutDesc d, uint32_t seed_lo, uint32_t seed_hi, int cap) {
  __shared__ TileShared sh;
  __shared__ float4 ctl[MS ? CAP_MAX_U : 1];
  extern __shared__ __align__(16) uint32_t win[];
  // cap is a multiple of four: whole 16-byte stores (a block of one wave clears
  // the 38 KB of 20 steps in 37 of them)
  for (int i = threadIdx.x; i < cap / 2; i += blockDim.x)
    reinterpret_cast<uint4*>(win)[i] = make_uint4(0u, 0u, 0u, 0u);
  // the first barrier inside rollout_tile orders this clear before any binning
  const int64_t first = (int64_t)blockIdx.x * P * (blockDim.x / L);
  rollout_tile<KT, P, SHIFT, MS, L>(d, first, seed_lo, seed_hi, sh, win, cap, ctl);
}

// Track simulator: one thread per track, the same control draw as the rollout
// with the track's own (beta, goal) and the simulation counter domain.
template <int KT, bool MS>
__global__ void __launch_bounds__(256)
    simulate_kernel(const RolloutDesc d, int32_t n, int32_t T, const double* __restrict__ start,
                    const float* __restrict__ beta, const float* __restrict__ goal, double x0,
                    double y0, double cell, uint32_t stream_id, uint32_t seed_lo,
                    uint32_t seed_hi, int32_t* __restrict__ lat, float* __restrict__ pos) {
#pragma clang fp contract(off)
  __shared__ float4 ctl[MS ? CAP_MAX_U : 1];
  if constexpr (MS) {
    for (int u = threadIdx.x; u < d.K * d.S; u += blockDim.x)
      ctl[u] = make_float4(d.T.fx[u], d.T.fy[u], d.T.s2[u], 0.f);
    __syncthreads();
  }
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  const double q = cell / kLatticeScale;
  int32_t X = (int32_t)rint((start[2 * r] - x0) / q);
  int32_t Y = (int32_t)rint((start[2 * r + 1] - y0) / q);
  const int32_t GX = (int32_t)rint(((double)goal[2 * r] - x0) / q);
  const int32_t GY = (int32_t)rint(((double)goal[2 * r + 1] - y0) / q);
  const float ib = (float)(1.0 / (-(double)beta[r] * q * (double)kLog2e));
  const bool shift = (double)beta[r] * (double)max(d.Rx, d.Ry) * q > kNoShiftLimit;
  uint4 w = make_uint4(0u, 0u, 0u, 0u);
  for (int t = 0; t <= T; ++t) {
    if (t > 0) {
      const int s = (t - 1) & 3;
      if (s == 0) w = philox10((uint32_t)r, (uint32_t)((t - 1) >> 2), stream_id, 0xFFFFFFFFu,
                               seed_lo, seed_hi);
      const float u = uniform24f(pick_word(w, s));
      int k;
      if constexpr (MS)
        k = shift ? draw_control<KT, true>((float)(X - GX), (float)(Y - GY), ib, u, d.T, d.S,
                                           d.smask, d.s_last, ctl)
                  : draw_control<KT, false>((float)(X - GX), (float)(Y - GY), ib, u, d.T, d.S,
                                            d.smask, d.s_last, ctl);
      else
        k = shift ? draw_heading<KT, true>((float)(X - GX), (float)(Y - GY), ib, u, d.T, d.K)
                  : draw_heading<KT, false>((float)(X - GX), (float)(Y - GY), ib, u, d.T, d.K);
      X += (int32_t)d.T.fx[k];
      Y += (int32_t)d.T.fy[k];
    }
    const size_t o = ((size_t)r * (T + 1) + t) * 2;
    if (lat) {
      lat[o] = X;
      lat[o + 1] = Y;
    }
    if (pos) {
      pos[o] = (float)(x0 + (double)X * q);
      pos[o + 1] = (float)(y0 + (double)Y * q);
    }
  }
}

__global__ void __launch_bounds__(256)
    philox_blocks_kernel(int64_t n, uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                         uint32_t slo, uint32_t shi, uint4* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = philox10(c0 + (uint32_t)i, c1, c2, c3, slo, shi);
}

static cap_status launch_zero(uint32_t* p, size_t n, uint32_t* q, size_t m, hipStream_t s) {
  const size_t blocks = std::min<size_t>((n / 4 + 255) / 256 + 1, 4096);
  hipLaunchKernelGGL(zero_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n, q, m);
  CAP_HIP(hipGetLastError());
  return CAP_OK;
}

// Words of one window buffer at most: the share of a CU's LDS that leaves the
// other blocks of that size their place (a 1024-thread block is alone on its CU at
// 128 registers).  A window of up to twice the buffer still fits (see
// rollout_tile_body).
static constexpr int most_window_words(int threads) {
  return (threads <= 256 ? 40 : threads <= 512 ? 64 : 128) * 1024 / (2 * (int)sizeof(uint32_t));
}

// Words of the last step's window, the widest.
static int64_t reach_words(const RolloutDesc& d) {
  const int64_t rx = (int64_t)d.H * d.Rx, ry = (int64_t)d.H * d.Ry;
  const int64_t x0 = std::max<int64_t>((d.X0 - rx) >> kLatticeShift, 0),
                x1 = std::min<int64_t>((d.X0 + rx) >> kLatticeShift, d.nx - 1),
                y0 = std::max<int64_t>((d.Y0 - ry) >> kLatticeShift, 0),
                y1 = std::min<int64_t>((d.Y0 + ry) >> kLatticeShift, d.ny - 1);
  return x1 < x0 || y1 < y0 ? 0 : (x1 - x0 + 2) / 2 * (y1 - y0 + 1);
}

// Words of one window buffer for blocks of `threads`: what the widest step window
// needs, at most the above.
static int plain_window_words(const RolloutDesc& d, int threads) {
  const int need = (int)std::min<int64_t>(reach_words(d), most_window_words(threads));
  return std::max(64, (need + 3) & ~3);
}

template <int KT, int P, bool MS, int L = 1>
static cap_status launch_plain_t(const RolloutDesc& d, uint32_t slo, uint32_t shi, int threads,
                                 hipStream_t s) {
  if (L == 1 && d.shift) threads = std::min(threads, plain_threads<KT, true, MS>());
  const int64_t per_block = (int64_t)P * (threads / L);
  const int64_t blocks = (d.N + per_block - 1) / per_block;
  const int cap = plain_window_words(d, threads);
  const size_t lds = window_lds_bytes(cap, P * threads);
  if constexpr (L == 1) {
    if (d.shift) {
      hipLaunchKernelGGL((rollout_plain_kernel<KT, P, true, MS, 1>), dim3((unsigned)blocks),
                         dim3(threads), lds, s, d, slo, shi, cap);
      CAP_HIP(hipGetLastError());
      return CAP_OK;
    }
  }
  hipLaunchKernelGGL((rollout_plain_kernel<KT, P, false, MS, L>), dim3((unsigned)blocks),
                     dim3(threads), lds, s, d, slo, shi, cap);
  CAP_HIP(hipGetLastError());
  return CAP_OK;
}

// Shape of the launch.  Few particles are bound by the latency of a step, which
// a block of one wave keeps shortest while one per CU holds them all.  More are
// bound by the device-scope atomics of the flush: a tile adds each cell it touched
// once per step, so larger tiles add less: from two waves per CU on blocks of four
// (30000 particles x 23 steps, K = 8: 128 threads 53.3 us, 256 threads 49.8), then as
// many as one block per CU asks.  2^18 particles x 50 steps (K = 16): 1024
// blocks of 256 threads issue 4.75e6 atomics and the call takes 337-378 us, with
// 256 blocks of 1024 threads 214; 8192 particles x 10 steps (96 controls): 32
// blocks of 256 threads 73.9 us, 128 of 64 threads 69.0.
//
// Where larger tiles do not pay, blocks stay smaller, as several of them on a CU
// fill each other's waits:
//   * a reach beyond the largest windows (both buffers), at 16 headings or more:
//     the particles spread until they share few cells (2^18 particles x 60 steps of
//     2.4 cells on 500 x 500 cells, K = 16: 1024 threads 777 us, 256 threads 720;
//     K = 4 622 and 772), up to 64 waves a CU (2 10^6 particles: 4.82 and 4.90 ms);
//   * several speeds, for their longer draws: more than 64 controls 256 threads
//     (70000 particles x 10 steps of 6 x 16 controls: 512 threads 84 us, 256 threads
//     76; 2^20 x 20 steps 1024 threads 1.03 ms, 512 and 256 0.97), 64 controls of 16
//     headings or more and the shifted draw 512 (2^20 x 20 steps of 4 x 16: 1024 threads
//     0.82 ms, 512 0.78, 256 1.07; of 2 x 8, sharp: 416, 382 and 413 us), else 1024 (of 2 x
//     16: 0.63, 0.82 and 1.00 ms; 50 steps of 8 x 8: 1.92, 2.27 and 2.65).
template <int KT, bool MS>
static cap_status launch_plain_k(const RolloutDesc& d, int64_t cus, uint32_t slo, uint32_t shi,
                                 hipStream_t s) {
  const int64_t waves = (d.N + 64 * cus - 1) / (64 * cus);   // per CU
  const int64_t blk = waves == 1 ? 1 : std::max<int64_t>(waves, 4);
  int most = 1024;
  if constexpr (MS) {
    // few particles: several lanes each, eight while those fit two waves per SIMD, then
    // four up to two (8 headings) or two and a half; 8192 particles x 10 steps of 96
    // controls: 52 us by one lane, 34 by eight; one lane | four, 12 steps: 6 x 16 controls,
    // 40000 particles 66 | 61 us, 65536 75 | 77; 3 x 32 controls, 32768 72 | 57, 40000 72 |
    // 72, 65536 79 | 91; 50 steps of 2 x 8 controls, 45000 131 | 144
    const auto threads = [&](int L) {
      return 64 * (int)std::min<int64_t>((L * d.N + 64 * cus - 1) / (64 * cus), 16);
    };
    if constexpr (KT >= 16)
      if (!d.shift && d.N <= 64 * cus) return launch_plain_t<KT, 1, MS, 8>(d, slo, shi, threads(8), s);
    if constexpr (KT >= 8)
      if (!d.shift && d.N <= (KT == 8 ? 128 : 160) * cus)
        return launch_plain_t<KT, 1, MS, 4>(d, slo, shi, threads(4), s);
    if (d.K * d.S > 64) most = 256;
    else if (d.shift || (KT >= 16 && d.K * d.S == 64)) most = 512;
  } else {
    const bool wide = (KT == 0 || KT >= 16) && reach_words(d) > 2 * most_window_words(1024);
    if (wide && waves <= 64) most = 256;
    else if (waves > 32) return launch_plain_t<KT, 4, MS>(d, slo, shi, 1024, s);
    else if (waves > 16) return launch_plain_t<KT, 2, MS>(d, slo, shi, 1024, s);
  }
  return launch_plain_t<KT, 1, MS>(d, slo, shi, (int)std::min<int64_t>(64 * blk, most), s);
}

static cap_status launch_plain(RolloutDesc& d, uint32_t slo, uint32_t shi, hipStream_t s) {
  const int cus = std::max(1, cap_device_cu_count());
  d.bounds = bounds_rule(d.N, cus);
  // blocks of 256 threads (below) have windows that the bounds mostly outgrow too
  // (600000 particles x 50 steps of 6 x 16 controls: always 1557 us, where shared 1524)
  if (d.K * d.S > 64) d.bounds = std::min<int32_t>(d.bounds, kBoundsShared);
  // specialised kernels assume a point-symmetric step table; several speeds
  // need one (checked when the descriptor is built)
  if (d.S > 1) {
    switch (d.K) {
      case 4: return launch_plain_k<4, true>(d, cus, slo, shi, s);
      case 8: return launch_plain_k<8, true>(d, cus, slo, shi, s);
      case 16: return launch_plain_k<16, true>(d, cus, slo, shi, s);
      default: return launch_plain_k<32, true>(d, cus, slo, shi, s);
    }
  }
  switch (d.sym ? d.K : 0) {
    case 4: return launch_plain_k<4, false>(d, cus, slo, shi, s);
    case 8: return launch_plain_k<8, false>(d, cus, slo, shi, s);
    case 16: return launch_plain_k<16, false>(d, cus, slo, shi, s);
    case 32: return launch_plain_k<32, false>(d, cus, slo, shi, s);
    default: return launch_plain_k<0, false>(d, cus, slo, shi, s);
  }
}

}  // namespace capred

using namespace capred;

extern "C" cap_status cap_predict_occupancy(const cap_model* model, const cap_grid* grid,
                                            const double z0[2], const double* belief_dev,
                                            int32_t N, int32_t H, uint64_t seed,
                                            uint32_t human_id, uint32_t cycle,
                                            uint32_t* counts_dev, uint32_t* offgrid_dev,
                                            uint8_t* trace_k_dev, int32_t* trace_pair_dev,
                                            void* stream) {
  Controls c;
  cap_status st = check_model(model, &c);
  if (st != CAP_OK) return st;
  if ((st = check_grid(grid)) != CAP_OK) return st;
  if (!z0 || !belief_dev || !counts_dev) return fail(CAP_E_INVALID, "z0, belief or counts is NULL");
  if (cycle >= 0x7FFFFFFFu) return fail(CAP_E_INVALID, "cycle must be < 2^31 - 1");
  RolloutDesc d;
  st = make_rollout_desc(c, model->dt, model->B, model->beta, model->G, model->goals, *grid, N,
                         H, &d);
  if (st != CAP_OK) return st;
  if ((st = set_start(&d, z0[0], z0[1], *grid)) != CAP_OK) return st;
  d.human = human_id;
  d.cycle = cycle;
  d.belief = belief_dev;
  d.counts = counts_dev;
  d.offgrid = offgrid_dev;
  d.trace_k = trace_k_dev;
  d.trace_pair = trace_pair_dev;
  hipStream_t s = as_stream(stream);
  if ((st = launch_zero(counts_dev, (size_t)H * grid->nx * grid->ny, offgrid_dev, (size_t)H, s)) !=
      CAP_OK)
    return st;
  return launch_plain(d, (uint32_t)seed, (uint32_t)(seed >> 32), s);
}

extern "C" cap_status cap_normalize(const uint32_t* counts_dev, int64_t n_cells, int32_t N,
                                    float* probs_dev, void* stream) {
  if (n_cells < 0 || N < 1) return fail(CAP_E_INVALID, "n_cells must be >= 0 and N >= 1");
  if (n_cells == 0) return CAP_OK;
  if (!counts_dev || !probs_dev) return fail(CAP_E_INVALID, "counts or probs is NULL");
  const size_t n = (size_t)n_cells;
  const size_t blocks = std::min<size_t>((n / 4 + 255) / 256 + 1, 8192);
  hipLaunchKernelGGL(normalize_kernel, dim3((unsigned)blocks), dim3(256), 0, as_stream(stream),
                     counts_dev, probs_dev, n, 0.f, (float)N);
  CAP_HIP(hipGetLastError());
  return CAP_OK;
}

extern "C" cap_status cap_simulate_tracks(int32_t K, double speed, int32_t n_speeds,
                                          const double* speeds, double dt, double x0,
                                          double y0, double cell, int32_t n, int32_t T,
                                          const double* start_dev, const float* beta_dev,
                                          const float* goal_dev, uint64_t seed,
                                          uint32_t stream_id, int32_t* lat_dev, float* pos_dev,
                                          void* stream) {
  Controls c;
  cap_status st = make_controls(K, speed, dt, n_speeds, speeds, 0u, &c);
  if (st != CAP_OK) return st;
  if (n < 0 || T < 0 || T > (1 << 24)) return fail(CAP_E_INVALID, "n >= 0 and 0 <= T <= 2^24 required");
  if (!(cell > 0.0) || !std::isfinite(x0) || !std::isfinite(y0))
    return fail(CAP_E_INVALID, "frame origin must be finite and cell > 0");
  if (n == 0) return CAP_OK;
  if (!start_dev || !beta_dev || !goal_dev) return fail(CAP_E_INVALID, "start/beta/goal is NULL");
  const float one = 1.0f;
  const float zero2[2] = {0.f, 0.f};
  cap_grid g{x0, y0, cell, 1, 1};
  RolloutDesc d;
  st = make_rollout_desc(c, dt, 1, &one, 1, zero2, g, 1, 1, &d);
  if (st != CAP_OK) return st;
  d.shift = 0;
  const uint32_t slo = (uint32_t)seed, shi = (uint32_t)(seed >> 32);
  const dim3 grid_dim((unsigned)((n + 255) / 256)), blk(256);
  hipStream_t s = as_stream(stream);
#define CAP_SIM(KT, MS)                                                                          \
  hipLaunchKernelGGL((simulate_kernel<KT, MS>), grid_dim, blk, 0, s, d, n, T, start_dev, beta_dev, \
                     goal_dev, x0, y0, cell, stream_id, slo, shi, lat_dev, pos_dev)
  switch (d.S > 1 ? -K : (d.sym ? K : 0)) {
    case -4: CAP_SIM(4, true); break;
    case -8: CAP_SIM(8, true); break;
    case -16: CAP_SIM(16, true); break;
    case -32: CAP_SIM(32, true); break;
    case 4: CAP_SIM(4, false); break;
    case 8: CAP_SIM(8, false); break;
    case 16: CAP_SIM(16, false); break;
    case 32: CAP_SIM(32, false); break;
    default: CAP_SIM(0, false); break;
  }
#undef CAP_SIM
  CAP_HIP(hipGetLastError());
  return CAP_OK;
}

extern "C" cap_status cap_philox_blocks(int64_t n, uint32_t c0, uint32_t c1, uint32_t c2,
                                        uint32_t c3, uint64_t seed, uint32_t* out_dev,
                                        void* stream) {
  if (n < 0 || n > ((int64_t)1 << 32)) return fail(CAP_E_INVALID, "n must be in [0, 2^32]");
  if (n == 0) return CAP_OK;
  if (!out_dev) return fail(CAP_E_INVALID, "out is NULL");
  if (reinterpret_cast<uintptr_t>(out_dev) & 15u) return fail(CAP_E_INVALID, "out must be 16-byte aligned");
  hipLaunchKernelGGL(philox_blocks_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                     as_stream(stream), n, c0, c1, c2, c3, (uint32_t)seed, (uint32_t)(seed >> 32),
                     reinterpret_cast<uint4*>(out_dev));
  CAP_HIP(hipGetLastError());
  return CAP_OK;
}
