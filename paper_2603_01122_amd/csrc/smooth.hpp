// smooth.hpp -- the Gaussian smoothing stage shared by the single-grid entry
// point and the batched plan: host-side kernel weights and the device routine
// that smooths one (32 rows x 64 columns) tile of one step's grid.
#pragma once

#include <vector>

#include "common.hpp"

namespace capred {

constexpr int kSmoothThreads = 256;
constexpr int kBandRows = 32;         // output rows per tile (8 per wave)
constexpr int kBandCols = 64;         // output columns per tile (one per lane)
constexpr int kMaxSmoothRadius = 16;

struct SmoothWeights {
  float w[2 * kMaxSmoothRadius + 1];
};

inline cap_status check_smoothing(double sigma, int radius, int max_radius) {
  if (radius < 0 || radius > max_radius)
    return fail(CAP_E_INVALID, "smoothing radius must be in [0, " + std::to_string(max_radius) + "]");
  if (radius > 0 && !(sigma > 0.0 && std::isfinite(sigma)))
    return fail(CAP_E_INVALID, "smoothing sigma must be finite and > 0");
  return CAP_OK;
}

// w[d + r] = fl32(exp(-d^2 / (2 sigma^2)) / sum_{|e| <= r} exp(-e^2 / (2 sigma^2))), FP64 then
// rounded once; r = 0 gives the single weight 1.
inline void smooth_weights(double sigma, int r, SmoothWeights* W) {
  std::vector<double> e(2 * r + 1);
  double Z = 0.0;
  for (int d = -r; d <= r; ++d) {
    e[d + r] = r == 0 ? 1.0 : std::exp(-(double)(d * d) / (2.0 * sigma * sigma));
    Z += e[d + r];
  }
  for (int i = 0; i < 2 * kMaxSmoothRadius + 1; ++i) W->w[i] = i <= 2 * r ? (float)(e[i] / Z) : 0.f;
}

// Compiled radii: a radius runs in the smallest one that holds it, the taps
// beyond it with weight 0 (x + 0 * finite = x, so the results are those of the
// exact radius).
__host__ __device__ constexpr int smooth_bucket(int r) { return r <= 2 ? 2 : r <= 3 ? 3 : r <= 4 ? 4 : r <= 8 ? 8 : 16; }

template <int RM>
struct SmoothTile {
  static constexpr int kHalo = (RM + 3) / 4 * 4;            // left and right, whole float4s
  static constexpr int kRows = kBandRows + 2 * RM;
  static constexpr int kPitch = kBandCols + 2 * kHalo;
  static constexpr size_t kBytes = (size_t)kRows * (kPitch + kBandCols) * sizeof(float);
};

inline size_t smooth_lds_bytes(int r) {
  switch (smooth_bucket(r)) {
    case 2: return SmoothTile<2>::kBytes;
    case 3: return SmoothTile<3>::kBytes;
    case 4: return SmoothTile<4>::kBytes;
    case 8: return SmoothTile<8>::kBytes;
    default: return SmoothTile<16>::kBytes;
  }
}

__host__ __device__ inline int smooth_tiles(int ny, int nx) {
  return ((ny + kBandRows - 1) / kBandRows) * ((nx + kBandCols - 1) / kBandCols);
}

// Smooths output rows [y0, y0 + 32) x columns [x0, x0 + 64) of one step: c and
// o point at that step's [ny][nx] counts and probabilities.  The tile with its
// halo is staged in LDS by row-coalesced loads (all of a thread's loads are in
// flight together); the x pass gives each thread four neighbouring columns of
// a row (its taps are whole 16-byte LDS reads, each used by four sums); the y
// pass gives each thread eight rows of a column, so 8 + 2 RM reads serve
// 8 (2 RM + 1) taps, and writes row-coalesced.  Bound by HBM (4 B read and
// written per cell, the halo from cache); the halo of a 64 x 32 tile costs
// 1.3 x the reads at RM = 3.  100 x 256 x 256 cells at r = 3: 19.4 us, 2.7 TB/s
// of reads and writes (75 us with a thread per column that read each tap from
// memory, one row after another; 10 x 50 x 50 cells: 6.6 us, before 45.6).  Rows off
// the grid are zeros without their sums (50 x 3 x 2000 cells at r = 9: 17.3 us with
// them, 11.4 without).
// Every thread of the block must call it; the caller separates two calls that
// reuse `tile` with another barrier.  un (nullable): that step's plane of a
// union grid of the same frame, raised to each nonzero output by an integer
// atomic max on the FP32 bits (exact for values >= 0).
template <int RM>
__device__ __forceinline__ void smooth_block(const uint32_t* __restrict__ c,
                                             float* __restrict__ o, int ny, int nx, int r,
                                             float Nf, const float* __restrict__ w, int y0,
                                             int x0, float* tile, float* un = nullptr) {
  using T = SmoothTile<RM>;
  float* in = tile;
  float* hx = tile + T::kRows * T::kPitch;
  const int tid = threadIdx.x;
  float wt[2 * RM + 1];
#pragma unroll
  for (int d = -RM; d <= RM; ++d) wt[d + RM] = d >= -r && d <= r ? w[d + r] : 0.f;
#pragma unroll 4
  for (int i = tid; i < T::kRows * T::kPitch; i += kSmoothThreads) {
    const int row = i / T::kPitch, col = i - row * T::kPitch;
    const int y = y0 - RM + row, x = x0 - T::kHalo + col;
    in[i] = y >= 0 && y < ny && x >= 0 && x < nx ? (float)c[(size_t)y * nx + x] : 0.f;
  }
  __syncthreads();
  for (int i = tid; i < T::kRows * (kBandCols / 4); i += kSmoothThreads) {
    const int row = i / (kBandCols / 4), q = i - row * (kBandCols / 4);
    if (y0 - RM + row < 0 || y0 - RM + row >= ny) {   // off the grid: zeros
      reinterpret_cast<float4*>(hx + row * kBandCols)[q] = make_float4(0.f, 0.f, 0.f, 0.f);
      continue;
    }
    float v[4 + 2 * T::kHalo];
    const float4* src = reinterpret_cast<const float4*>(in + row * T::kPitch) + q;
#pragma unroll
    for (int k = 0; k < 1 + T::kHalo / 2; ++k) {
      const float4 f = src[k];
      v[4 * k] = f.x;
      v[4 * k + 1] = f.y;
      v[4 * k + 2] = f.z;
      v[4 * k + 3] = f.w;
    }
    float h[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = -RM; d <= RM; ++d)
#pragma unroll
      for (int k = 0; k < 4; ++k) h[k] = fmaf(wt[d + RM], v[T::kHalo + k - d], h[k]);
    reinterpret_cast<float4*>(hx + row * kBandCols)[q] = make_float4(h[0], h[1], h[2], h[3]);
  }
  __syncthreads();
  constexpr int kPer = kBandRows / (kSmoothThreads / kBandCols);
  const int col = tid & (kBandCols - 1), j0 = (tid / kBandCols) * kPer, x = x0 + col;
  float v[kPer + 2 * RM];
#pragma unroll
  for (int k = 0; k < kPer + 2 * RM; ++k) v[k] = hx[(j0 + k) * kBandCols + col];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    float acc = 0.f;
#pragma unroll
    for (int d = -RM; d <= RM; ++d) acc = fmaf(wt[d + RM], v[k + RM - d], acc);
    const int y = y0 + j0 + k;
    if (x < nx && y < ny) {
      const float p = acc / Nf;
      o[(size_t)y * nx + x] = p;
      if (un && p > 0.f)
        __hip_atomic_fetch_max(reinterpret_cast<uint32_t*>(un) + (size_t)y * nx + x,
                               __float_as_uint(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

}  // namespace capred
