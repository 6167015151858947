// belief.hip -- cap_belief_update and cap_belief_reset (single human).
#include "belief.hpp"

namespace capred {

// Policy terms times controls (a Delta costs about three of them) above which
// the update is split over blocks: at 7680 (10 goals x 96 controls x 5 betas,
// one observation) one block takes 10.9 us; the split's second launch alone
// takes 4 us, and at 17280 (30 observations of 16 controls, 3 goals x 9 betas)
// the two launches take 5.5 + 4 us.
constexpr double kSplitWork = 8192.0;

// Blocks of the update (grid.x) share the pairs: one block does everything and
// normalises; several take one pair each and belief_normalize_kernel follows.
__global__ void __launch_bounds__(kBeliefThreadsWide)
    belief_update_kernel(const BeliefModel m, const float* __restrict__ obs, int n_obs,
                         double* log_belief, double* belief_out) {
  __shared__ BeliefShared<kBeliefThreadsWide> sh;
  if (gridDim.x == 1) {
    belief_terms_any(m, obs, n_obs, log_belief, 0, m.G, 0, m.B, sh);
    belief_normalize(m.G * m.B, log_belief, belief_out);
  } else {
    const int g = (int)blockIdx.x / m.B, b = (int)blockIdx.x - g * m.B;
    belief_terms_any(m, obs, n_obs, log_belief, g, g + 1, b, b + 1, sh);
  }
}

__global__ void __launch_bounds__(64)
    belief_normalize_kernel(int J, double* log_belief, double* belief_out) {
  belief_normalize(J, log_belief, belief_out);
}

__global__ void belief_reset_kernel(int J, double* log_belief) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < J) log_belief[j] = -log((double)J);
}

}  // namespace capred

using namespace capred;

extern "C" cap_status cap_belief_update(const cap_model* model, const float* obs_dev,
                                        int32_t n_obs, double* log_belief_dev,
                                        double* belief_dev, void* stream) {
  Controls c;
  cap_status st = check_model(model, &c);
  if (st != CAP_OK) return st;
  if (n_obs < 0) return fail(CAP_E_INVALID, "n_obs must be >= 0");
  if (!log_belief_dev) return fail(CAP_E_INVALID, "log_belief is NULL");
  if (n_obs > 0 && !obs_dev) return fail(CAP_E_INVALID, "obs is NULL");
  const BeliefModel m = make_belief_model(c, model->dt, model->B, model->beta, model->G,
                                          model->goals);
  // One block while its share of a CU's FP64 work stays below the cost of a
  // second launch; beyond that one block per (goal, beta) pair.
  const double deltas = (double)n_obs * m.G * m.U;
  const bool split = m.G * m.B > 1 && deltas * (3.0 + m.B) > kSplitWork;
  hipStream_t s = as_stream(stream);
  hipLaunchKernelGGL(belief_update_kernel, dim3(split ? m.G * m.B : 1), dim3(kBeliefThreadsWide),
                     0, s, m, obs_dev, n_obs, log_belief_dev, belief_dev);
  if (split)
    hipLaunchKernelGGL(belief_normalize_kernel, dim3(1), dim3(64), 0, s, m.G * m.B,
                       log_belief_dev, belief_dev);
  CAP_HIP(hipGetLastError());
  return CAP_OK;
}

extern "C" cap_status cap_belief_reset(int32_t G, int32_t B, double* log_belief_dev,
                                       void* stream) {
  if (G < 1 || B < 1 || G > CAP_MAX_G || B > CAP_MAX_B || G * B > CAP_MAX_J)
    return fail(CAP_E_INVALID, "G, B out of range");
  if (!log_belief_dev) return fail(CAP_E_INVALID, "log_belief is NULL");
  hipLaunchKernelGGL(belief_reset_kernel, dim3(1), dim3(CAP_MAX_J), 0, as_stream(stream), G * B,
                     log_belief_dev);
  CAP_HIP(hipGetLastError());
  return CAP_OK;
}
