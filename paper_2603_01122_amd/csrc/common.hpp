// common.hpp -- internal definitions shared by the libcapred translation units:
// error reporting, host-side model tables, and the device building blocks of
// the rollout (counter-based Philox, Boltzmann heading choice).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <string>

#include "../../include/capred.h"

namespace capred {

// ---------------------------------------------------------------- errors
void set_error(const std::string& msg);
cap_status fail(cap_status code, const std::string& msg);
cap_status hip_fail(hipError_t e, const char* what);

#define CAP_HIP(call)                                   \
  do {                                                  \
    hipError_t e_ = (call);                             \
    if (e_ != hipSuccess) return hip_fail(e_, #call);   \
  } while (0)

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

constexpr double kPi = 3.14159265358979323846;
constexpr int kLatticeShift = 16;          // q = cell / 2^16
constexpr double kLatticeScale = 65536.0;
constexpr float kLog2e = 1.4426950408889634f;

// Largest beta * step length (metres) for which exp2 of the unshifted logits
// cannot overflow in FP32 (sum of up to 32 terms of 2^(80 log2 e)).
constexpr double kNoShiftLimit = 80.0;

// ---------------------------------------------------------------- host lattice
// Lattice pitch and rounding of metres to lattice units (round half to even).
// Written without FP contraction so that every host computes identical bits.
inline double lattice_pitch(double cell) { return cell / kLatticeScale; }

inline double lattice_coord(double z, double origin, double cell) {
#pragma clang fp contract(off)
  return std::nearbyint((z - origin) / lattice_pitch(cell));
}

inline double heading_angle(int k, int K) {
#pragma clang fp contract(off)
  return 2.0 * kPi * (double)k / (double)K;
}

// Lattice step of heading k: rint(v dt cos(theta_k) / q), rint(v dt sin(theta_k) / q).
inline void lattice_step(int k, int K, double speed, double dt, double cell, int32_t* sx,
                         int32_t* sy) {
#pragma clang fp contract(off)
  const double L = speed * dt;
  const double q = lattice_pitch(cell);
  const double th = heading_angle(k, K);
  *sx = (int32_t)std::nearbyint(L * std::cos(th) / q);
  *sy = (int32_t)std::nearbyint(L * std::sin(th) / q);
}

// Continuous step of heading k in metres, rounded to FP32.
inline void continuous_step(int k, int K, double speed, double dt, float* sx, float* sy) {
#pragma clang fp contract(off)
  const double L = speed * dt;
  const double th = heading_angle(k, K);
  *sx = (float)(L * std::cos(th));
  *sy = (float)(L * std::sin(th));
}

// ---------------------------------------------------------------- device
// Three-input exclusive or in one gfx950 V_BITOP3_B32 (truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Philox4x32-10 (Salmon et al., SC'11): per round two 32x32->64-bit products of
// counter words 0 and 2, recombined with words 1 and 3 and the round key; the
// key advances by the Weyl constants between rounds.
__device__ __forceinline__ uint4 philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                          uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // one v_mad_u64_u32 per product gives both halves
    const uint64_t p0 = (uint64_t)c0 * 0xD2511F53u;
    const uint64_t p1 = (uint64_t)c2 * 0xCD9E8D57u;
    const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
    const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
    c0 = n0;
    c1 = (uint32_t)p1;
    c2 = n2;
    c3 = (uint32_t)p0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return make_uint4(c0, c1, c2, c3);
}

// u = (2 (w >> 9) + 1) 2^-24: 24 significant bits, exact in FP32 and FP64.
// In FP32 as two instructions: one funnel shift places w >> 9 in the mantissa
// of 1.0 (x = 1 + (w >> 9) 2^-23), then x - (1 - 2^-24), exact by Sterbenz's
// lemma (x and 1 - 2^-24 are within a factor of two).
__device__ __forceinline__ float uniform24f(uint32_t w) {
  const uint32_t x = __builtin_amdgcn_alignbit(0x7Fu, w, 9u);  // 0x3F800000 | (w >> 9)
  return __uint_as_float(x) - 0x1.fffffep-1f;
}
__device__ __forceinline__ double uniform24d(uint32_t w) {
  return (double)((w >> 9) * 2u + 1u) * 5.9604644775390625e-8;
}

// Global-memory (address space 1) view of a generic pointer.  Pointers that a
// kernel loads from descriptor tables in device memory are generic to the
// compiler, which then emits FLAT accesses; a FLAT access also counts on the
// LDS wait counter, so every later LDS wait (each barrier, each LDS atomic
// whose result is used) would wait for its round trip to memory.
template <typename T>
using global_ptr = __attribute__((address_space(1))) T*;

template <typename T>
__device__ __forceinline__ global_ptr<T> as_global(T* p) {
  return (global_ptr<T>)p;
}

// Relaxed device-scope integer add through the global path (no return value).
__device__ __forceinline__ void global_add(uint32_t* p, uint32_t v) {
  __hip_atomic_fetch_add(as_global(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Per-model control constants for the lattice rollout, in lattice units:
// step (fx, fy) of control u = s K + k (integers, exact in FP32) and its
// squared length s2 (FP32).
struct HeadingTable {
  float fx[CAP_MAX_U];
  float fy[CAP_MAX_U];
  float s2[CAP_MAX_U];
};

// Inverse CDF over K non-decreasing prefix sums: #{k < K-1 : C_k <= thr},
// which equals min{k : thr < C_k} (capped at K-1).  For K a power of two the
// count is found by a branchless binary search whose register selections are
// explicit conditional moves (per-lane dynamic indexing of registers would
// spill to scratch); otherwise by counting.
template <int KT>
__device__ __forceinline__ int cdf_index(const float* C, float thr, int Krt) {
  constexpr bool kPow2 = KT >= 4 && (KT & (KT - 1)) == 0;
  if constexpr (kPow2) {
    // Level l probes C[c * (KT >> l) + (KT >> (l + 1)) - 1] where the bits
    // b_0..b_{l-1} decided so far spell c (b_0 most significant); the probe is
    // picked by a tree of 2^l - 1 conditional moves on those bits.
    constexpr int L = KT == 4 ? 2 : KT == 8 ? 3 : KT == 16 ? 4 : KT == 32 ? 5 : 6;
    bool b[L];
    int pos = 0;
#pragma unroll
    for (int l = 0; l < L; ++l) {
      float v[KT / 2];
#pragma unroll
      for (int c = 0; c < (1 << l); ++c) v[c] = C[c * (KT >> l) + (KT >> (l + 1)) - 1];
#pragma unroll
      for (int st = l - 1; st >= 0; --st)
#pragma unroll
        for (int j = 0; j < (1 << st); ++j) v[j] = b[st] ? v[2 * j + 1] : v[2 * j];
      b[l] = v[0] <= thr;
      pos += b[l] ? (KT >> (l + 1)) : 0;
    }
    return pos;
  } else {
    constexpr int KM = KT > 0 ? KT : CAP_MAX_K;
    const int K = KT > 0 ? KT : Krt;
    int kk = 0;
#pragma unroll
    for (int k = 0; k < KM - 1; ++k) {
      if (KT == 0 && k >= K - 1) break;
      kk += (C[k] <= thr) ? 1 : 0;
    }
    return kk;
  }
}

// Boltzmann heading draw at lattice offset a = x - g (lattice units).  The
// logit of heading k is beta (|a| - |a + s_k|) (shift-invariant form of
// beta Q_k); it is computed from the cancellation-free difference
//   Delta_k = |a + s_k| - |a| = n_k / (|a + s_k| + |a|),  n_k = 2 a.s_k + |s_k|^2,
// whose absolute error stays a few ulp of the step length however far the
// goal is.  With nb = -beta q log2(e) and ib = 1/nb (both per particle), the
// base-2 exponent nb Delta_k is n_k / (|a + s_k| ib + |a| ib): one FMA, one
// reciprocal and one multiply.  |a + s_k|^2 = |a|^2 + n_k is taken through
// |.| (a free source modifier) against rounding below zero at the goal.
// Weights w_k = exp2(exponent) (optionally shifted by the largest exponent),
// prefix sums C_k, heading = cdf_index(C, u C_{K-1}).
//
// For KT > 0 the step table is point-symmetric (s_{k+KT/2} = -s_k, checked on
// the host), so one dot product 2 a.s_k serves both opposite headings:
// n_{k} = |s_k|^2 + 2 a.s_k and n_{k+KT/2} = |s_k|^2 - 2 a.s_k.  KT == 0 is the
// general table with a run-time K.
//
// SHIFT (a compile-time variant, used when beta * step is large enough for
// exp2 to overflow) subtracts the largest exponent before exponentiating.
//
// draw_headings: M particles' draws in one pass (KT > 0): the operations of each particle
// are the same and in the same order for every M, so its heading is the same
// bit for bit; with M = 2 the two particles' heading terms stand side by side,
// which gives the scheduler two independent sqrt -> rcp -> exp2 chains.
template <int KT, bool SHIFT, int M>
__device__ __forceinline__ void draw_headings(const float* ax, const float* ay, const float* ib,
                                              const float* u, const HeadingTable& T, int* k_out) {
  static_assert(KT > 0 && KT % 2 == 0, "needs a compile-time, point-symmetric table");
  constexpr int KH = KT / 2;
  float D2[M], Dib[M], ax2[M], ay2[M], acc[M];
  float C[M][KT];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    D2[m] = fmaf(ax[m], ax[m], ay[m] * ay[m]);
    Dib[m] = fast_sqrt(D2[m]) * ib[m];
    ax2[m] = ax[m] + ax[m];
    ay2[m] = ay[m] + ay[m];
  }
  // exponents of both halves, then the prefix sum in heading order
#pragma unroll
  for (int k = 0; k < KH; ++k) {
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const float dot = fmaf(ax2[m], T.fx[k], ay2[m] * T.fy[k]);
      const float np = T.s2[k] + dot, nm = T.s2[k] - dot;
      const float dp = fast_sqrt(fabsf(D2[m] + np)), dm = fast_sqrt(fabsf(D2[m] + nm));
      C[m][k] = np * fast_rcp(fmaf(dp, ib[m], Dib[m]));
      C[m][k + KH] = nm * fast_rcp(fmaf(dm, ib[m], Dib[m]));
    }
  }
  if constexpr (SHIFT) {
#pragma unroll
    for (int m = 0; m < M; ++m) {
      float mx = C[m][0];
#pragma unroll
      for (int k = 1; k < KT; ++k) mx = fmaxf(mx, C[m][k]);
#pragma unroll
      for (int k = 0; k < KT; ++k) C[m][k] -= mx;
    }
  }
#pragma unroll
  for (int m = 0; m < M; ++m) {
    acc[m] = fast_exp2(C[m][0]);
    C[m][0] = acc[m];
  }
#pragma unroll
  for (int k = 1; k < KT; ++k)
#pragma unroll
    for (int m = 0; m < M; ++m) {
      acc[m] += fast_exp2(C[m][k]);
      C[m][k] = acc[m];
    }
#pragma unroll
  for (int m = 0; m < M; ++m) k_out[m] = cdf_index<KT>(C[m], u[m] * acc[m], KT);
}

// ---------------------------------------------------------------- far draws
// Most particles are many steps away from their goal, and there the exponents
// of all K headings follow from a few harmonics of the heading angle.  With
// r = |a|, x = |s| / r and psi the angle between a and s_k,
//   (|a + s_k| - |a|) / |s| = (1 - x^2/8) cos psi - (x/4) cos 2 psi
//                             + (x^2/8) cos 3 psi + const + e,  |e| <= 0.1154 x^3
// (x <= 0.12; the constant cancels in the policy, and e is what is left at the best
// one: its x^3 term is (1 - c^2) (5 c^2 - 1) / 8, c = cos psi, which alone spans
// 0.2251 x^3).  Of a particle's features
// f_m = nb |s| (...) u^m (u the unit vector of a) the exponents of the four
// headings theta + 90 j are even + odd, -even + odd', even - odd and
// -even - odd', so that 16 headings take 36 operations instead of the 96 and the
// 16 square roots and reciprocals of draw_headings.  The VALU does them: FP32
// matrix instructions do not overlap with it here, and 24 of them per draw (16
// headings x 6 coefficients) took as long as what they replaced.
//
// The result is a filter, not an approximation of the draw: the heading of the
// inverse CDF is taken only where u lies farther than `tol` (relative to the
// total) from the CDF boundaries beside it, a bound on the difference of the two
// computations; otherwise the caller runs draw_headings.  So the headings are
// draw_headings' in every case, bit for bit.  tol = c0 + |nb s| (c1 + 0.0405 x^3):
//   * draw_headings itself: each exponent within 6.1 2^-23 |nb s| (dot product,
//     square roots and reciprocal within 1 ulp, products), so with a weight's
//     relative error w a CDF value errs by at most w/2; exp2 within 1 ulp; K - 1
//     additions and the threshold's product, 2^-24 each;
//   * here: features and their sums within 13 2^-24 |nb s|, the cut-off e |nb s|,
//     the lattice's rounding of the steps (0.71 units, 0.71 |nb|), exp2 and the
//     same additions.
// Exponents are base 2, so an error of v |nb s| in them is w = ln 2 v |nb s| in a
// weight.  Together K 2.4e-7 + 2e-7 + |nb s| (6e-7 + 0.0400 x^3 + 0.25 / |s|); the
// host takes 1.25 times the rounding terms.  (The cut-off's part is not reached:
// the largest found over psi, x, |nb s| and K = 8, 16, 32 is 0.016 |nb s| x^3.)  At most 2 (K - 1) tol of the draws fall
// back: 2e-4 at K = 16 and small |nb s|.
//
// Bound by VALU issue as before, with fewer slots: 120 instructions a draw
// instead of 170 at K = 16 (17 transcendental instead of 49, two slots each), 174
// instead of 219 a particle-step with everything else.  A cycle of the
// 16-human workload takes 0.91 ms instead of 1.18, one of 64 humans x 2^20
// particles (K = 32) 125 ms instead of 178 (each at its best launch shape).
struct FarConst {
  float d2;       // smallest |a|^2 (lattice units) the filter takes; inf: none
  float s4;       // -|s| / 4
  float c0, c1;   // tol = c0 + |nb s| (c1 + kFarCut x^3)
};
constexpr float kFarX = 0.12f;       // largest x
constexpr float kFarCut = 0.0405f;

// cos(11.25 i degrees), i = 0..8
constexpr float kCos32[9] = {1.f,          0.98078528f, 0.92387953f, 0.83146961f, 0.70710678f,
                             0.55557023f, 0.38268343f, 0.19509032f, 0.f};
// cos and sin of i * 11.25 degrees, any i >= 0
constexpr float cos32(int i) {
  i &= 31;
  return i <= 8 ? kCos32[i] : i <= 16 ? -kCos32[16 - i] : i <= 24 ? -kCos32[i - 16] : kCos32[32 - i];
}
constexpr float sin32(int i) { return cos32(i + 24); }

// Exponents of headings I, I + K/4, I + K/2, I + 3K/4 and of the following
// base headings.  f3 is half the third feature.
template <int KT, int I>
__device__ __forceinline__ void far_exponents(float f1x, float f1y, float f2x, float f2y,
                                              float f3x, float f3y, float* E) {
  if constexpr (I < KT / 4) {
    constexpr int a = I * (32 / KT);   // theta_I in units of 11.25 degrees
    float o0, o1, e, h;                // exponents +-h e +- o0 (0, 180), +- o1 (90, 270)
    if constexpr (a == 0) {
      o0 = fmaf(2.f, f3x, f1x);
      o1 = fmaf(-2.f, f3y, f1y);
      e = f2x;
      h = 1.f;
    } else if constexpr (a == 4) {
      const float p = fmaf(-2.f, f3x, f1x), q = fmaf(2.f, f3y, f1y);
      o0 = p + q;
      o1 = q - p;
      e = f2y;
      h = 1.f;
    } else if constexpr (a == 2) {
      const float m = fmaf(2.f, f3y, f1x), n = fmaf(2.f, f3x, f1y);
      o0 = fmaf(cos32(2), m, sin32(2) * n);
      o1 = fmaf(cos32(2), n, -(sin32(2) * m));
      e = f2x + f2y;
      h = cos32(4);
    } else if constexpr (a == 6) {
      const float m = fmaf(-2.f, f3y, f1x), n = fmaf(-2.f, f3x, f1y);
      o0 = fmaf(cos32(6), m, sin32(6) * n);
      o1 = fmaf(cos32(6), n, -(sin32(6) * m));
      e = f2y - f2x;
      h = cos32(4);
    } else {
      constexpr float c3 = 2.f * cos32(3 * a), s3 = 2.f * sin32(3 * a);
      o0 = fmaf(c3, f3x, fmaf(s3, f3y, fmaf(cos32(a), f1x, sin32(a) * f1y)));
      o1 = fmaf(s3, f3x, fmaf(-c3, f3y, fmaf(cos32(a), f1y, -(sin32(a) * f1x))));
      e = fmaf(cos32(2 * a), f2x, sin32(2 * a) * f2y);
      h = 1.f;
    }
    if constexpr (a == 4) {
      E[I] = fmaf(cos32(4), o0, e);
      E[I + KT / 4] = fmaf(cos32(4), o1, -e);
      E[I + KT / 2] = fmaf(-cos32(4), o0, e);
      E[I + 3 * KT / 4] = fmaf(-cos32(4), o1, -e);
    } else if constexpr (a == 2 || a == 6) {
      E[I] = fmaf(h, e, o0);
      E[I + KT / 4] = fmaf(-h, e, o1);
      E[I + KT / 2] = fmaf(h, e, -o0);
      E[I + 3 * KT / 4] = fmaf(-h, e, -o1);
    } else {
      E[I] = e + o0;
      E[I + KT / 4] = o1 - e;
      E[I + KT / 2] = e - o0;
      E[I + 3 * KT / 4] = -e - o1;
    }
    far_exponents<KT, I + 1>(f1x, f1y, f2x, f2y, f3x, f3y, E);
  }
}

// cdf_index for a power-of-two K, with the distance of thr to the nearest
// boundary (the search passes both neighbours of thr).
template <int KT>
__device__ __forceinline__ int cdf_index_margin(const float* C, float thr, float* margin) {
  constexpr int L = KT == 4 ? 2 : KT == 8 ? 3 : KT == 16 ? 4 : 5;
  bool b[L];
  int pos = 0;
  float md = INFINITY;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    float v[KT / 2];
#pragma unroll
    for (int c = 0; c < (1 << l); ++c) v[c] = C[c * (KT >> l) + (KT >> (l + 1)) - 1];
#pragma unroll
    for (int st = l - 1; st >= 0; --st)
#pragma unroll
      for (int j = 0; j < (1 << st); ++j) v[j] = b[st] ? v[2 * j + 1] : v[2 * j];
    b[l] = v[0] <= thr;
    pos += b[l] ? (KT >> (l + 1)) : 0;
    md = fminf(md, fabsf(v[0] - thr));
  }
  *margin = md;
  return pos;
}

// Headings of M far particles; true if all of this lane's are certain.  D2 =
// |a|^2 >= F.d2, nbs = nb |s|.
template <int KT, int M>
__device__ __forceinline__ bool far_headings(const float* ax, const float* ay, const float* D2,
                                             const float* nbs, const float* u, const FarConst& F,
                                             int* k_out) {
  static_assert(KT == 8 || KT == 16 || KT == 32, "headings in quarter turns");
  float C[M][KT], acc[M], tol[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const float ir = __builtin_amdgcn_rsqf(D2[m]);
    const float x4 = F.s4 * ir, xx = x4 * x4;                      // -x / 4, x^2 / 16
    const float n1 = nbs[m] * ir * fmaf(xx, -2.f, 1.f);            // nb s (1 - x^2/8) / r
    tol[m] = fmaf(nbs[m], fmaf(x4 * xx, 64.f * kFarCut, -F.c1), F.c0);   // nbs, x4 <= 0
    const float xi = x4 * ir;
    const float wx = ax[m] * xi, wy = ay[m] * xi;                  // -(x/4) u
    const float f1x = ax[m] * n1, f1y = ay[m] * n1;
    const float f2x = fmaf(f1x, wx, -(f1y * wy)), f2y = fmaf(f1x, wy, f1y * wx);
    const float f3x = fmaf(f2x, wx, -(f2y * wy)), f3y = fmaf(f2x, wy, f2y * wx);
    far_exponents<KT, 0>(f1x, f1y, f2x, f2y, f3x, f3y, C[m]);
  }
#pragma unroll
  for (int m = 0; m < M; ++m) acc[m] = C[m][0] = fast_exp2(C[m][0]);
#pragma unroll
  for (int k = 1; k < KT; ++k)
#pragma unroll
    for (int m = 0; m < M; ++m) {
      acc[m] += fast_exp2(C[m][k]);
      C[m][k] = acc[m];
    }
  bool sure = true;
#pragma unroll
  for (int m = 0; m < M; ++m) {
    float margin;
    k_out[m] = cdf_index_margin<KT>(C[m], u[m] * acc[m], &margin);
    sure = sure && margin > tol[m] * acc[m];
  }
  return sure;
}

template <int KT, bool SHIFT>
__device__ __forceinline__ int draw_heading(float ax, float ay, float ib, float u,
                                            const HeadingTable& T, int Krt) {
  if constexpr (KT > 0) {
    int k;
    draw_headings<KT, SHIFT, 1>(&ax, &ay, &ib, &u, T, &k);
    return k;
  } else {
    const float D2 = fmaf(ax, ax, ay * ay);
    const float D = fast_sqrt(D2);
    const float Dib = D * ib;
    const float ax2 = ax + ax, ay2 = ay + ay;
    float C[CAP_MAX_K];
    float acc = 0.f;
    float m = -INFINITY;
#pragma unroll
    for (int k = 0; k < CAP_MAX_K; ++k) {
      if (k >= Krt) break;
      const float n = fmaf(ax2, T.fx[k], fmaf(ay2, T.fy[k], T.s2[k]));
      const float d = fast_sqrt(fabsf(D2 + n));
      C[k] = n * fast_rcp(fmaf(d, ib, Dib));
      if constexpr (SHIFT) m = fmaxf(m, C[k]);
    }
#pragma unroll
    for (int k = 0; k < CAP_MAX_K; ++k) {
      if (k >= Krt) break;
      acc += fast_exp2(SHIFT ? C[k] - m : C[k]);
      C[k] = acc;
    }
    return cdf_index<KT>(C, u * acc, Krt);
  }
}

// Multi-speed draw: the inverse CDF over all U = S KT controls (u = s KT + k,
// prefix sums in u order) in two passes.  Pass 1 accumulates the weights of
// every allowed speed block in u order and keeps the running sum at the end of
// each block; the speed block s* = min{s : x < sum_s} (x = u C_{U-1}, capped at
// the last allowed speed) follows from those S sums.  Pass 2 recomputes block
// s* from the same constants (LDS copy `ctl`, per-lane index) starting from the
// sum before it, so its prefix sums are bit-identical to the flat sequence,
// and the heading is cdf_index over them.  Blocks of masked speeds add nothing
// (weight 0, Q = -inf).  Requires a point-symmetric table per speed.
template <int KT, bool SHIFT>
__device__ __forceinline__ int draw_control(float ax, float ay, float ib, float u,
                                            const HeadingTable& T, int S, uint32_t smask,
                                            int s_last, const float4* ctl) {
  static_assert(KT >= 4 && (KT & (KT - 1)) == 0, "multi-speed draw needs a power-of-two K");
  constexpr int KH = KT / 2;
  const float D2 = fmaf(ax, ax, ay * ay);
  const float D = fast_sqrt(D2);
  const float Dib = D * ib;
  const float ax2 = ax + ax, ay2 = ay + ay;
  float m = 0.f;
  if constexpr (SHIFT) {
    m = -INFINITY;
#pragma unroll
    for (int s = 0; s < CAP_MAX_S; ++s) {
      if (s >= S) break;
      if (!((smask >> s) & 1u)) continue;
#pragma unroll
      for (int k = 0; k < KH; ++k) {
        const int c = s * KT + k;
        const float dot = fmaf(ax2, T.fx[c], ay2 * T.fy[c]);
        const float np = T.s2[c] + dot, nm = T.s2[c] - dot;
        const float dp = fast_sqrt(fabsf(D2 + np)), dm = fast_sqrt(fabsf(D2 + nm));
        m = fmaxf(m, fmaxf(np * fast_rcp(fmaf(dp, ib, Dib)), nm * fast_rcp(fmaf(dm, ib, Dib))));
      }
    }
  }
  float bs[CAP_MAX_S];
  float acc = 0.f;
#pragma unroll
  for (int s = 0; s < CAP_MAX_S; ++s) {
    if (s < S && ((smask >> s) & 1u)) {
      float e[KT];
#pragma unroll
      for (int k = 0; k < KH; ++k) {
        const int c = s * KT + k;
        const float dot = fmaf(ax2, T.fx[c], ay2 * T.fy[c]);
        const float np = T.s2[c] + dot, nm = T.s2[c] - dot;
        const float dp = fast_sqrt(fabsf(D2 + np)), dm = fast_sqrt(fabsf(D2 + nm));
        e[k] = np * fast_rcp(fmaf(dp, ib, Dib));
        e[k + KH] = nm * fast_rcp(fmaf(dm, ib, Dib));
      }
#pragma unroll
      for (int k = 0; k < KT; ++k) acc += fast_exp2(SHIFT ? e[k] - m : e[k]);
    }
    bs[s] = acc;
  }
  const float thr = u * acc;
  int ss = 0;
#pragma unroll
  for (int s = 0; s < CAP_MAX_S - 1; ++s) ss += (s < s_last && bs[s] <= thr) ? 1 : 0;
  float base = 0.f;
#pragma unroll
  for (int s = 0; s < CAP_MAX_S - 1; ++s) base = (s == ss - 1) ? bs[s] : base;
  float C[KT];
  const float4* cb = ctl + ss * KT;
#pragma unroll
  for (int k = 0; k < KH; ++k) {
    const float4 c = cb[k];
    const float dot = fmaf(ax2, c.x, ay2 * c.y);
    const float np = c.z + dot, nm = c.z - dot;
    const float dp = fast_sqrt(fabsf(D2 + np)), dm = fast_sqrt(fabsf(D2 + nm));
    C[k] = np * fast_rcp(fmaf(dp, ib, Dib));
    C[k + KH] = nm * fast_rcp(fmaf(dm, ib, Dib));
  }
  float a2 = base;
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    a2 += fast_exp2(SHIFT ? C[k] - m : C[k]);
    C[k] = a2;
  }
  return ss * KT + cdf_index<KT>(C, thr, KT);
}

// ---------------------------------------------------------------- wide draws
// draw_control (unshifted) of one particle by L = 4 or 8 neighbouring lanes, for
// launches whose particles leave the device idle: with one lane per particle a
// step is one lane's S KT controls in series, at one wave per SIMD 5 us a step
// for 96 controls; by 8 lanes 2.1 us (8192 particles x 10 steps of 6 x 16
// controls, the whole launch 52 -> 34 us).  The chain of S KT dependent additions,
// 8-10 cycles each with so few waves, is what remains.  Lane `sub` forms the weights of the heading pairs k, k + KT/2
// with k = sub, sub + L, ... of every speed, by draw_control's operations; the
// prefix sums then run over the lanes in control order (each addition takes its
// weight from the lane that holds it by a DPP move in the same instruction), so
// the sums, and the control, are draw_control's bit for bit.  At L = 8 the
// running sums are those of the group's first quad, which sees the second quad's
// weights mirrored.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __uint_as_float(
      (uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), CTRL, 0xF, 0xF, true));
}

// Calls f(weight of lane j) for the L lanes of the group in order.
template <int L, class F>
__device__ __forceinline__ void in_lane_order(float w, F f) {
  f(dpp_f<0x00>(w));
  f(dpp_f<0x55>(w));
  f(dpp_f<0xAA>(w));
  f(dpp_f<0xFF>(w));
  if constexpr (L == 8) {
    const float m = dpp_f<0x141>(w);   // lane i of the first quad: lane 7 - i's
    f(dpp_f<0xFF>(m));
    f(dpp_f<0xAA>(m));
    f(dpp_f<0x55>(m));
    f(dpp_f<0x00>(m));
  }
}

// The first quad's value in both.
template <int L>
__device__ __forceinline__ int from_first_quad(int v, int sub) {
  if constexpr (L == 8) {
    const int m = __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true);
    return sub < 4 ? v : m;
  }
  return v;
}

// This lane's rows of the control table for its NP heading pairs, by speed, in
// registers where they are few (one pair); else the draw reads them from ctl.
template <int KT, int L>
struct WideRows {
  static constexpr int NP = KT / 2 / L;      // heading pairs of a lane
  static_assert(NP * L * 2 == KT, "whole pairs per lane");
  static constexpr bool kHeld = NP == 1;
  float x[kHeld ? CAP_MAX_S : 1][NP], y[kHeld ? CAP_MAX_S : 1][NP], z[kHeld ? CAP_MAX_S : 1][NP];
  __device__ __forceinline__ void load(const float4* ctl, int S, int sub) {
    if constexpr (kHeld)
#pragma unroll
      for (int s = 0; s < CAP_MAX_S; ++s)
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          const float4 c = ctl[min(s, S - 1) * KT + sub + L * i];
          x[s][i] = c.x;
          y[s][i] = c.y;
          z[s][i] = c.z;
        }
  }
};

// Every lane of the wave must call it; ctl as for draw_control.
template <int KT, int L>
__device__ __forceinline__ int wide_control(float ax, float ay, float ib, float u, int S,
                                            uint32_t smask, int s_last,
                                            const WideRows<KT, L>& rows, const float4* ctl,
                                            int sub) {
  constexpr int NP = WideRows<KT, L>::NP;
  constexpr bool kHeld = WideRows<KT, L>::kHeld;
  const float D2 = fmaf(ax, ax, ay * ay);
  const float D = fast_sqrt(D2);
  const float Dib = D * ib;
  const float ax2 = ax + ax, ay2 = ay + ay;
  // weights of the opposite headings (fx, fy) and (-fx, -fy)
  const auto weights = [&](float fx, float fy, float s2, float* wp, float* wm) {
    const float dot = fmaf(ax2, fx, ay2 * fy);
    const float np = s2 + dot, nm = s2 - dot;
    const float dp = fast_sqrt(fabsf(D2 + np)), dm = fast_sqrt(fabsf(D2 + nm));
    *wp = fast_exp2(np * fast_rcp(fmaf(dp, ib, Dib)));
    *wm = fast_exp2(nm * fast_rcp(fmaf(dm, ib, Dib)));
  };
  // Two speeds at a time, without a branch between them: the second one's weights
  // fill the waits of the first one's chain of additions.  A speed that is not
  // allowed adds zeros.
  float wp[CAP_MAX_S][NP], wm[CAP_MAX_S][NP];
  float bs[CAP_MAX_S];
  float acc = 0.f;
#pragma unroll
  for (int s0 = 0; s0 < CAP_MAX_S; s0 += 2) {
    if (s0 < S) {
#pragma unroll
      for (int s = s0; s < s0 + 2; ++s) {
        const bool allowed = s < S && ((smask >> s) & 1u);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          if constexpr (kHeld) {
            weights(rows.x[s][i], rows.y[s][i], rows.z[s][i], &wp[s][i], &wm[s][i]);
          } else {
            const float4 c = ctl[min(s, S - 1) * KT + sub + L * i];
            weights(c.x, c.y, c.z, &wp[s][i], &wm[s][i]);
          }
          wp[s][i] = allowed ? wp[s][i] : 0.f;
          wm[s][i] = allowed ? wm[s][i] : 0.f;
        }
      }
#pragma unroll
      for (int s = s0; s < s0 + 2; ++s) {
#pragma unroll
        for (int i = 0; i < NP; ++i) in_lane_order<L>(wp[s][i], [&](float w) { acc += w; });
#pragma unroll
        for (int i = 0; i < NP; ++i) in_lane_order<L>(wm[s][i], [&](float w) { acc += w; });
        bs[s] = acc;
      }
    } else {
#pragma unroll
      for (int s = s0; s < s0 + 2; ++s) {
        bs[s] = acc;
#pragma unroll
        for (int i = 0; i < NP; ++i) wp[s][i] = wm[s][i] = 0.f;
      }
    }
  }
  const float thr = u * acc;
  int ss = 0;
  float prev = 0.f;
#pragma unroll
  for (int s = 0; s < CAP_MAX_S - 1; ++s) {
    const bool right = s < s_last && bs[s] <= thr;
    ss += right ? 1 : 0;
    prev = right ? bs[s] : prev;
  }
  ss = from_first_quad<L>(ss, sub);
  if constexpr (kHeld) {
#pragma unroll
    for (int s = 1; s < CAP_MAX_S; ++s)
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        wp[0][i] = ss == s ? wp[s][i] : wp[0][i];
        wm[0][i] = ss == s ? wm[s][i] : wm[0][i];
      }
  } else {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const float4 c = ctl[ss * KT + sub + L * i];
      weights(c.x, c.y, c.z, &wp[0][i], &wm[0][i]);
    }
  }
  int count = 0, left = KT - 1;   // the last boundary is the next block's
  const auto step = [&](float w) {
    prev += w;
    if (left-- > 0) count += prev <= thr ? 1 : 0;
  };
#pragma unroll
  for (int i = 0; i < NP; ++i) in_lane_order<L>(wp[0][i], step);
#pragma unroll
  for (int i = 0; i < NP; ++i) in_lane_order<L>(wm[0][i], step);
  return ss * KT + from_first_quad<L>(count, sub);
}

}  // namespace capred
