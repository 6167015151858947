// rollout.hpp -- device side of Alg. 1 for one tile of particles of one human:
// (beta, g) draw from the belief, H Boltzmann-heading lattice steps held in
// registers, and per-step emplacement through an LDS-privatised histogram
// window flushed to the global uint32 grid with coalesced atomics.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace capred {

// Everything the rollout needs about one human (trivially copyable; passed by
// value to the single-human kernel and stored in device memory for batches).
struct RolloutDesc {
  int32_t N, H, K, B, G, nx, ny;
  int32_t S;                // speeds (controls u = s K + k, U = S K)
  int32_t s_last;           // last allowed speed
  uint32_t smask;           // allowed speeds of the prediction (bit s)
  int32_t X0, Y0;           // start on the lattice (grid frame)
  int32_t Rx, Ry;           // max |S_kx|, |S_ky|: reach per step, lattice units
  uint32_t human, cycle;
  int32_t bounds;           // bounds_rule: windows from the tile's true bounds
  int32_t shift;            // 1: subtract the largest exponent (large beta * step)
  int32_t sym;              // 1: S_{k+K/2} = -S_k for every k < K/2 (K even)
  HeadingTable T;           // lattice-unit steps (exact integers) and squared lengths (FP32)
  FarConst far;             // the filter of far particles' draws (one speed)
  float ibeta[CAP_MAX_B];   // 1 / (-beta q log2(e)), q = lattice pitch
  int32_t GX[CAP_MAX_G], GY[CAP_MAX_G];
  const double* belief;     // [G][B]
  uint32_t* counts;         // [H][ny][nx]
  uint32_t* offgrid;        // [H] or null
  uint8_t* trace_k;         // [N][H] or null
  int32_t* trace_pair;      // [N] or null
};

// When the tiles of a launch of so many particles take their true bounds (see
// rollout_tile_body).  Few particles: never; a step's latency is what counts and
// their atomics are cheap.  From one wave per CU on: where the particles share
// cells, as atomics on the same word wait for each other.  From eight waves per CU
// on: always, as the atomics' number is what counts.  60 steps of 2.4 cells on 200
// x 200 cells, never | always: flat belief (K = 16), 8000 particles 72 | 85 us, 30000
// 108 | 115, 2^17 342 | 351, 2^18 549 | 547, 600000 859 | 844; sharp (beta * step 3.6
// to 72), 8000 84 | 95, 30000 147 | 91, 2^17 578 | 132.  A plan of blocks of 512 threads
// and 24 KiB windows, 16 humans x 30000, K = 8: 906 | 809 us.
enum : int32_t { kBoundsNever = 0, kBoundsShared = 1, kBoundsAlways = 2 };

inline int32_t bounds_rule(int64_t particles, int cus) {
  if (particles >= (int64_t)512 * cus) return kBoundsAlways;
  return particles >= (int64_t)64 * cus ? kBoundsShared : kBoundsNever;
}

struct TileShared {
  double P[CAP_MAX_J];      // pair CDF (sequential FP64 prefix sums), then the sort's counts
  int2 S[CAP_MAX_K];        // lattice steps for the dynamic heading index (one speed)
  int2 goal[CAP_MAX_G];
  float ibeta[CAP_MAX_B];
  uint32_t off[2];          // off-grid counters of the two in-flight steps
  uint32_t ntouch[3];       // first-touched window words per step (rotating)
  int box[2][4];            // the tile's bounds: min x, min y, max x, max y (alternating)
  int last_pos;
};

__device__ __forceinline__ int64_t floor_shift16(int64_t v) { return v >> kLatticeShift; }

// Histogram window of a step: every particle was within [lx, hx] x [ly, hy]
// (lattice units) k steps ago, so its cell lies in [floor((lx - k Rx)/2^16),
// floor((hx + k Rx)/2^16)] (clipped to the grid).  Uniform across the block.
struct Window {
  int x0, y0, w, h;
};

__device__ __forceinline__ Window step_window_of(int32_t lx, int32_t ly, int32_t hx, int32_t hy,
                                                 int32_t Rx, int32_t Ry, int nx, int ny, int k) {
  // 64-bit only for the reach k * R (up to 2^36); the shifted bounds fit 32 bits,
  // so the clamps stay in scalar 32-bit arithmetic
  const int64_t rx = (int64_t)k * Rx, ry = (int64_t)k * Ry;
  int x0 = (int)floor_shift16((int64_t)lx - rx), x1 = (int)floor_shift16((int64_t)hx + rx);
  int y0 = (int)floor_shift16((int64_t)ly - ry), y1 = (int)floor_shift16((int64_t)hy + ry);
  x0 = max(x0, 0);
  y0 = max(y0, 0);
  x1 = min(x1, nx - 1);
  y1 = min(y1, ny - 1);
  Window win;
  win.x0 = x0;
  win.y0 = y0;
  win.w = x1 >= x0 ? x1 - x0 + 1 : 0;
  win.h = y1 >= y0 ? y1 - y0 + 1 : 0;
  return win;
}

// LDS words of a window: two 16-bit counters per word (a tile never holds 65536
// particles), rows padded to an even number of cells.
__device__ __forceinline__ int window_words(const Window& w) { return ((w.w + 1) >> 1) * w.h; }

// Reach window of step t for a start (X0, Y0) on the lattice.
__device__ __forceinline__ Window step_window_at(const RolloutDesc& d, int32_t X0, int32_t Y0,
                                                 int t) {
  return step_window_of(X0, Y0, X0, Y0, d.Rx, d.Ry, d.nx, d.ny, t);
}

// Least v of the wave's lanes, in lane 63.
__device__ __forceinline__ int wave_min63(int v) {
#define CAP_MIN_DPP(ctrl) v = min(v, __builtin_amdgcn_update_dpp(v, v, ctrl, 0xF, 0xF, false))
  CAP_MIN_DPP(0x111);   // row_shr 1, 2, 4, 8, then the rows below
  CAP_MIN_DPP(0x112);
  CAP_MIN_DPP(0x114);
  CAP_MIN_DPP(0x118);
  CAP_MIN_DPP(0x142);
  CAP_MIN_DPP(0x143);
#undef CAP_MIN_DPP
  return v;
}

__device__ __forceinline__ uint32_t pick_word(const uint4& w, int s) {
  return s == 0 ? w.x : (s == 1 ? w.y : (s == 2 ? w.z : w.w));
}

// LDS bytes of the histogram window of one block: two window buffers of
// `cap` words (two 16-bit cell counters per word) and two lists of the words
// first touched in a step (16-bit word indices, one per particle at most).
// A step whose window needs more than `cap` words (and at most 2 cap) uses
// both buffers as one and the first list.
__host__ __device__ constexpr size_t window_lds_bytes(int cap, int particles_per_tile) {
  return (size_t)2 * cap * sizeof(uint32_t) + (size_t)2 * particles_per_tile * sizeof(uint16_t);
}

// Deals a tile's particles to the lanes in the order of their (goal, beta)
// pairs (a counting sort in LDS; each wave takes P * 64 neighbours of the sorted
// order).  Results do not depend on which lane holds a particle, but the draws'
// far filter works on whole waves: sorted, the few particles that have reached
// their goal (or draw sharply) sit together instead of sending every wave the
// long way.  From kSortSteps steps on, where the sort's barriers are paid for.
// hist: CAP_MAX_J + 1 words of LDS; the lists: P * blockDim.x entries each.
constexpr int kSortSteps = 24;

template <int P>
__device__ __forceinline__ void sort_by_pair(int tid, int64_t first, int tile_n, int J,
                                             uint32_t* hist, uint16_t* lists, uint32_t* idx,
                                             int* pair, bool* act) {
  const int nthr = blockDim.x, lane = tid & 63;
  __syncthreads();   // hist may lie where the pair CDF was read
  for (int j = tid; j <= J; j += nthr) hist[j] = 0u;
  __syncthreads();
  uint32_t rank[P];
#pragma unroll
  for (int p = 0; p < P; ++p)   // lanes without a particle sort last, as pair J
    rank[p] = atomicAdd(hist + (act[p] ? pair[p] : J), 1u);
  __syncthreads();
  if (tid < 64) {   // exclusive prefix of the J + 1 counts, a run of bins per lane
    const int per = (J + 64) / 64, j0 = min(lane * per, J + 1), j1 = min(j0 + per, J + 1);
    uint32_t n = 0;
    for (int j = j0; j < j1; ++j) n += hist[j];
    uint32_t before = n;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t v = __shfl_up(before, o, 64);
      if (lane >= o) before += v;
    }
    before -= n;
    for (int j = j0; j < j1; ++j) {
      const uint32_t c = hist[j];
      hist[j] = before;
      before += c;
    }
  }
  __syncthreads();
  uint16_t* who = lists;
  uint16_t* what = lists + P * nthr;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const uint32_t at = hist[act[p] ? pair[p] : J] + rank[p];
    who[at] = (uint16_t)(p * nthr + tid);
    what[at] = (uint16_t)pair[p];
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int at = ((tid >> 6) * P + p) * 64 + lane;
    idx[p] = (uint32_t)first + who[at];
    pair[p] = what[at];
    act[p] = at < tile_n;
  }
  __syncthreads();   // the lists are the steps' from here on
}

// Processes particles [first, first + P * blockDim.x) of human d (clipped to N).
// win: window_lds_bytes(cap, P * blockDim.x) bytes of LDS, zero on entry and
// on exit (cap <= 65536).  A step's window is flushed from the list of words
// its particles touched first, so the flush costs one entry per occupied
// word, whatever the window's area.  Windows of up to cap words alternate
// between the two buffers, so that a step's binning overlaps the previous
// step's flush; windows of up to 2 cap words (and 2^16 words, the reach of a
// list entry) take both buffers and wait at one more barrier for the previous
// flush; larger windows bin with global atomics.
//
// A step's window is what the particles can have reached since their bounds were
// last known: the start's at first, and from the step on whose window would
// outgrow a buffer, the tile's true bounds, taken anew every fourth step while
// that is so (four wave reductions and a barrier).  A cloud spans a fraction of
// its reach (the 64-human scene at step 200: 6500 words of 29000), so that steps
// which went to global atomics one particle at a time, at the 2.7e10 a second
// that the device takes, stay in LDS: 16 humans x 10^5 particles x 100 steps of
// 2.4 cells on 256 x 256 cells, a cycle of 4.21 ms before and 2.42 after; eight
// humans of the 64-human scene 16.2 -> 15.9 ms.  Launches of few particles do so
// only where it pays (bounds_rule).
//
// MS (several speeds): draw_control over the S K controls; `ctl` is an LDS
// array of CAP_MAX_U float4 that receives (fx, fy, s2) of every control, read
// per lane for the block recomputation and the step (unused otherwise).
//
// PAIR: draw the particles two at a time (draw_headings with M = 2), for fixed K of
// at most 16 without the shifted exponent, where the two chains fit in the
// registers of four waves per SIMD without spilling.
//
// L > 1 (several speeds, K >= 2 L, not the shifted exponent): L neighbouring lanes
// share a particle (wide_control); all carry its state, the first of them
// emplaces it, and a tile holds P * blockDim.x / L particles.
template <int KT, int P, bool SHIFT, bool MS, bool PAIR, int L>
__device__ __forceinline__ void rollout_tile_body(const RolloutDesc& d, int64_t first,
                                                  uint32_t seed_lo, uint32_t seed_hi,
                                                  TileShared& sh, uint32_t* win, int cap,
                                                  float4* ctl) {
  // Opaque, so that a persistent block derives its lanes' addresses anew in each
  // tile: kept across the tiles they took the registers of the tile's own values
  // and spilled to scratch (38 registers at K = 16, P = 4), and a launch with
  // scratch starts later: the 16-human cycle 0.927 ms with, 0.905 without.
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int nthr = blockDim.x;
  const int J = d.G * d.B;
  // ---- shared tables
  // pair CDF: FP64 prefix sums in pair order, one thread; the other threads
  // bring the terms into LDS first, so that it does not wait for memory
  for (int j = tid; j < J; j += nthr) sh.P[j] = as_global(d.belief)[j];
  if constexpr (MS) {
    for (int u = tid; u < d.K * d.S; u += nthr)
      ctl[u] = make_float4(d.T.fx[u], d.T.fy[u], d.T.s2[u], 0.f);
  } else {
    for (int k = tid; k < d.K; k += nthr) sh.S[k] = make_int2((int)d.T.fx[k], (int)d.T.fy[k]);
  }
  for (int g = tid; g < d.G; g += nthr) sh.goal[g] = make_int2(d.GX[g], d.GY[g]);
  for (int b = tid; b < d.B; b += nthr) sh.ibeta[b] = d.ibeta[b];
  __syncthreads();
  if (tid == 0) {
    double acc = 0.0;
    int last = 0;
#pragma unroll 8
    for (int j = 0; j < J; ++j) {
      const double b = sh.P[j];
      acc += b;
      sh.P[j] = acc;
      if (b > 0.0) last = j;
    }
    sh.last_pos = last;
    sh.off[0] = 0u;
    sh.off[1] = 0u;
    sh.ntouch[0] = sh.ntouch[1] = sh.ntouch[2] = 0u;
  }
  if (tid < 8) sh.box[tid >> 2][tid & 3] = INT_MAX;
  __syncthreads();

  // ---- per-particle (beta, g) draw, held for the whole horizon
  constexpr bool kFar = !SHIFT && !MS && (KT == 8 || KT == 16 || KT == 32);
  const uint32_t c3_pair = 2u * d.cycle, c3_head = 2u * d.cycle + 1u;
  const int per = nthr / L;                                               // particles at a time
  const int tile_n = (int)min((int64_t)P * per, (int64_t)d.N - first);    // particles of the tile
  uint32_t idx[P];
  int pair[P];
  bool act[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int local = p * per + tid / L;
    idx[p] = (uint32_t)first + (uint32_t)local;
    act[p] = local < tile_n;
    pair[p] = 0;
    if (act[p]) {
      const uint4 w = philox10(idx[p], 0u, d.human, c3_pair, seed_lo, seed_hi);
      const double u = uniform24d(w.x);
      int lo = 0, hi = J;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (sh.P[mid] > u) hi = mid;
        else lo = mid + 1;
      }
      pair[p] = lo < J ? lo : sh.last_pos;
      if (d.trace_pair && tid % L == 0) as_global(d.trace_pair)[idx[p]] = pair[p];
    }
  }
  uint16_t* lists = reinterpret_cast<uint16_t*>(win + 2 * cap);
  if (kFar && d.H >= kSortSteps)
    sort_by_pair<P>(tid, first, tile_n, J, reinterpret_cast<uint32_t*>(sh.P), lists, idx, pair,
                    act);
  int32_t X[P], Y[P], GXp[P], GYp[P];
  float ib[P], nbs[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    X[p] = d.X0;
    Y[p] = d.Y0;
    // lanes past the last particle: far from a goal, every heading alike
    GXp[p] = (int32_t)((uint32_t)d.X0 - (1u << 28));
    GYp[p] = d.Y0;
    ib[p] = 1.f;
    nbs[p] = 0.f;
    if (act[p]) {
      const int g = pair[p] / d.B, b = pair[p] - g * d.B;
      GXp[p] = sh.goal[g].x;
      GYp[p] = sh.goal[g].y;
      ib[p] = sh.ibeta[b];
      nbs[p] = -4.f * d.far.s4 / ib[p];
    }
    act[p] = act[p] && tid % L == 0;   // from here on: emplaces a particle
  }
  WideRows<(L > 1 ? KT : 2), L> rows;
  if constexpr (L > 1) rows.load(ctl, d.S, tid % L);
  // The descriptor's fields that every step reads, in scalar registers for the
  // whole tile: it lies in memory that the loop's stores could alias, so each
  // use would be a load and a wait.  Several speeds by one lane read them from
  // there: their controls' table fills the scalar registers, and what is held
  // besides goes to vector-register lanes, one VALU access each (K = 16: 55 more a
  // step; 16 humans x 30000 particles of 6 x 16 controls, 30 steps: 782 us read, 823
  // held).
  constexpr bool kRead = MS && L == 1;
  using Int = std::conditional_t<kRead, const int32_t&, const int32_t>;
  Int H = d.H, nx = d.nx, ny = d.ny, Rx = d.Rx, Ry = d.Ry, S = d.S, s_last = d.s_last;
  std::conditional_t<kRead, const uint32_t&, const uint32_t> human = d.human, smask = d.smask;
  std::conditional_t<kRead, uint32_t* const&, uint32_t* const> counts = d.counts;
  std::conditional_t<kRead, uint8_t* const&, uint8_t* const> trace_k = d.trace_k;
  const FarConst fc = d.far;
  const size_t plane = kRead ? 0 : (size_t)nx * (size_t)ny;   // (read: each step's own)
  uint4 rw[P];
  const int list_cap = P * nthr;
  int m3 = 1;  // t mod 3
  // after step t_box the particles lie in [lox, hix] x [loy, hiy]
  int lox = d.X0, loy = d.Y0, hix = lox, hiy = loy, t_box = 0, box_buf = 0;
  for (int t = 1; t <= H; ++t, m3 = (m3 == 2 ? 0 : m3 + 1)) {
    const int s = (t - 1) & 3;
    if (s == 0) {
      // The round keys (key + r * Weyl constant) are derived from the seed here,
      // by scalar adds in every block, rather than held across the loop: kept,
      // they would pin 20 scalar registers that the step's other uniform values
      // need (the overflow goes to vector-register lanes, one VALU access each).
      uint32_t klo = seed_lo, khi = seed_hi;
      asm volatile("" : "+s"(klo), "+s"(khi));
#pragma unroll
      for (int p = 0; p < P; ++p)
        rw[p] = philox10(idx[p], (uint32_t)((t - 1) >> 2), human, c3_head, klo, khi);
      // The windows outgrow the buffer within these four steps: take the
      // particles' true bounds, or (kBoundsShared) only if the words that the last
      // step touched held two particles or more on average; its count is cleared
      // after this step's barrier, and 0 if that step used global atomics.  (The rule
      // is read here and off the straight path: held in a register, eight humans of
      // 2^20 particles, K = 32, took 15.97 ms instead of 15.55.)
      bool take = t > 1 && window_words(step_window_of(lox, loy, hix, hiy, Rx, Ry, nx, ny,
                                                       min(t + 3, H) - t_box)) > cap;
      if (take && __builtin_expect(d.bounds != kBoundsAlways, 0)) {
        const int touched = __builtin_amdgcn_readfirstlane(sh.ntouch[m3 == 0 ? 2 : m3 - 1]);
        take = d.bounds == kBoundsShared && touched > 0 && 2 * touched <= tile_n;
      }
      if (take) {
        int b[4] = {INT_MAX, INT_MAX, INT_MAX, INT_MAX};
#pragma unroll
        for (int p = 0; p < P; ++p)
          if (act[p]) {
            b[0] = min(b[0], X[p]);
            b[1] = min(b[1], Y[p]);
            b[2] = min(b[2], ~X[p]);
            b[3] = min(b[3], ~Y[p]);
          }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          b[i] = wave_min63(b[i]);
          if ((tid & 63) == 63) atomicMin(&sh.box[box_buf][i], b[i]);
        }
        __syncthreads();
        lox = __builtin_amdgcn_readfirstlane(sh.box[box_buf][0]);
        loy = __builtin_amdgcn_readfirstlane(sh.box[box_buf][1]);
        hix = ~__builtin_amdgcn_readfirstlane(sh.box[box_buf][2]);
        hiy = ~__builtin_amdgcn_readfirstlane(sh.box[box_buf][3]);
        t_box = t - 1;
        // the other one was read before an earlier step's barrier and is next
        // taken after a later one's
        box_buf ^= 1;
        if (tid < 4) sh.box[box_buf][tid] = INT_MAX;
      }
    }
    const Window wd = step_window_of(lox, loy, hix, hiy, Rx, Ry, nx, ny, t - t_box);
    const int half_w = (wd.w + 1) >> 1;
    const int words = window_words(wd);
    const bool single = words > cap && words <= 2 * cap && words <= 65536;
    const bool lds_mode = words <= cap || single;
    uint32_t* buf = single ? win : win + (t & 1) * cap;
    uint16_t* list = single ? lists : lists + (t & 1) * list_cap;
    // both buffers: the previous step's flush (of either buffer) must be over
    if (single) __syncthreads();
    uint32_t* grid_t = counts + (size_t)(t - 1) * (kRead ? (size_t)nx * (size_t)ny : plane);
    // Draws of all P particles first, then their emplacement: the draws are
    // independent dependency chains (transcendental latency), which the
    // scheduler can interleave only while no branch separates them.  Each
    // particle's step word is rw[p].x; the remaining words move down, so the
    // word is picked without branching on the step's phase.
    int kk[P];
    if constexpr (MS) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const float u = uniform24f(rw[p].x);
        rw[p] = make_uint4(rw[p].y, rw[p].z, rw[p].w, 0u);
        const float ax = (float)(X[p] - GXp[p]), ay = (float)(Y[p] - GYp[p]);
        int k;
        if constexpr (L > 1)
          k = wide_control<KT, L>(ax, ay, ib[p], u, S, smask, s_last, rows, ctl, tid % L);
        else
          k = draw_control<KT, SHIFT>(ax, ay, ib[p], u, d.T, S, smask, s_last, ctl);
        const float4 c = ctl[k];
        X[p] += (int32_t)c.x;
        Y[p] += (int32_t)c.y;
        kk[p] = k;
      }
    } else {
      // computed for inactive lanes too (harmless state), so that the draws
      // stay in few basic blocks; only emplacement is predicated
      constexpr int M = PAIR ? 2 : 1;
      static_assert(P % M == 0, "paired draws need an even P");
#pragma unroll
      for (int p = 0; p < P; p += M) {
        float ax[M], ay[M], ibm[M], um[M];
        int ko[M];
#pragma unroll
        for (int m = 0; m < M; ++m) {
          ax[m] = (float)(X[p + m] - GXp[p + m]);
          ay[m] = (float)(Y[p + m] - GYp[p + m]);
          ibm[m] = ib[p + m];
          um[m] = uniform24f(rw[p + m].x);
          rw[p + m] = make_uint4(rw[p + m].y, rw[p + m].z, rw[p + m].w, 0u);
        }
        bool sure = false;   // uniform in the wave
        if constexpr (kFar) {
          float D2[M];
          bool far = true;
#pragma unroll
          for (int m = 0; m < M; ++m) {
            D2[m] = fmaf(ax[m], ax[m], ay[m] * ay[m]);
            far = far && D2[m] >= fc.d2;
          }
          if (__all(far))
            sure = __all(far_headings<KT, M>(ax, ay, D2, nbs + p, um, fc, ko));
        }
        if (!sure) {
          // keeps the table's loads (48 scalars at K = 16) out of the common path
          if constexpr (kFar) asm volatile("" ::: "memory");
          if constexpr (PAIR)
            draw_headings<KT, SHIFT, 2>(ax, ay, ibm, um, d.T, ko);
          else
            ko[0] = draw_heading<KT, SHIFT>(ax[0], ay[0], ibm[0], um[0], d.T, d.K);
        }
#pragma unroll
        for (int m = 0; m < M; ++m) {
          const int2 st = sh.S[ko[m]];
          X[p + m] += st.x;
          Y[p + m] += st.y;
          kk[p + m] = ko[m];
        }
      }
    }
    // The draws' results are fixed here (an empty asm that reads and writes
    // them), so that the compiler does not sink each draw into the branchy
    // emplacement of its particle below.
#pragma unroll
    for (int p = 0; p < P; ++p) asm volatile("" : "+v"(X[p]), "+v"(Y[p]), "+v"(kk[p]));
    if (trace_k) {
#pragma unroll
      for (int p = 0; p < P; ++p)
        if (act[p]) as_global(trace_k)[(size_t)idx[p] * H + (t - 1)] = (uint8_t)kk[p];
    }
    uint32_t off = 0;   // off-grid particles of the wave
    if (lds_mode) {
      // The P adds go out before any result is waited for, and the wave appends
      // the words that its adds turned non-empty with one addition to the
      // list's length, so that a step has two LDS round trips instead of 2 P.
      // The particle's cell lies in the unclipped reach window, so it is on the
      // grid exactly when it lies in the clipped window.
      uint32_t widx[P], old[P];
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const unsigned lx = (unsigned)((X[p] >> kLatticeShift) - wd.x0),
                       ly = (unsigned)((Y[p] >> kLatticeShift) - wd.y0);
        const bool in = act[p] && lx < (unsigned)wd.w && ly < (unsigned)wd.h;
        widx[p] = __umul24(ly, (unsigned)half_w) + (lx >> 1);  // both below 2^24
        old[p] = 1u;
        if (in) old[p] = atomicAdd(buf + widx[p], 1u << ((lx & 1u) << 4));
        off += __popcll(__ballot(act[p] && !in));
      }
#pragma unroll
      for (int p = 0; p < P; ++p) asm volatile("" : "+v"(old[p]));
      uint64_t fresh[P];
      uint32_t n_fresh = 0;
#pragma unroll
      for (int p = 0; p < P; ++p) {
        fresh[p] = __ballot(old[p] == 0u);
        n_fresh += __popcll(fresh[p]);
      }
      if (n_fresh) {
        uint32_t at = 0;
        if ((tid & 63) == 0) at = atomicAdd(&sh.ntouch[m3], n_fresh);
        at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int p = 0; p < P; ++p) {
          const uint32_t below = __builtin_amdgcn_mbcnt_hi(
              (uint32_t)(fresh[p] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)fresh[p], 0u));
          if (old[p] == 0u) list[at + below] = (uint16_t)widx[p];
          at += __popcll(fresh[p]);
        }
      }
    } else {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const int cx = X[p] >> kLatticeShift, cy = Y[p] >> kLatticeShift;
        const bool in = act[p] && (unsigned)cx < (unsigned)nx && (unsigned)cy < (unsigned)ny;
        if (in) global_add(grid_t + (size_t)cy * nx + cx, 1u);
        off += __popcll(__ballot(act[p] && !in));
      }
    }
    if (off && (tid & 63) == 0) atomicAdd(&sh.off[t & 1], off);
    __syncthreads();
    // ---- flush the touched words of step t's window, clear them
    if (lds_mode) {
      // Word w of the window is row ry = floor(w / half_w), cells 2 rx and 2 rx + 1
      // with rx = w - ry half_w.  ry = trunc((w + 1/2) * fl(1/half_w)) exactly:
      // (w + 1/2) / half_w lies at least 1/(2 half_w) from an integer, while the
      // two roundings (reciprocal within 1 ulp, product) move it by at most
      // 2^-22 (w + 1/2) / half_w <= 2^-22 * 65536 / half_w, since w < 2^16.
      const float rhw = fast_rcp((float)half_w), hrhw = 0.5f * rhw;
      // byte offset of the window's first cell within the step's plane (< 2^30)
      const uint32_t base4 = 4u * ((uint32_t)wd.y0 * (uint32_t)nx + (uint32_t)wd.x0);
      const uint32_t nx4 = 4u * (uint32_t)nx;
      char* gbase = reinterpret_cast<char*>(grid_t);
      const uint32_t nt = sh.ntouch[m3];
      for (uint32_t i = tid; i < nt; i += nthr) {
        const uint32_t w = list[i];
        const uint32_t v = buf[w];
        buf[w] = 0u;
        const uint32_t ry = (uint32_t)fmaf((float)w, rhw, hrhw);
        const uint32_t rx = w - __umul24(ry, (uint32_t)half_w);
        const uint32_t off4 = __umul24(ry, nx4) + base4 + (rx << 3);
        uint32_t* g = reinterpret_cast<uint32_t*>(gbase + off4);
        const uint32_t lo = v & 0xFFFFu, hi = v >> 16;
        if (lo) global_add(g, lo);
        if (hi) global_add(g + 1, hi);
      }
    }
    if (tid == 0) {
      const uint32_t v = sh.off[t & 1];
      if (v && d.offgrid) global_add(d.offgrid + (t - 1), v);
      sh.off[t & 1] = 0u;
      // the list counter of step t-1 was read before this step's barrier and
      // is next appended to at step t+2, after the next barrier
      sh.ntouch[m3 == 0 ? 2 : m3 - 1] = 0u;
    }
  }
  __syncthreads();
}

// A tile of one human.  The shifted exponent is a property of the human
// (d.shift: beta * step too large for the unshifted exp2), not of the launch:
// a launch compiled with SHIFT also carries the unshifted body and takes it,
// uniformly per tile, for humans that do not need the shift, so that their
// draws are the same bits whichever humans share the launch.
template <int KT, int P, bool SHIFT, bool MS, int L = 1>
__device__ __forceinline__ void rollout_tile(const RolloutDesc& d, int64_t first, uint32_t seed_lo,
                                             uint32_t seed_hi, TileShared& sh, uint32_t* win,
                                             int cap, float4* ctl) {
  static_assert(L == 1 || (MS && !SHIFT), "the wide draw has no shifted form");
  if constexpr (SHIFT) {
    if (!d.shift) {
      rollout_tile_body<KT, P, false, MS, false, 1>(d, first, seed_lo, seed_hi, sh, win, cap, ctl);
      return;
    }
  }
  constexpr bool kPair = !SHIFT && !MS && KT > 0 && KT <= 16 && P % 2 == 0;
  rollout_tile_body<KT, P, SHIFT, MS, kPair, L>(d, first, seed_lo, seed_hi, sh, win, cap, ctl);
}

}  // namespace capred
