// Iterative 1D Jacobi stencil: the time loop inside one persistent kernel
// versus one kernel launch per step, and many steps per launch (gfx950).
//
// Section VII-B of Zhang et al. points out a benefit of grid barriers that
// the reduction does not show: a persistent kernel that holds the time loop
// of an iterative stencil keeps its data in on-chip memory across the
// barriers, where one launch per step (the implicit barrier) must stream
// the whole array through HBM or the caches every step.
//
// The step is u'[i] = u[i] + r ((u[i-1] + u[i+1]) - 2 u[i]) for
// 1 <= i <= n-2, with u[0] and u[n-1] fixed, each operation one binary32
// operation in that order (no contraction but one that rounds the same), so
// every form reproduces the step-by-step definition bit for bit.
//
//   * relaunch:   k_jacobi_step per step, ping-pong between u and the
//                 caller's scratch array;
//   * persistent: workgroup g owns the block [g m, (g+1) m) and holds it,
//                 with a halo of K values on each side, in its threads'
//                 registers.  It runs K steps on the shrinking valid range
//                 (redundantly recomputing the halo, so neighbours need no
//                 exchange inside the K steps), then publishes its first and
//                 last K values (device-scope atomic stores), meets the other
//                 workgroups at a grid barrier that neither writes back nor
//                 invalidates an L2, and reads its neighbours' values into
//                 its halo (device-scope atomic loads).  One barrier per K
//                 steps; HBM is touched only at the start, at the end and for
//                 the 2 K boundary values per workgroup and barrier.
//   * blocked:    k_jacobi_tile advances windows held in single wavefronts
//                 by up to hundreds of steps per launch, with no exchange
//                 inside a launch; the form the library chooses by itself.
#include <algorithm>
#include <type_traits>

#include "device_prims.h"
#include "internal.h"
#include "stencil_plan.h"

namespace redsum {

// One step at an interior point, in the method's operation order.
__device__ __forceinline__ float jacobi_point(float left, float centre, float right, float r) {
#pragma clang fp contract(off)
  const float neighbours = left + right;
  const float twice = 2.0f * centre;
  return centre + r * (neighbours - twice);
}

__global__ __launch_bounds__(1024) void k_jacobi_step(const float* __restrict__ u, float* __restrict__ v, int64_t n,
                                                      float r) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const float c = u[i];
    v[i] = (i == 0 || i == n - 1) ? c : jacobi_point(u[i - 1], c, u[i + 1], r);
  }
}

__global__ __launch_bounds__(1024) void k_copy_f32(const float* __restrict__ src, float* __restrict__ dst, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

struct StencilArgs {
  float* u;        // values, in and out
  float* scratch;  // n values: boundary publication, alternating with u
  int64_t n;
  int64_t m;       // block length per workgroup
  int steps;
  int k;           // steps per grid barrier = halo width, 1 <= k <= m
  float r;
  BarrierWords* words;
  unsigned spin_limit;
  unsigned bar_groups;
};

// The window of a workgroup (its block and k-wide halos, at most
// kWindowMax values) is held in registers: thread t owns the VPT
// consecutive window values from VPT t on.  A step reads the two values
// beside a thread's run from its neighbours, through LDS: each thread
// stores its first and last value to one of two edge buffers (alternating
// by step), meets the others at the step's only workgroup barrier, and
// reads the neighbours' edges.  A buffer is written again two steps later,
// after the next barrier, which every thread reaches after its reads.  The
// kernel is built for VPT = 2, 4, 8, 16 and 32.
constexpr int kWindowMax = 16384;

// Widest halo (steps per grid barrier) the library picks by itself.
constexpr int64_t kAutoHalo = 128;

template <int VPT>
__global__ __launch_bounds__(1024) void k_jacobi_persistent(StencilArgs a) {
  static_assert(VPT >= 2, "a run has a first and a last value");
  unsigned gen = grid_barrier_gen(a.words);  // thread 0: the barrier generation of this launch
  extern __shared__ float edge[];            // [2 buffers][first, last][blockDim.x]
  const int64_t n = a.n;
  const int k = a.k;
  const int64_t lo = (int64_t)blockIdx.x * a.m;
  const int64_t hi = std::min(lo + a.m, n);
  const int blen = (int)(hi - lo);
  const int len = blen + 2 * k;
  const int64_t base = lo - k;  // window value j is element base + j
  const int tid = threadIdx.x;
  const int bs = blockDim.x;
  const int j0 = VPT * tid;     // this thread's window values j0 .. j0 + VPT - 1

  float x[VPT];
#pragma unroll
  for (int i = 0; i < VPT; ++i) {
    const int64_t e = base + j0 + i;
    x[i] = (j0 + i < len && e >= 0 && e < n) ? a.u[e] : 0.0f;
  }

  // Window positions of the array's end points, which never change (-1 or
  // len when the window does not hold them).
  const int jz = (int)std::max<int64_t>(std::min<int64_t>(-base, len), -1);
  const int jn = (int)std::max<int64_t>(std::min<int64_t>(n - 1 - base, len), -1);
  const bool holds_end = (jz >= j0 && jz < j0 + VPT) || (jn >= j0 && jn < j0 + VPT);

  int sync = 0, buf = 0;
  for (int step = 0; step < a.steps;) {
    const int kk = std::min(k, a.steps - step);
    for (int s = 1; s <= kk; ++s) {
      // After step s only the window values of the elements
      // [lo - k + s, hi + k - s) are valid: the range shrinks by one value
      // on each side per step, so no valid value depends on one outside it.
      // The values outside (the halo being used up, and positions past the
      // array's ends) are updated too and never read for a valid one; the
      // halo is reloaded at the next exchange.  Only the array's end points
      // keep their value.
      float* eb = edge + 2 * bs * buf;
      eb[tid] = x[0];
      eb[bs + tid] = x[VPT - 1];
      __syncthreads();
      // Window value j0 - 1 is the left neighbour's last, j0 + VPT the right
      // neighbour's first (thread 0 and the last thread read a value that
      // only feeds positions outside the valid range).
      const float left = tid > 0 ? eb[bs + tid - 1] : 0.0f;
      const float right = tid + 1 < bs ? eb[tid + 1] : 0.0f;
      float y[VPT];
      y[0] = jacobi_point(left, x[0], x[1], a.r);
#pragma unroll
      for (int i = 1; i < VPT - 1; ++i) y[i] = jacobi_point(x[i - 1], x[i], x[i + 1], a.r);
      y[VPT - 1] = jacobi_point(x[VPT - 2], x[VPT - 1], right, a.r);
      if (!holds_end) {
#pragma unroll
        for (int i = 0; i < VPT; ++i) x[i] = y[i];
      } else {  // the run that holds element 0 or n - 1
#pragma unroll
        for (int i = 0; i < VPT; ++i) x[i] = (j0 + i == jz || j0 + i == jn) ? x[i] : y[i];
      }
      buf ^= 1;
    }
    step += kk;
    if (step < a.steps) {
      // Publish the first and last k values of the block (time `step`) to
      // the buffer of this barrier's parity, meet, read the neighbours'.
      // The first publication goes to scratch: u is still being read for
      // the initial halos.  The edges cross the barrier as device-scope
      // atomic stores and loads, so the barrier neither writes back nor
      // invalidates an L2.
      float* pub = (sync & 1) ? a.u : a.scratch;
      const int w = std::min(k, blen);
#pragma unroll
      for (int i = 0; i < VPT; ++i) {
        const int j = j0 + i;
        if ((j >= k && j < k + w) || (j >= k + blen - w && j < k + blen)) publish(&pub[base + j], x[i]);
      }
      grid_barrier_published(a.words, gridDim.x, a.bar_groups, a.spin_limit, gen);
#pragma unroll
      for (int i = 0; i < VPT; ++i) {
        const int j = j0 + i;
        const int64_t e = base + j;
        // left halo: the left neighbour's last k values; right halo: the
        // right neighbour's first k values
        if ((j < k && e >= 0) || (j >= k + blen && j < len && e < n)) x[i] = load_published(&pub[e]);
      }
      ++sync;
    }
  }
  // Neighbours read u for their initial halos and, at odd exchanges, as the
  // publication buffer: the block is written back only once every
  // workgroup is past its last read of u (each workgroup's loads complete
  // before it arrives; no data crosses this barrier).
  grid_barrier_published(a.words, gridDim.x, a.bar_groups, a.spin_limit, gen);
#pragma unroll
  for (int i = 0; i < VPT; ++i) {
    const int j = j0 + i;
    if (j >= k && j < k + blen) a.u[base + j] = x[i];
  }
}

// ---------------------------------------------------------------------------
// Blocked steps: many steps per launch on windows that live in one
// wavefront's registers.
//
// One launch per step is bound by the 8 bytes per value that it moves, and
// by the launch below about a million values; the persistent form by the
// exchange through LDS and the workgroup barrier of every step.  Here a
// wavefront loads a window of 64 V consecutive interior values and advances
// it k steps with no exchange at all: lane l holds the V values from V l on,
// the two values beside its run come from the adjacent lanes by DPP wave
// shifts that fold into the additions that use them, and the k outermost
// values on each side, which go stale one per step, are recomputed by the
// neighbouring windows.  The kernel boundary is the only synchronization, so
// nothing has to be co-resident and any length runs.  What bounds it is VALU
// issue: 4 operations per value and step (5 in the method, see FMA below)
// at 2.6 to 3.2 cycles each with two or more wavefronts per SIMD, 4.6 to 4.8
// with one (by the counters: 4 M values, 200 steps, four wavefronts: 31,070
// VALU instructions per SIMD in 81,000 cycles, waits for memory 14 % of the
// wavefronts' time; 64 K values: 1368 per wavefront in 6500 cycles).
// ---------------------------------------------------------------------------

// One step on the window.  The neighbour sums run one value ahead of the
// update, so it is in place without moves.
//   FMA   the doubling and the subtraction are one fused operation, which
//         rounds the same, since 2 c is exact, unless 2 c overflows;
//   ENDS  the window may lie at an end of the interior: `left` holds the
//         array's first value in lane 0 and `right` its last one in lane 63,
//         lanes that the wave shifts do not write.
template <int V, bool FMA, bool ENDS>
__device__ __forceinline__ void window_step(float (&x)[V], float r, float& left, float& right) {
#pragma clang fp contract(off)
  float nb, nb_last;
  if constexpr (ENDS) {
    left = dpp_update<kWaveShr1>(left, x[V - 1]);
    right = dpp_update<kWaveShl1>(right, x[0]);
    nb = left + x[1];
    nb_last = x[V - 2] + right;
  } else {
    nb = dpp_move<kWaveShr1, 0xF, 0xF>(x[V - 1]) + x[1];
    nb_last = x[V - 2] + dpp_move<kWaveShl1, 0xF, 0xF>(x[0]);
  }
  // In groups of four values, with the compiler kept from moving operations
  // between a group's four stages: each operation's operands are then at
  // least four operations old (a result takes two issue slots), which the
  // compiler's own order does not keep to (24 M values, 64 steps with
  // V = 16: 130 us against 177).  Windows of up to 8 values per lane run
  // one wavefront per SIMD and are left to the compiler (64 K values, V = 4:
  // 69 us against 74 for 1000 steps).
  constexpr int G = V > 8 ? 4 : V;
  auto fence = [] {
    if constexpr (V > 8) __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int g = 0; g < V; g += G) {
    float d[G];
    d[0] = nb;
#pragma unroll
    for (int i = g + 1; i < g + G; ++i) d[i - g] = i + 1 < V ? x[i - 1] + x[i + 1] : nb_last;
    if (g + G < V) nb = x[g + G - 1] + x[g + G + 1];
    fence();
#pragma unroll
    for (int i = g; i < g + G; ++i) {
      if constexpr (FMA)
        d[i - g] = __builtin_fmaf(-2.0f, x[i], d[i - g]);
      else
        d[i - g] = d[i - g] - 2.0f * x[i];
    }
    fence();
#pragma unroll
    for (int i = g; i < g + G; ++i) d[i - g] = r * d[i - g];
    fence();
#pragma unroll
    for (int i = g; i < g + G; ++i) x[i] = x[i] + d[i - g];
    fence();
  }
}

// `steps` steps on the window.  The fused form rounds as the method's five
// operations do while no doubling overflows: for 0 <= r <= 1/2 a step
// enlarges the largest magnitude by rounding only (by less than 2^-20 of
// it), so from below 2^100 none overflows in 2^24 steps.  Other values (NaN
// and infinities among them) take the five operations.
template <int V>
__device__ __forceinline__ void window_steps(float (&x)[V], int steps, float r, float left, float right, bool ends) {
  bool small = __builtin_fabsf(left) < 0x1p100f && __builtin_fabsf(right) < 0x1p100f;
#pragma unroll
  for (int i = 0; i < V; ++i) small = small && __builtin_fabsf(x[i]) < 0x1p100f;  // false for NaN
  // r in a vector register: with two or more wavefronts per SIMD a
  // multiplication by a scalar register issues at half the rate (4.1 against
  // 2.1 cycles).
  const bool fma = r >= 0.0f && r <= 0.5f && steps <= (1 << 24) && __ballot(!small) == 0;
  asm volatile("" : "+v"(r));
  auto loop = [&](auto f, auto e) {
    constexpr bool F = decltype(f)::value, EN = decltype(e)::value;
    constexpr int U = 4;  // steps per loop iteration
    int s = 0;
    for (; s + U <= steps; s += U) {
#pragma unroll
      for (int q = 0; q < U; ++q) window_step<V, F, EN>(x, r, left, right);
    }
    for (; s < steps; ++s) window_step<V, F, EN>(x, r, left, right);
  };
  if (fma && !ends)
    loop(std::true_type{}, std::false_type{});
  else if (fma)
    loop(std::true_type{}, std::true_type{});
  else
    loop(std::false_type{}, std::true_type{});
}

// Lane l's V values from p + V l on, by the widest loads that the array's
// alignment (4 bytes) and V allow.
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
typedef float v2f_any __attribute__((ext_vector_type(2), aligned(4)));

template <int V>
__device__ __forceinline__ void load_window(float (&x)[V], const float* p) {
  if constexpr (V % 4 == 0) {
#pragma unroll
    for (int i = 0; i < V; i += 4) {
      const v4f_any v = *reinterpret_cast<const v4f_any*>(p + i);
      x[i] = v.x, x[i + 1] = v.y, x[i + 2] = v.z, x[i + 3] = v.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < V; i += 2) {
      const v2f_any v = *reinterpret_cast<const v2f_any*>(p + i);
      x[i] = v.x, x[i + 1] = v.y;
    }
  }
}

// Stores the values of the lane's run [j0, j0 + V) that lie in [a, b).
template <int V>
__device__ __forceinline__ void store_window(const float (&x)[V], float* p, int j0, int a, int b) {
  constexpr int C = V % 4 == 0 ? 4 : 2;
#pragma unroll
  for (int i = 0; i < V; i += C) {
    const int j = j0 + i;
    if (j >= a && j + C <= b) {
      if constexpr (C == 4)
        *reinterpret_cast<v4f_any*>(p + i) = v4f_any{x[i], x[i + 1], x[i + 2], x[i + 3]};
      else
        *reinterpret_cast<v2f_any*>(p + i) = v2f_any{x[i], x[i + 1]};
    } else if (j + C > a && j < b) {
#pragma unroll
      for (int e = 0; e < C; ++e)
        if (j + e >= a && j + e < b) p[i + e] = x[i + e];
    }
  }
}

// Wavefront w advances the interior values [w m, (w + 1) m) (element 1 + i
// of the array is interior value i, of N) by `steps` <= k steps from src to
// dst.  Its window of 64 V values starts k before them, moved inward where
// it would leave the interior (N >= 64 V).
template <int V>
__global__ __launch_bounds__(kTileWG) void k_jacobi_tile(const float* __restrict__ src, float* __restrict__ dst,
                                                         int64_t N, int m, int k, int steps, float r) {
  constexpr int W = kWave * V;
  const int64_t w = (int64_t)blockIdx.x * (kTileWG / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t lo = w * m;
  if (lo >= N) return;
  const int64_t hi = std::min(lo + m, N);
  const int64_t base = std::min(std::max<int64_t>(lo - k, 0), N - W);
  const int lane = __lane_id();
  const int j0 = V * lane;
  float x[V];
  load_window<V>(x, src + 1 + base + j0);
  const float left = src[base], right = src[1 + base + W];
  window_steps<V>(x, steps, r, left, right, base == 0 || base + W == N);
  store_window<V>(x, dst + 1 + base + j0, j0, (int)(lo - base), (int)(hi - base));
  if (lo == 0 && lane == 0) dst[0] = left;
  if (hi == N && lane == 0) dst[N + 1] = right;
}

// The whole interior (N <= 64 V values) in one wavefront, in place: the
// values at and past its end keep what they hold.
template <int V>
__global__ __launch_bounds__(kWave) void k_jacobi_one_window(float* u, int N, int steps, float r) {
  const int j0 = V * (int)__lane_id();
  float x[V];
#pragma unroll
  for (int i = 0; i < V; ++i) x[i] = j0 + i <= N ? u[1 + j0 + i] : 0.0f;  // position N: the array's last value
  float left = u[0], right = u[N + 1];
  for (int s = 0; s < steps; ++s) {
    float y[V];
#pragma unroll
    for (int i = 0; i < V; ++i) y[i] = x[i];
    window_step<V, false, true>(y, r, left, right);
#pragma unroll
    for (int i = 0; i < V; ++i) x[i] = j0 + i < N ? y[i] : x[i];
  }
#pragma unroll
  for (int i = 0; i < V; ++i)
    if (j0 + i < N) u[1 + j0 + i] = x[i];
}

namespace {

const void* persistent_kernel(int vpt) {
  switch (vpt) {
    case 2: return reinterpret_cast<const void*>(&k_jacobi_persistent<2>);
    case 4: return reinterpret_cast<const void*>(&k_jacobi_persistent<4>);
    case 8: return reinterpret_cast<const void*>(&k_jacobi_persistent<8>);
    case 16: return reinterpret_cast<const void*>(&k_jacobi_persistent<16>);
    default: return reinterpret_cast<const void*>(&k_jacobi_persistent<32>);
  }
}

// LDS of the two edge buffers of a workgroup of wg threads.
size_t edge_bytes(int wg) { return (size_t)4 * wg * sizeof(float); }

// Workgroups of the kernel for `vpt` values per thread that all CUs hold at
// once with wg threads each.
int stencil_coresident(int vpt, int wg, const DeviceInfo& dev, int* n_wg) {
  int per_cu = 0;
  RED_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, persistent_kernel(vpt), wg, edge_bytes(wg)));
  *n_wg = per_cu * dev.cus;
  return RED_OK;
}

// Kernels of the blocked-step shapes that plan_tiles() chooses from.
const void* tile_kernel(int v) {
  switch (v) {
    case 2: return reinterpret_cast<const void*>(&k_jacobi_tile<2>);
    case 4: return reinterpret_cast<const void*>(&k_jacobi_tile<4>);
    case 6: return reinterpret_cast<const void*>(&k_jacobi_tile<6>);
    case 8: return reinterpret_cast<const void*>(&k_jacobi_tile<8>);
    case 12: return reinterpret_cast<const void*>(&k_jacobi_tile<12>);
    case 16: return reinterpret_cast<const void*>(&k_jacobi_tile<16>);
    case 20: return reinterpret_cast<const void*>(&k_jacobi_tile<20>);
    case 24: return reinterpret_cast<const void*>(&k_jacobi_tile<24>);
    case 28: return reinterpret_cast<const void*>(&k_jacobi_tile<28>);
    default: return reinterpret_cast<const void*>(&k_jacobi_tile<36>);
  }
}

const void* one_window_kernel(int v) {
  return v == 2   ? reinterpret_cast<const void*>(&k_jacobi_one_window<2>)
         : v == 4 ? reinterpret_cast<const void*>(&k_jacobi_one_window<4>)
                  : reinterpret_cast<const void*>(&k_jacobi_one_window<8>);
}

// `steps` steps of N = n - 2 interior values in the shape t (t.launches > 0).
int tile_launch(TilePlan t, float* u, float* scratch, int64_t N, int steps, float r, hipStream_t s) {
  if (t.launches == 1) {
    int n32 = (int)N;
    void* args[] = {&u, &n32, &steps, &r};
    return launch(one_window_kernel(t.v), 1, kWave, args, s, false);
  }
  const int grid = (int)((t.waves + kTileWG / kWave - 1) / (kTileWG / kWave));
  float* src = u;
  float* dst = scratch;
  for (int64_t i = 0; i < t.launches; ++i) {
    int now = (int)(steps * (i + 1) / t.launches - steps * i / t.launches);
    void* args[] = {&src, &dst, &N, &t.m, &t.k, &now, &r};
    int rc = launch(tile_kernel(t.v), grid, kTileWG, args, s, false);
    if (rc) return rc;
    std::swap(src, dst);
  }
  return RED_OK;
}

}  // namespace

int stencil_launch(float* u, float* scratch, int64_t n, int steps, float r, int steps_per_sync, const red_plan& p,
                   Workspace* ws, hipStream_t s, const DeviceInfo& dev) {
  if (n < 3 || steps == 0) return RED_OK;
  int variant = p.variant;
  // AUTO without a workgroup size or grid of the caller's (which are shapes
  // of the other forms): blocked steps, or one launch per step where that is
  // faster (stencil_plan.h).  From three steps on, blocked steps were faster
  // than both other forms at every size (1000 steps on 64 K values: 65 us
  // against 200 for the persistent form; 200 steps on 4 M: 77 against 188;
  // 40 steps on 24 M, which only one launch per step could run: 92 against
  // 1250).
  if (variant == RED_VARIANT_AUTO && p.wg == 0 && p.grid == 0) {
    const TilePlan t = plan_tiles(n - 2, steps, dev.cus, dev.clock_khz);
    if (t.launches > 0) {
      const int slot = timer_begin(s);
      const int rc = tile_launch(t, u, scratch, n - 2, steps, r, s);
      timer_end(s, slot);
      return rc;
    }
    variant = RED_VARIANT_RELAUNCH;
  }
  // The geometry (workgroups, block length) is set for the caller's halo,
  // or for a halo of 8 when the library chooses it.
  const int k_req = steps_per_sync > 0 ? steps_per_sync : 8;
  // Window capacity: kWindowMax values, or 32 per thread of the caller's
  // workgroup size.
  const int64_t wmax = p.wg > 0 ? std::min<int64_t>(kWindowMax, (int64_t)32 * p.wg) : kWindowMax;

  // Persistent geometry: one workgroup per CU unless the array needs more
  // windows, then a whole number of workgroups per CU, so that no CU holds
  // one block more than the others (4 M values in windows of 16 K would
  // need 259: 512 of half the size keep every CU equally loaded); at least
  // 64 values per workgroup.
  int grid = 0, wg = p.wg > 0 ? p.wg : 512, vpt = 0;
  int64_t m = 0;
  int k = 0;
  if (variant != RED_VARIANT_RELAUNCH) {
    const int64_t cap = std::max<int64_t>(1, wmax - 2 * (int64_t)k_req);  // block values per window
    const int64_t need = (n + cap - 1) / cap;
    int64_t g = p.grid > 0 ? p.grid
                           : need <= dev.cus ? (int64_t)dev.cus : (need + dev.cus - 1) / dev.cus * dev.cus;
    g = std::max<int64_t>(1, std::min<int64_t>(g, (n + 63) / 64));
    m = (n + g - 1) / g;
    grid = (int)((n + m - 1) / m);
    // Halo width: the caller's steps per barrier, else the widest halo up to
    // kAutoHalo that the window holds beside the block.  The halo values are
    // recomputed redundantly, so a wider one trades a little arithmetic for
    // fewer grid barriers.
    k = steps_per_sync > 0 ? (int)std::min<int64_t>(k_req, m)
                           : (int)std::max<int64_t>(1, std::min<int64_t>({kAutoHalo, m, (wmax - m) / 2}));
    const int64_t len = m + 2 * (int64_t)k;
    // Values per thread and threads per workgroup: the caller's workgroup
    // size with the fewest values per thread that cover the window; else
    // the fewest values per thread (2 to 32) whose workgroup, rounded to
    // whole wavefronts, stays within 1024 threads and is co-resident with
    // the grid (small windows spread over more wavefronts: 0.28 against
    // 0.37 us per step with 8 values per thread at 64 K values).
    int g_max = 0;
    if (len <= wmax) {
      if (p.wg > 0) {
        for (int v = 4; v <= 32 && !vpt; v *= 2)
          if ((int64_t)v * wg >= len) vpt = v;
        int rc = stencil_coresident(vpt, wg, dev, &g_max);
        if (rc) return rc;
      } else {
        for (int v = 2; v <= 32 && !vpt; v *= 2) {
          const int t = (int)((len + v - 1) / v + kWave - 1) / kWave * kWave;
          if (t > 1024) continue;
          int gm = 0;
          int rc = stencil_coresident(v, t, dev, &gm);
          if (rc) return rc;
          if (gm >= grid) {
            vpt = v;
            wg = t;
            g_max = gm;
          }
        }
      }
    }
    if (!vpt || g_max < grid) {
      if (variant == RED_VARIANT_PERSISTENT)
        return set_error(RED_EINVAL,
                         "persistent stencil: %d workgroups of %lld values with halos do not fit the co-resident "
                         "workgroups' registers (at most %lld values per workgroup; %d co-resident)",
                         grid, (long long)len, (long long)wmax, g_max);
      variant = RED_VARIANT_RELAUNCH;  // AUTO: the array does not fit on chip
    } else {
      variant = RED_VARIANT_PERSISTENT;
    }
  }

  if (variant == RED_VARIANT_RELAUNCH) {
    int gridr = p.grid > 0 ? p.grid : 4 * dev.cus;
    gridr = (int)std::max<int64_t>(1, std::min<int64_t>(gridr, (n + wg - 1) / wg));
    float* src = u;
    float* dst = scratch;
    for (int t = 0; t < steps; ++t) {
      void* args[] = {&src, &dst, &n, &r};
      int rc = launch(reinterpret_cast<const void*>(&k_jacobi_step), gridr, wg, args, s, false);
      if (rc) return rc;
      std::swap(src, dst);
    }
    if (src != u) {
      void* args[] = {&src, &u, &n};
      return launch(reinterpret_cast<const void*>(&k_copy_f32), gridr, wg, args, s, false);
    }
    return RED_OK;
  }

  StencilArgs a;
  a.u = u;
  a.scratch = scratch;
  a.n = n;
  a.m = m;
  a.steps = steps;
  a.k = k;
  a.r = r;
  a.words = ws->words;
  a.spin_limit = watchdog_spins();
  a.bar_groups = ((p.flags & RED_FLAG_XCD) && xcd_tree_fits(dev.nxcc)) ? (kBarrierXcd | (unsigned)dev.nxcc)
                                                            : barrier_groups(grid);
  void* args[] = {&a};
  const bool coop = (p.flags & RED_FLAG_PLAIN_LAUNCH) == 0;
  const int slot = timer_begin(s);
  int rc = launch(persistent_kernel(vpt), grid, wg, args, s, coop, edge_bytes(wg));
  timer_end(s, slot);
  return rc;
}

}  // namespace redsum
