// qv_vi.hip -- offline value bounds on gfx950 that score the leaves of the
// QV-tree:
//   * Q-MDP value iteration: the MDP value iteration of Sec. V-B, which is
//     the alpha-vector recursion of Sec. IV-A with a perfect sensor;
//   * the fast informed bound (FIB), the alpha-vector equation of Sec. IV-A:
//       alpha^a(x) = R(x,a) + gamma sum_z max_a' sum_x' O(z|x') T(x,a,x') alpha^a'(x').
// Both are Jacobi sweeps in FP32.  The residual of sweep k, max |x_k - x_{k-1}|
// over free cells (and actions), is formed in FP64 (exact for a difference
// of two FP32 values); workgroups leave their maxima in slots, and a maximum
// does not depend on their order.
//
// Value iteration needs little arithmetic per cell and sweep, so its launches
// do several sweeps each: a workgroup holds a region of the grid, of which the
// inner part stays exact for as many sweeps as the rim is wide.  A grid that
// one workgroup holds is solved in one launch.  FIB and the blind bound do one
// sweep per launch, or, on small grids, all sweeps in one cooperative launch:
// every workgroup is resident, and after each sweep the workgroups meet at a
// grid barrier, read the sweep's residual and max |value| and so all stop
// after the same sweep (the stopping rule sees the same numbers everywhere).
// Launches after the one in which the rule fired do nothing, and the host
// looks at the residuals every few launches.  All forms do the same arithmetic
// per cell, so their results are bitwise equal.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "qv_internal.h"

namespace qv {

constexpr int kViChunk = 64;   // sweeps between two looks at the residuals
constexpr int kMaxCoopGrid = 4096;   // workgroups of a one-launch solve at most
// workgroups of a sweep launch at most: four per CU; more would only add
// residual slots for every workgroup to read
constexpr int kSweepGrid = 1024;
// FIB's are a wavefront per action; of two, twice as many (512x512, 2 actions,
// dense rows, a sweep: 38 us, 33 so)
constexpr int kFibGrid = 2048;
constexpr int kMaxWaves = 16;   // wavefronts of a sweep workgroup at most

// ---------------------------------------------------------------------------
// grid barrier and the shared stopping rule
// ---------------------------------------------------------------------------

// Values that other workgroups of the same launch read (V_k, alpha_k) are
// stored with agent-scope atomic stores and loaded with agent-scope atomic
// loads.  In the AMDGPU memory model such accesses are performed at the
// device's coherence point (past the per-XCD L2, which is not coherent
// across XCDs), so no cache-wide fence is needed; read-only tables (map
// signature, stay table, rewards) keep their L2 copies across sweeps.
template <bool COH>
__device__ __forceinline__ float ld_val(const float *p) {
  if constexpr (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return *p;
}
template <bool COH>
__device__ __forceinline__ void st_val(float *p, float v) {
  if constexpr (COH)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    *p = v;
}

// Grid barrier of a cooperative launch, round r = 1, 2, ...: the counter
// *bar reaches r * gridDim.x once every workgroup has arrived.  Every
// thread first waits until its own stores (and the workgroup's residual
// atomics) have completed at the coherence point (s_waitcnt 0); after the
// workgroup barrier lane 0 arrives with an agent-scope atomic add and polls
// the counter.  A workgroup that sees the full count therefore reads, with
// its agent-scope loads, everything every workgroup wrote before arriving.
// The wait is bounded: after kSpinLimit polls (seconds, far beyond any
// sweep) lane 0 raises *abort and leaves, and every other waiting workgroup
// leaves as soon as it sees the flag, so the launch always ends; the
// caller then stops.
constexpr long long kSpinLimit = 1ll << 22;

__device__ __forceinline__ void grid_sync(unsigned long long *bar, unsigned long long target,
                                          unsigned int *abort) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(bar, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    long long polls = 0;
    while (__hip_atomic_load(bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
      if (__hip_atomic_load(abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
      if (++polls > kSpinLimit) {
        __hip_atomic_store(abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  __syncthreads();
}

// Control block of one solve in the workspace.
struct SweepCtl {
  unsigned long long *res, *vmax;   // [max_sweeps + 2]: bit patterns of r_k, max |x_k|
  unsigned long long *bar;          // grid barrier counter
  double *out_res;                  // residual of the last sweep
  int *out_k;                       // number of sweeps run
  unsigned int *abort;              // set when a barrier wait gave up
  unsigned int *arrive, *stop;      // value iteration: workgroups done, whether the rule fired
  double *part;                     // [2][2][grid]: per-workgroup r, max |x| of a sweep
  int max_sweeps;
  double tol;
};

__device__ __forceinline__ double load_bits(const unsigned long long *p) {
  return __longlong_as_double(
      (long long)__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Largest of the 64 lanes' values (>= 0), in every lane, on the DPP network:
// lane permutes through LDS would be the longest part of a small sweep.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_max(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo =
      (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROW_MASK, 0xF, false);
  const uint32_t hi =
      (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROW_MASK, 0xF, false);
  return fmax(v, __longlong_as_double((long long)((uint64_t)hi << 32 | lo)));
}
__device__ __forceinline__ double wave_max(double v) {
  v = dpp_max<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]
  v = dpp_max<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]
  v = dpp_max<0x141, 0xF>(v);   // row_half_mirror
  v = dpp_max<0x140, 0xF>(v);   // row_mirror
  v = dpp_max<0x142, 0xA>(v);   // row_bcast:15
  v = dpp_max<0x143, 0xC>(v);   // row_bcast:31
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), 63);
  return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// One-launch form: workgroup g's (r, max |x|) of sweep k go to slot g of the
// sweep's parity buffer (plain coherent stores, no atomic on a shared word);
// after the grid barrier wavefront 0 of every workgroup takes the maxima
// over all slots (the same values everywhere: max is order independent),
// and workgroup 0 records them as sweep k's residual.  Returns whether the
// rule fires (in lane 0 of wavefront 0).
__device__ __forceinline__ void sweep_part_store(const SweepCtl &c, int k, double r, double v,
                                                 double *red) {
  r = wave_max(r);
  v = wave_max(v);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  if (lane == 0) {
    red[wave] = r;
    red[kMaxWaves + wave] = v;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)blockDim.x / kWave; ++w) {
      r = fmax(r, red[w]);
      v = fmax(v, red[kMaxWaves + w]);
    }
    double *p = c.part + (size_t)(k & 1) * 2 * gridDim.x;
    __hip_atomic_store(p + blockIdx.x, r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(p + gridDim.x + blockIdx.x, v, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
}

__device__ __forceinline__ int sweep_part_decide(const SweepCtl &c, int k) {
  const int lane = threadIdx.x & (kWave - 1);
  const double *p = c.part + (size_t)(k & 1) * 2 * gridDim.x;
  double r = 0.0, v = 0.0;
  for (int g = lane; g < (int)gridDim.x; g += kWave) {
    r = fmax(r, __hip_atomic_load(p + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    v = fmax(v, __hip_atomic_load(p + gridDim.x + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  }
  r = wave_max(r);
  v = wave_max(v);
  if (blockIdx.x == 0 && lane == 0) {
    c.res[k] = (unsigned long long)__double_as_longlong(r);
    c.vmax[k] = (unsigned long long)__double_as_longlong(v);
  }
  return (r == 0.0 || r <= c.tol * fmax(1.0, v)) ? 1 : 0;
}

// Per-sweep form: the workgroups' (r, max |x|) go to slots of a parity buffer
// as above, and sweep k reads those of sweep k - 1 first.  (A max of every
// workgroup into one word by atomics cost about 40 ns each, one after
// another: 82 of the 123 us of a FIB sweep of 512x512.)

// Workgroup maxima of sweep k's slots (g of them), in every thread.
__device__ __forceinline__ void sweep_slots_max(const SweepCtl &c, int k, int g, double *red,
                                                double &r, double &v) {
  const double *p = c.part + (size_t)(k & 1) * 2 * g;
  r = v = 0.0;
  for (int i = threadIdx.x; i < g; i += blockDim.x) {
    r = fmax(r, p[i]);
    v = fmax(v, p[g + i]);
  }
  r = wave_max(r);
  v = wave_max(v);
  const int wave = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) {
    red[wave] = r;
    red[kMaxWaves + wave] = v;
  }
  __syncthreads();
  for (int w = 0; w < (int)blockDim.x / kWave; ++w) {
    r = fmax(r, red[w]);
    v = fmax(v, red[kMaxWaves + w]);
  }
  __syncthreads();
}

// Start of sweep k: records sweep k - 1's residual; if its rule fired
// (r = 0 or r <= tol * max(1, max |x|)), hands its slots on to the next sweep,
// so that all later ones stop too, and returns true.
__device__ __forceinline__ bool sweep_stopped(const SweepCtl &c, int k, double *red) {
  if (k <= 1) return false;
  const int g = gridDim.x;
  double r, v;
  sweep_slots_max(c, k - 1, g, red, r, v);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    c.res[k - 1] = (unsigned long long)__double_as_longlong(r);
    c.vmax[k - 1] = (unsigned long long)__double_as_longlong(v);
  }
  if (!(r == 0.0 || r <= c.tol * fmax(1.0, v))) return false;
  if (threadIdx.x < 2) {
    const size_t at = (size_t)threadIdx.x * g + blockIdx.x;
    c.part[(size_t)(k & 1) * 2 * g + at] = c.part[(size_t)((k - 1) & 1) * 2 * g + at];
  }
  return true;
}

// The residual of the last sweep launched (k, of g workgroups).
__global__ __launch_bounds__(kBlock) void k_sweep_close(SweepCtl c, int k, int g) {
  __shared__ double red[2 * kMaxWaves];
  double r, v;
  sweep_slots_max(c, k, g, red, r, v);
  if (threadIdx.x == 0) {
    c.res[k] = (unsigned long long)__double_as_longlong(r);
    c.vmax[k] = (unsigned long long)__double_as_longlong(v);
  }
}

__global__ void k_sweep_fill(unsigned long long *res, unsigned long long *vmax, int n,
                             unsigned long long *bar, float *x0, float *x1, long long nx) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    res[i] = 0ull;
    vmax[i] = 0ull;
  }
  if (i == 0) {
    bar[0] = 0ull;   // barrier counter
    bar[2] = 0ull;   // sweep count and abort flag
    bar[3] = 0ull;   // arrivals and stop flag
  }
  if (i < nx) {
    x0[i] = 0.f;
    x1[i] = 0.f;
  }
}

// ---------------------------------------------------------------------------
// Q-MDP value iteration
// ---------------------------------------------------------------------------

// The slip table in a register per lane: lane 3 a + k % 3 of register k / 3
// holds T'(a,k), so that an entry is one lane read and not a scalar load that
// the next instruction waits for.
struct SlipLanes {
  float v[3];
  uint64_t nz[3];   // lanes that are not 0
  __device__ __forceinline__ explicit SlipLanes(const DevModel &m) {
    const int lane = threadIdx.x & (kWave - 1);
    const bool has = lane < 3 * m.A;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      v[i] = has ? m.slip[lane / 3 * 9 + 3 * i + lane % 3] : 0.f;
      nz[i] = __ballot(v[i] != 0.f);
    }
  }
  __device__ __forceinline__ bool moves(int a, int k) const {
    return (nz[k / 3] >> (3 * a + k % 3)) & 1ull;
  }
  __device__ __forceinline__ float at(int a, int k) const {
    return __int_as_float(
        __builtin_amdgcn_readlane(__float_as_int(v[k / 3]), 3 * a + k % 3));
  }
};

// Row t of an alpha or reward table into registers.
template <int AM, bool COH>
__device__ __forceinline__ void value_row(const float *al, int t, int A, bool vec, float (&v)[AM]) {
  if constexpr (!COH && AM % 4 == 0) {
    if (vec) {   // rows of AM values, 16-byte aligned
      const float4 *q = reinterpret_cast<const float4 *>(al + (size_t)t * AM);
#pragma unroll
      for (int i = 0; i < AM / 4; ++i) {
        const float4 f = q[i];
        v[4 * i] = f.x;
        v[4 * i + 1] = f.y;
        v[4 * i + 2] = f.z;
        v[4 * i + 3] = f.w;
      }
      return;
    }
  }
  // (columns beyond A repeat column 0)
#pragma unroll
  for (int ap = 0; ap < AM; ++ap) v[ap] = ld_val<COH>(al + (size_t)t * A + (ap < A ? ap : 0));
}

// A workgroup's region: kViX columns by kViY rows, a thread per column and
// strip of kViStrip rows.  With a rim of kViRim cells on each side the inner
// kViOutX x kViOutY cells are exact after kViRim sweeps (what lies beyond the
// region reads as 0, and the error moves in by one cell a sweep).  Why these
// sizes: 512x512 makes 256 regions, one per CU; the rim costs 2.2 times the
// cells and saves seven of eight launches, each longer than a sweep's work.
// A thread's cells, their map bits and reward rows and the slip table stay in
// registers for all sweeps of a launch (two wavefronts per SIMD leave room for
// 256).  Bound by the vector ALU and, between sweeps, the barrier.  Measured,
// 512x512, 218 sweeps: one launch per sweep 3.6 ms, this 1.2 ms; skipping the
// moves of probability 0 by a scalar branch each, 1.5 ms.
constexpr int kViX = 48, kViStrip = 5, kViGroups = 10, kViY = kViStrip * kViGroups;
constexpr int kViRim = 8, kViOutX = kViX - 2 * kViRim, kViOutY = kViY - 2 * kViRim;
constexpr int kViBlock = 512, kViPitch = kViX + 2;
static_assert(kViX * kViGroups <= kViBlock, "a thread per column and strip");

// Work of a launch.  Block: `ns` sweeps k0 + 1 .. k0 + ns from V_{k0} into
// Vout, unless the rule fired before.  Table: `ns` sweeps, then Q of the next
// one.  Solve: sweeps until the rule fires, then Q of the last.
enum ViMode { kViBlockMode, kViTableMode, kViSolveMode };

template <int AM>
struct ViShared {
  float v[2][(kViY + 2) * kViPitch];
  float stay[AM * 256];
  double red[kViRim][2][kViBlock / kWave];
  int last;
};

// Q(s,a) = R(s,a) + gamma * (sum_k T'(a,k) V(s + d_k) + stay(s,a) V(s)) for
// the strip's cells, the expectation over T(s,a,.) of Sec. V: V reads as 0
// where a move fails (its mass is in `stay`).  w: the strip's 3-column window.
template <int AM>
__device__ __forceinline__ void vi_strip_q(const DevModel &m, const float (&T)[AM][9],
                                           const float *stay, const uint32_t (&info)[kViStrip],
                                           const float (&w)[kViStrip + 2][3],
                                           const float (&R)[kViStrip][AM], int a,
                                           float (&q)[kViStrip]) {
#pragma unroll
  for (int r = 0; r < kViStrip; ++r) q[r] = 0.f;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    if (k == 4) continue;
    const float t = T[a][k];
#pragma unroll
    for (int r = 0; r < kViStrip; ++r) q[r] = fmaf(t, w[r + k / 3][k % 3], q[r]);
  }
#pragma unroll
  for (int r = 0; r < kViStrip; ++r) {
    q[r] = fmaf(stay[a * 256 + (int)sig_out8(info[r])], w[r + 1][1], q[r]);
    q[r] = fmaf(m.gamma, (info[r] & kSigGoal) ? w[r + 1][1] : q[r], R[r][a]);
  }
}

template <int AM, ViMode MODE>
__global__ __launch_bounds__(kViBlock) void k_vi(DevModel m, const uint32_t *sig,
                                                 const float *staytab, int regions_x,
                                                 const float *Vin, float *Vout, float *Q, int k0,
                                                 int ns, double *slots, SweepCtl c) {
  __shared__ ViShared<AM> sh;
  const int A = m.A, W = m.W, H = m.H, tid = threadIdx.x;
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  const int col = tid % kViX, strip = tid / kViX;
  const bool act = strip < kViGroups;
  const int ry = blockIdx.x / regions_x, rx = blockIdx.x - ry * regions_x;
  const int rim = MODE == kViSolveMode ? 0 : kViRim;
  const int x = rx * kViOutX - rim + col, y0 = ry * kViOutY - rim + strip * kViStrip;
  // ---- the strip's cells
  uint32_t info[kViStrip];
  float R[kViStrip][AM];
  bool own[kViStrip];
  const bool rvec = A == AM && AM % 4 == 0 && (reinterpret_cast<uintptr_t>(m.R) & 15u) == 0;
  const bool stopped = MODE == kViBlockMode && *c.stop;
#pragma unroll
  for (int r = 0; r < kViStrip; ++r) {
    const int y = y0 + r, ly = strip * kViStrip + r;
    const bool in = act && x >= 0 && x < W && y >= 0 && y < H;
    const int t = in ? y * W + x : 0;
    info[r] = in ? sig[t] : 0u;
    own[r] = in && (MODE == kViSolveMode ||
                    (col >= kViRim && col < kViRim + kViOutX && ly >= kViRim &&
                     ly < kViRim + kViOutY));
    value_row<AM, false>(m.R, t, A, rvec, R[r]);
    const float v = in && MODE != kViSolveMode ? Vin[t] : 0.f;
    if (act) sh.v[0][(ly + 1) * kViPitch + col + 1] = (info[r] & kSigFree) ? v : 0.f;
  }
  for (int i = tid; i < A * 256; i += kViBlock) sh.stay[i] = staytab[i];
  // the entries around the region, in both buffers
  for (int i = tid; i < 2 * (kViX + kViY + 2); i += kViBlock) {
    const int e = i < 2 * kViPitch ? (i < kViPitch ? i : (kViY + 1) * kViPitch + i - kViPitch)
                                   : (1 + (i - 2 * kViPitch) / 2) * kViPitch +
                                         ((i & 1) ? kViPitch - 1 : 0);
    sh.v[0][e] = sh.v[1][e] = 0.f;
  }
  const SlipLanes sl(m);
  if (stopped) return;   // (the same in every thread)
  float T[AM][9];   // the slip table (kept there: as scalars it does not fit)
#pragma unroll
  for (int a = 0; a < AM; ++a)
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      if (k == 4) continue;
      T[a][k] = sl.at(a < A ? a : 0, k);
      asm volatile("" : "+v"(T[a][k]));
    }
  __syncthreads();
  const float *stay = sh.stay;
  const int pos = strip * kViStrip * kViPitch + col;
  auto window = [&](const float *v, float (&w)[kViStrip + 2][3]) {
#pragma unroll
    for (int r = 0; r < kViStrip + 2; ++r)
#pragma unroll
      for (int j = 0; j < 3; ++j) w[r][j] = v[pos + r * kViPitch + j];
  };
  int kend = 0;
  for (int k = 1; k <= ns; ++k) {
    const float *vi = sh.v[(k - 1) & 1];
    float *vo = sh.v[k & 1];
    double res = 0.0, vm = 0.0;
    if (act) {
      float w[kViStrip + 2][3], best[kViStrip], q[kViStrip];
      window(vi, w);
#pragma unroll
      for (int r = 0; r < kViStrip; ++r) best[r] = -INFINITY;
#pragma unroll
      for (int a = 0; a < AM; ++a) {
        if (a >= A) continue;
        vi_strip_q<AM>(m, T, stay, info, w, R, a, q);
#pragma unroll
        for (int r = 0; r < kViStrip; ++r) best[r] = fmaxf(best[r], q[r]);
      }
#pragma unroll
      for (int r = 0; r < kViStrip; ++r) {
        const bool fr = (info[r] & kSigFree) != 0u;
        vo[pos + (r + 1) * kViPitch + 1] = fr ? best[r] : 0.f;
        if (fr && own[r]) {
          res = fmax(res, fabs((double)best[r] - (double)w[r + 1][1]));
          vm = fmax(vm, fabs((double)best[r]));
        }
      }
    }
    if constexpr (MODE != kViTableMode) {
      res = wave_max(res);
      vm = wave_max(vm);
      if (lane == 0) {
        sh.red[(k - 1) % kViRim][0][wave] = res;
        sh.red[(k - 1) % kViRim][1][wave] = vm;
      }
    }
    __syncthreads();
    if constexpr (MODE == kViSolveMode) {
      res = vm = 0.0;
#pragma unroll
      for (int i = 0; i < kViBlock / kWave; ++i) {
        res = fmax(res, sh.red[(k - 1) % kViRim][0][i]);
        vm = fmax(vm, sh.red[(k - 1) % kViRim][1][i]);
      }
      kend = k;
      if (tid == 0) *c.out_res = res;
      if (res == 0.0 || res <= c.tol * fmax(1.0, vm)) break;
    }
  }
  if constexpr (MODE == kViBlockMode) {
    const float *v = sh.v[ns & 1];
#pragma unroll
    for (int r = 0; r < kViStrip; ++r)
      if (own[r]) Vout[(y0 + r) * W + x] = v[pos + (r + 1) * kViPitch + 1];
    // the region's maxima, by sweep; the last workgroup to leave them folds
    // all regions' and sets the stop flag if the rule fired in this block
    const int G = gridDim.x;
    if (tid < 2 * ns) {
      const int j = tid >> 1;
      double f = 0.0;
      for (int i = 0; i < kViBlock / kWave; ++i) f = fmax(f, sh.red[j][tid & 1][i]);
      __hip_atomic_store(slots + (size_t)tid * G + blockIdx.x, f, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0)
      sh.last = __hip_atomic_fetch_add(c.arrive, 1u, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT) == (unsigned)G - 1u;
    __syncthreads();
    if (!sh.last) return;
    for (int j = wave; j < ns; j += kViBlock / kWave) {
      double res = 0.0, vm = 0.0;
      for (int g = lane; g < G; g += kWave) {
        res = fmax(res, __hip_atomic_load(slots + (size_t)(2 * j) * G + g, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT));
        vm = fmax(vm, __hip_atomic_load(slots + (size_t)(2 * j + 1) * G + g, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT));
      }
      res = wave_max(res);
      vm = wave_max(vm);
      if (lane == 0) {
        c.res[k0 + 1 + j] = (unsigned long long)__double_as_longlong(res);
        c.vmax[k0 + 1 + j] = (unsigned long long)__double_as_longlong(vm);
        if (res == 0.0 || res <= c.tol * fmax(1.0, vm)) *c.stop = 1u;
      }
    }
    if (tid == 0) *c.arrive = 0u;
    return;
  }
  // Q from the values in buffer `at`: in a solve those before the last sweep
  const int at = MODE == kViSolveMode ? (kend - 1) & 1 : ns & 1;
  if (act) {
    float w[kViStrip + 2][3], q[kViStrip];
    window(sh.v[at], w);
#pragma unroll
    for (int a = 0; a < AM; ++a) {
      if (a >= A) continue;
      vi_strip_q<AM>(m, T, stay, info, w, R, a, q);
#pragma unroll
      for (int r = 0; r < kViStrip; ++r)
        if (own[r])
          Q[((size_t)(y0 + r) * W + x) * A + a] = (info[r] & kSigFree) ? q[r] : 0.f;
    }
  }
  if (MODE == kViSolveMode && tid == 0) *c.out_k = kend;
}

// ---------------------------------------------------------------------------
// fast informed bound
// ---------------------------------------------------------------------------

// What a sweep needs to know of a free cell x, gathered once per solve:
//   bits 0..35  wall readings of the successors k = 0..8 (4 bits each; of x
//               itself where move k fails),
//   bits 36..43 the moves that succeed (order of the map signature),
//   bits 44..52 successor k carries a landmark,
//   bits 53..56 the wall bits in which the successors' readings differ,
//   bit  57     the goal.
// fib_terms of a record: the number of its differing bits.
constexpr int kFibOut = 36, kFibLm = 44, kFibDiff = 53, kFibGoal = 57;
constexpr int kFibClasses = 5;

__device__ __forceinline__ uint64_t fib_record(const DevModel &m, const uint32_t *sig, int x,
                                               uint32_t sg) {
  uint64_t rec = (uint64_t)sig_out8(sg) << kFibOut;
  if (sg & kSigGoal) return rec | (1ull << kFibGoal);   // absorbing: only itself
  uint32_t all1 = 15u, any1 = 0u;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const bool ok = k == 4 || ((sg >> (k < 4 ? k : k - 1)) & 1u);
    const uint32_t st = sig[ok ? x + (k / 3 - 1) * m.W + (k % 3 - 1) : x];
    const uint32_t w = sig_wall(st), lm = sig_lm(st);
    all1 &= w;
    any1 |= w;
    rec |= (uint64_t)w << (4 * k);
    if (ok && lm != 0u && lm <= (uint32_t)m.L) rec |= 1ull << (kFibLm + k);
  }
  return rec | (uint64_t)(any1 & ~all1) << kFibDiff;
}

__device__ __forceinline__ int fib_terms(uint64_t rec) {
  return __builtin_popcount((uint32_t)(rec >> kFibDiff) & 15u);
}

// The free cells in order of the number of differing wall bits, most first
// (the long work starts early), by index within a class: count per block and
// class, scan, scatter.  ctl[0] is the number of free cells.
__global__ __launch_bounds__(kBlock) void k_fib_count(DevModel m, const uint32_t *sig,
                                                      int32_t *counts) {
  __shared__ int32_t n[kFibClasses];
  if (threadIdx.x < kFibClasses) n[threadIdx.x] = 0;
  __syncthreads();
  const int x = blockIdx.x * kBlock + threadIdx.x;
  if (x < m.S) {
    const uint32_t sg = sig[x];
    if (sg & kSigFree) atomicAdd(&n[kFibClasses - 1 - fib_terms(fib_record(m, sig, x, sg))], 1);
  }
  __syncthreads();
  if (threadIdx.x < kFibClasses) counts[threadIdx.x * gridDim.x + blockIdx.x] = n[threadIdx.x];
}

__global__ __launch_bounds__(1024) void k_fib_scan(int32_t *counts, int n, int32_t *ctl) {
  __shared__ int32_t sums[16];
  __shared__ int32_t base;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  if (threadIdx.x == 0) base = 0;
  __syncthreads();
  for (int i0 = 0; i0 < n; i0 += 1024) {
    const int i = i0 + threadIdx.x;
    const int v = i < n ? counts[i] : 0;
    const int incl = wave_scan_incl(v);
    if (lane == kWave - 1) sums[wave] = incl;
    __syncthreads();
    int before = base;
    for (int w = 0; w < wave; ++w) before += sums[w];
    if (i < n) counts[i] = before + incl - v;
    __syncthreads();
    if (threadIdx.x == 1023) base = before + incl;
    __syncthreads();
  }
  if (threadIdx.x == 0) ctl[0] = base;
}

__global__ __launch_bounds__(kBlock) void k_fib_scatter(DevModel m, const uint32_t *sig,
                                                        const int32_t *counts, int32_t *cells,
                                                        uint64_t *recs) {
  __shared__ int32_t n[kBlock / kWave][kFibClasses];
  const int x = blockIdx.x * kBlock + threadIdx.x;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const uint32_t sg = x < m.S ? sig[x] : 0u;
  const bool free = (sg & kSigFree) != 0u;
  const uint64_t rec = free ? fib_record(m, sig, x, sg) : 0ull;
  const int cls = free ? kFibClasses - 1 - fib_terms(rec) : kFibClasses;
  int rank = 0;
  for (int c = 0; c < kFibClasses; ++c) {
    const uint64_t in = __ballot(cls == c);
    if (cls == c) rank = __popcll(in & ((1ull << lane) - 1ull));
    if (lane == 0) n[wave][c] = __popcll(in);
  }
  __syncthreads();
  if (!free) return;
  int at = counts[cls * gridDim.x + blockIdx.x] + rank;
  for (int w = 0; w < wave; ++w) at += n[w][cls];
  cells[at] = x;
  recs[at] = rec;
}

// The FIB right-hand side.  The successors of a free cell x are its neighbours
// k != 4 that a move enters and x itself, which takes the stay mass:
// T(x,a,x + d_k) = T'(a,k), T(x,a,x) = stay(x,a).  With C[zw][w] the
// wall-reading likelihood and lambda(x') = 1 - rho on a landmark cell, else 1,
// the sum over z splits into
//   zl = 0:  sum_zw max_a' sum_k C[zw][w(x_k)] lambda(x_k) T_k(a) alpha^a'(x_k),
//   zl = l:  rho T_k(a) max_a' alpha^a'(x_k) for the successor x_k that is
//            landmark l (only it can report l, and sum_zw C[zw][w] = 1).
// C is a product over the wall bits.  The factors of a bit in which all
// successors agree leave the max and sum to 1 over that bit of zw, so zw runs
// only over the bits in which they differ: 2^bits terms instead of 16, one
// in the open.  Moves of probability 0 are left out: of nine, the slip tables
// in use make three or four.  The goal is absorbing: its right-hand side is
// R + gamma max_a' alpha^a'(goal).
//
// A workgroup of one wavefront per action takes 64 cells at a time: the
// wavefronts stage the nine successors' rows and the reward row in LDS (zero
// where a move fails, scaled by lambda on a landmark), then each forms its
// action's value from the rows its moves need, held in registers.  Bound by
// the vector ALU and the latency of the row loads; one thread per cell with
// all rows and actions took 160 VGPRs, three wavefronts per SIMD, and left
// both exposed.  Measured, 512x512, 8 actions of three moves, a sweep: 123 us before
// (16 terms of nine moves for every cell, and the residual's atomics), 24.8 now.
template <int AM>
struct FibShared {
  static constexpr int Q = AM / 4, E = AM % 4;   // a row: Q 4-vectors and E (0 or 1) values
  float4 q[10][Q][kWave];                        // successors 0..8, reward row 9
  float e[E ? 10 : 1][E ? kWave : 1];
  float mk[9][kWave];                            // rho max_a' of a landmark's row, else 0
  float out[AM * (kWave + 1)];
  float stay[AM * 256];
  float ctab[256];
  int cell[kWave];
};

template <int AM>
__device__ __forceinline__ float fib_row_max(const float (&v)[AM]) {
  float mx = v[0];
#pragma unroll
  for (int ap = 1; ap < AM; ++ap) mx = fmaxf(mx, v[ap]);
  return mx;
}

template <int AM>
__device__ __forceinline__ void fib_put(FibShared<AM> &sh, int k, const float (&v)[AM]) {
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
  for (int i = 0; i < AM / 4; ++i)
    sh.q[k][i][lane] = make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
  if constexpr (AM % 4 != 0) sh.e[k][lane] = v[AM - 1];
}

template <int AM>
__device__ __forceinline__ void fib_get(const FibShared<AM> &sh, int k, float (&v)[AM]) {
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
  for (int i = 0; i < AM / 4; ++i) {
    const float4 f = sh.q[k][i][lane];
    v[4 * i] = f.x;
    v[4 * i + 1] = f.y;
    v[4 * i + 2] = f.z;
    v[4 * i + 3] = f.w;
  }
  if constexpr (AM % 4 != 0) v[AM - 1] = sh.e[k][lane];
}

// Entry a (uniform) of a staged row.
template <int AM>
__device__ __forceinline__ float fib_get1(const FibShared<AM> &sh, int k, int a) {
  const int lane = threadIdx.x & (kWave - 1);
  if (AM % 4 != 0 && a == AM - 1) return sh.e[k][lane];
  return reinterpret_cast<const float *>(&sh.q[k][a / 4][lane])[a % 4];
}

// The sorted cells of a FIB solve in its workspace.
struct FibCells {
  int32_t *cells, *counts, *ctl;   // [S], [classes][blocks], number of free cells
  uint64_t *recs;                  // [S]
  int nfree;
};

// The moves of an action that have a probability, without k = 4 (uniform).
// FULL: all eight of every action have one (a slip table learned from runs),
// so which they are is known at compile time: without a branch per move the
// terms' table reads go out together and the rows' registers are fixed.
// Measured, 512x512, 9 actions, a sweep: 138 us with branches, 93 so.
template <int NJ, bool FULL>
struct FibMoves {
  int k_[NJ], n;
  float T[NJ];
  __device__ __forceinline__ bool has(int j) const { return FULL || j < n; }
  __device__ __forceinline__ int k(int j) const { return FULL ? (j < 4 ? j : j + 1) : k_[j]; }
  __device__ __forceinline__ FibMoves(const SlipLanes &sl, int a) : n(0) {
    if constexpr (FULL) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) T[j] = sl.at(a, k(j));
      return;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      k_[j] = 4;
      T[j] = 0.f;
    }
#pragma unroll
    for (int kk = 0; kk < 9; ++kk) {
      if (kk == 4 || !sl.moves(a, kk)) continue;
      const float t = sl.at(a, kk);
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if (j == n) {
          k_[j] = kk;
          T[j] = t;
        }
      ++n;
    }
  }
};

// Tables of a launch, once per workgroup: the stay entries, and entry D*16 +
// mis of ctab, the product over the wall bits j of D of (bit j of mis set ?
// f_j : 1 - f_j).
template <int AM>
__device__ __forceinline__ void fib_tables(const DevModel &m, const float *staytab,
                                           FibShared<AM> &sh) {
  for (int i = threadIdx.x; i < m.A * 256; i += blockDim.x) sh.stay[i] = staytab[i];
  for (int i = threadIdx.x; i < 256; i += blockDim.x) {
    const uint32_t D = (uint32_t)i >> 4, mis = (uint32_t)i & 15u;
    float c = 1.f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if ((D >> j) & 1u) c *= ((mis >> j) & 1u) ? m.flip[j] : 1.f - m.flip[j];
    sh.ctab[i] = c;
  }
}

// The rows that a wavefront stages for a group of 64 cells, in flight while
// the group before is computed.
template <int AM>
struct FibRows {
  static constexpr int N = AM == 4 ? 10 : 2;   // rows k = a, a + A, .. < 10 (A > 4: two at most)
  float v[N][AM];
  int x;
  uint64_t rec;
  bool has;
};

template <int AM>
__device__ __forceinline__ void fib_cells_load(const FibCells &fc, int g, FibRows<AM> &f) {
  const int j = g * kWave + (int)(threadIdx.x & (kWave - 1));
  f.has = j < fc.nfree;
  f.x = f.has ? fc.cells[j] : 0;
  f.rec = f.has ? fc.recs[j] : 0ull;
}

template <int AM, bool COH>
__device__ __forceinline__ void fib_rows_load(const DevModel &m, int a, const float *ain, bool vec,
                                              bool rvec, FibRows<AM> &f) {
  const int A = m.A, W = m.W;
  const uint32_t out8 = (uint32_t)(f.rec >> kFibOut) & 255u;
#pragma unroll
  for (int i = 0; i < FibRows<AM>::N; ++i) {
    const int k = a + i * A;
    if (k > 9) continue;
    if (k == 9) {
      value_row<AM, false>(m.R, f.x, A, rvec, f.v[i]);
    } else {
      const bool ok = k == 4 || ((out8 >> (k < 4 ? k : k - 1)) & 1u);
      value_row<AM, COH>(ain, ok ? f.x + (k / 3 - 1) * W + (k % 3 - 1) : f.x, A, vec, f.v[i]);
    }
  }
}

template <int AM>
__device__ __forceinline__ void fib_rows_put(const DevModel &m, int a, FibRows<AM> &f,
                                             FibShared<AM> &sh) {
  const int A = m.A, lane = threadIdx.x & (kWave - 1);
  const float rho = m.lm_p;
  const uint32_t out8 = (uint32_t)(f.rec >> kFibOut) & 255u;
  if (a == 0) sh.cell[lane] = f.has ? f.x : -1;
#pragma unroll
  for (int i = 0; i < FibRows<AM>::N; ++i) {
    const int k = a + i * A;
    if (k > 9) continue;
    if (k < 9) {
      const bool ok = f.has && (k == 4 || ((out8 >> (k < 4 ? k : k - 1)) & 1u));
      float mk = 0.f, s = 1.f;
      if ((f.rec >> (kFibLm + k)) & 1ull) {
        mk = rho * fib_row_max<AM>(f.v[i]);
        s = 1.f - rho;
      }
      // (selected, not multiplied: a failed move's row may hold anything)
#pragma unroll
      for (int ap = 0; ap < AM; ++ap) f.v[i][ap] = ok ? s * f.v[i][ap] : 0.f;
      sh.mk[k][lane] = mk;
    }
    fib_put<AM>(sh, k, f.v[i]);
  }
}

// One FIB sweep over the sorted free cells (blocked cells keep their 0);
// `f` holds the workgroup's first group of cells.
template <int AM, int NJ, bool FULL, bool COH>
__device__ __forceinline__ void fib_pass(const DevModel &m, const FibCells &fc,
                                         const FibMoves<NJ, FULL> &mv, FibShared<AM> &sh, int a,
                                         const float *ain, float *aout, bool vec, bool rvec,
                                         FibRows<AM> f, double &r, double &vm) {
  const int A = m.A, lane = threadIdx.x & (kWave - 1);
  const int groups = (fc.nfree + kWave - 1) / kWave;
  for (int g = blockIdx.x; g < groups; g += gridDim.x) {
    const int x = f.x;
    const uint64_t rec = f.rec;
    const bool has = f.has;
    const uint32_t out8 = (uint32_t)(rec >> kFibOut) & 255u;
    fib_rows_put<AM>(m, a, f, sh);
    const bool lms = __ballot(((uint32_t)(rec >> kFibLm) & 511u) != 0u) != 0ull;
    const bool more = g + (int)gridDim.x < groups;
    if (more) fib_cells_load<AM>(fc, g + gridDim.x, f);
    __syncthreads();
    // ---- this wavefront's action
    {
      float v4[AM], v[NJ][AM];
      fib_get<AM>(sh, 4, v4);
      const bool lm4 = (rec >> (kFibLm + 4)) & 1ull;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if (mv.has(j)) fib_get<AM>(sh, mv.k(j), v[j]);
      const float R = fib_get1<AM>(sh, 9, a), stay = sh.stay[a * 256 + (int)out8];
      if (more) fib_rows_load<AM, COH>(m, a, ain, vec, rvec, f);
      float acc = 0.f;
      if (lms) {
        acc = stay * sh.mk[4][lane];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          if (mv.has(j)) acc = fmaf(mv.T[j], sh.mk[mv.k(j)][lane], acc);
      }
      const uint32_t diff = (uint32_t)(rec >> kFibDiff) & 15u;
      if (__ballot(diff != 0u) == 0ull) {   // one term, C = 1
        float s[AM];
#pragma unroll
        for (int ap = 0; ap < AM; ++ap) s[ap] = stay * v4[ap];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          if (mv.has(j)) {
#pragma unroll
            for (int ap = 0; ap < AM; ++ap) s[ap] = fmaf(mv.T[j], v[j][ap], s[ap]);
          }
        acc += fib_row_max<AM>(s);
      } else {
        // byte offsets of the successors' entries of ctab row `diff` for zw = 0
        const uint32_t row = diff << 6;
        const uint32_t e4 = row | (((uint32_t)(rec >> 16) & diff) << 2);
        uint32_t e[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) e[j] = row | (((uint32_t)(rec >> (4 * mv.k(j))) & diff) << 2);
        const char *ct = reinterpret_cast<const char *>(sh.ctab);
        uint32_t zw = 0u;   // (its bits shifted by two, as the offsets)
        do {
          const float g4 = *reinterpret_cast<const float *>(ct + (e4 ^ zw)) * stay;
          float s[AM];
#pragma unroll
          for (int ap = 0; ap < AM; ++ap) s[ap] = g4 * v4[ap];
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            if (mv.has(j)) {
              const float gj = *reinterpret_cast<const float *>(ct + (e[j] ^ zw)) * mv.T[j];
#pragma unroll
              for (int ap = 0; ap < AM; ++ap) s[ap] = fmaf(gj, v[j][ap], s[ap]);
            }
          acc += fib_row_max<AM>(s);
          zw = (zw - (diff << 2)) & (diff << 2);   // the next subset of the differing bits
        } while (zw != 0u);
      }
      // the old value: row 4's entry, before lambda
      float old = fib_get1<AM>(sh, 4, a);
      float o = fmaf(m.gamma, acc, R);
      if ((rec >> kFibGoal) & 1ull) o = fmaf(m.gamma, fib_row_max<AM>(v4), R);
      if (lm4) old = ld_val<COH>(ain + (size_t)x * A + a);
      if (has) {
        r = fmax(r, fabs((double)o - (double)old));
        vm = fmax(vm, fabs((double)o));
      }
      sh.out[a * (kWave + 1) + lane] = o;
    }
    __syncthreads();
    // ---- a value per thread, rows contiguous
    const int c = threadIdx.x / A, ca = threadIdx.x - c * A, xc = sh.cell[c];
    if (xc >= 0) st_val<COH>(aout + (size_t)xc * A + ca, sh.out[ca * (kWave + 1) + c]);
    if (more) __syncthreads();
  }
}

// The blind-policy right-hand side at free cell x for every action: each
// action's own vector, alpha^a(x) = R(x,a) + gamma sum_x' T(x,a,x') alpha^a(x')
// (no max over actions: the value of taking a forever, a lower bound).
template <int AM, bool COH>
__device__ __forceinline__ void blind_cell(const DevModel &m, const SlipLanes &sl,
                                           const uint32_t *sig,
                                           const float *staytab, const float *al, int x,
                                           uint32_t sg, float (&out)[AM]) {
  const int A = m.A, W = m.W;
  if (sg & kSigGoal) {
#pragma unroll
    for (int a = 0; a < AM; ++a)
      out[a] = a < A ? fmaf(m.gamma, ld_val<COH>(al + (size_t)x * A + a),
                            m.R[(size_t)x * A + a])
                     : 0.f;
    return;
  }
  const int pat = (int)sig_out8(sg);
  float acc[AM];
#pragma unroll
  for (int a = 0; a < AM; ++a) acc[a] = 0.f;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const bool ok = (k == 4) || ((sg >> (k < 4 ? k : k - 1)) & 1u);
    const int t = ok ? x + (k / 3 - 1) * W + (k % 3 - 1) : x;
#pragma unroll
    for (int a = 0; a < AM; ++a) {
      if (a >= A) continue;
      const float av = ld_val<COH>(al + (size_t)t * A + a);
      const float tk = k == 4 ? staytab[a * 256 + pat] : sl.at(a, k);
      acc[a] = fmaf(tk, ok ? av : 0.f, acc[a]);
    }
  }
#pragma unroll
  for (int a = 0; a < AM; ++a)
    out[a] = a < A ? fmaf(m.gamma, acc[a], m.R[(size_t)x * A + a]) : 0.f;
}

// One blind-bound sweep over the cells blockIdx.x * kBlock + threadIdx.x + j * stride.
template <int AM, bool COH>
__device__ __forceinline__ void blind_pass(const DevModel &m, const SlipLanes &sl,
                                           const uint32_t *sig,
                                           const float *staytab, const float *ain, float *aout,
                                           long long stride, double &r, double &vm) {
  const int A = m.A;
  for (long long x = (long long)blockIdx.x * kBlock + threadIdx.x; x < m.S; x += stride) {
    const uint32_t sg = sig[x];
    float o[AM];
    if (sg & kSigFree) {
      blind_cell<AM, COH>(m, sl, sig, staytab, ain, (int)x, sg, o);
#pragma unroll
      for (int a = 0; a < AM; ++a) {
        if (a >= A) continue;
        r = fmax(r, fabs((double)o[a] - (double)ld_val<COH>(ain + x * A + a)));
        vm = fmax(vm, fabs((double)o[a]));
      }
    } else {
#pragma unroll
      for (int a = 0; a < AM; ++a) o[a] = 0.f;
    }
#pragma unroll
    for (int a = 0; a < AM; ++a)
      if (a < A) st_val<COH>(aout + x * A + a, o[a]);
  }
}

// Sweeps k = 1, 2, .. of a cooperative solve: SWEEP(k, in, out, r, vm) does
// one; x0 holds 0, sweep k writes x[k & 1].  Returns the last sweep, or 0 if a
// barrier wait gave up.
template <class SWEEP>
__device__ __forceinline__ int coop_sweeps(const SweepCtl &c, float *x0, float *x1, double *red,
                                           int *s_stop, SWEEP sweep) {
  if (threadIdx.x == 0) *s_stop = 0;
  for (int k = 1; k <= c.max_sweeps; ++k) {
    double r = 0.0, vm = 0.0;
    sweep((k & 1) ? x0 : x1, (k & 1) ? x1 : x0, r, vm);
    sweep_part_store(c, k, r, vm, red);
    grid_sync(c.bar, (unsigned long long)k * gridDim.x, c.abort);
    if (threadIdx.x < kWave) {
      const int conv = sweep_part_decide(c, k);
      if (threadIdx.x == 0)
        *s_stop = __hip_atomic_load(c.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? 2
                                                                                         : conv;
    }
    __syncthreads();
    if (*s_stop) return *s_stop == 2 ? 0 : k;   // the same decision in every workgroup
  }
  return c.max_sweeps;
}

// The last sweep's values to `out`, its number and residual to the host's words.
__device__ __forceinline__ void coop_result(const SweepCtl &c, int kend, const float *x0,
                                            const float *x1, float *out, long long n) {
  const float *last = (kend & 1) ? x1 : x0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    out[i] = ld_val<true>(last + i);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *c.out_k = kend;
    *c.out_res = load_bits(c.res + kend);
  }
}

// Every FIB sweep in one launch (cooperative); 64 threads per action.
template <int AM, int NJ, bool FULL>
__global__ __launch_bounds__(AM * kWave) void k_fib_coop(DevModel m, FibCells fc,
                                                         const float *staytab, float *al0,
                                                         float *al1, float *out, SweepCtl c) {
  __shared__ FibShared<AM> sh;
  __shared__ double red[2 * kMaxWaves];
  __shared__ int s_stop;
  const int a = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const FibMoves<NJ, FULL> mv(SlipLanes(m), a);
  fib_tables<AM>(m, staytab, sh);
  const bool rvec = m.A == AM && (reinterpret_cast<uintptr_t>(m.R) & 15u) == 0;
  FibRows<AM> f;
  fib_cells_load<AM>(fc, blockIdx.x, f);
  __syncthreads();
  const int kend = coop_sweeps(c, al0, al1, red, &s_stop,
                               [&](const float *in, float *o, double &r, double &vm) {
    fib_rows_load<AM, true>(m, a, in, false, rvec, f);
    fib_pass<AM, NJ, FULL, true>(m, fc, mv, sh, a, in, o, false, rvec, f, r, vm);
  });
  if (kend) coop_result(c, kend, al0, al1, out, (long long)m.S * m.A);
}

// Per-sweep form of sweep k (nothing once the rule has fired).
template <int AM, int NJ, bool FULL>
__global__ __launch_bounds__(AM * kWave, NJ == 4 ? 4 : 2) void k_fib_sweep(DevModel m, FibCells fc,
                                                          const float *staytab, const float *ain,
                                                          float *aout, int k, SweepCtl c) {
  __shared__ FibShared<AM> sh;
  __shared__ double red[2 * kMaxWaves];
  const int a = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const bool vec = m.A == AM, rvec = vec && (reinterpret_cast<uintptr_t>(m.R) & 15u) == 0;
  FibRows<AM> f;
  fib_cells_load<AM>(fc, blockIdx.x, f);
  fib_tables<AM>(m, staytab, sh);
  const FibMoves<NJ, FULL> mv(SlipLanes(m), a);
  fib_rows_load<AM, false>(m, a, ain, vec, rvec, f);   // (in flight during the check)
  if (sweep_stopped(c, k, red)) return;
  double r = 0.0, vm = 0.0;
  fib_pass<AM, NJ, FULL, false>(m, fc, mv, sh, a, ain, aout, vec, rvec, f, r, vm);
  sweep_part_store(c, k, r, vm, red);
}

// The blind bound, in the same two forms.
template <int AM>
__global__ __launch_bounds__(kBlock) void k_blind_coop(DevModel m, const uint32_t *sig,
                                                       const float *staytab, float *al0,
                                                       float *al1, float *out, SweepCtl c) {
  __shared__ double red[2 * kMaxWaves];
  __shared__ int s_stop;
  const SlipLanes sl(m);
  const int kend = coop_sweeps(c, al0, al1, red, &s_stop,
                               [&](const float *in, float *o, double &r, double &vm) {
    blind_pass<AM, true>(m, sl, sig, staytab, in, o, (long long)gridDim.x * kBlock, r, vm);
  });
  if (kend) coop_result(c, kend, al0, al1, out, (long long)m.S * m.A);
}

template <int AM>
__global__ __launch_bounds__(kBlock) void k_blind_sweep(DevModel m, const uint32_t *sig,
                                                        const float *staytab, const float *ain,
                                                        float *aout, int k, SweepCtl c) {
  __shared__ double red[2 * kMaxWaves];
  const SlipLanes sl(m);
  if (sweep_stopped(c, k, red)) return;
  double r = 0.0, vm = 0.0;
  blind_pass<AM, false>(m, sl, sig, staytab, ain, aout, (long long)gridDim.x * kBlock, r, vm);
  sweep_part_store(c, k, r, vm, red);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

// Workspace: sig [S], staytab [A][256], two value buffers of `vals` floats,
// res and vmax [max_sweeps + 2], then barrier counter, residual and sweep
// count, error word.
static size_t sweep_ws(long long S, int A, long long vals, int max_sweeps) {
  size_t off = 0;
  off += align_up((size_t)S * 4, 256);
  off += align_up((size_t)A * 256 * 4, 256);
  off += 2 * align_up((size_t)vals * 4, 256);
  off += 2 * align_up((size_t)(max_sweeps + 2) * 8, 256);
  off += 256;   // barrier counter, residual, sweep count
  off += 256;   // error word
  off += align_up((size_t)4 * kMaxCoopGrid * 8, 256);   // per-workgroup residual partials
  return off;
}

// Regions of a value iteration, and its residual slots behind the sweep
// workspace.
static int vi_regions_x(int W) { return (W + kViOutX - 1) / kViOutX; }
static int vi_regions(int W, int H) {
  return vi_regions_x(W) * ((H + kViOutY - 1) / kViOutY);
}

size_t vi_ws(const qv_model *m, int max_sweeps) {
  const long long S = (long long)m->W * m->H;
  return sweep_ws(S, m->A, S, max_sweeps) +
         align_up((size_t)2 * kViRim * vi_regions(m->W, m->H) * 8, 256);
}

// The FIB solve's sorted cells lie behind the sweep workspace.
static int fib_blocks(long long S) { return (int)((S + kBlock - 1) / kBlock); }
static FibCells fib_cells(char *p, long long S, size_t *bytes) {
  FibCells f;
  size_t off = 0;
  f.cells = (int32_t *)(p + off);
  off += align_up((size_t)S * 4, 256);
  f.recs = (uint64_t *)(p + off);
  off += align_up((size_t)S * 8, 256);
  f.counts = (int32_t *)(p + off);
  off += align_up((size_t)kFibClasses * fib_blocks(S) * 4, 256);
  f.ctl = (int32_t *)(p + off);
  off += 256;
  f.nfree = 0;
  if (bytes) *bytes = off;
  return f;
}

size_t fib_ws(const qv_model *m, int max_sweeps) {
  const long long S = (long long)m->W * m->H;
  size_t bytes;
  fib_cells(nullptr, S, &bytes);
  return sweep_ws(S, m->A, S * m->A, max_sweeps) + bytes;
}

struct SweepWs {
  uint32_t *sig;
  float *staytab;
  float *x[2];
  int32_t *err;
  SweepCtl c;
};

static SweepWs carve(const DevModel &m, long long vals, int max_sweeps, float tol, char *ws) {
  SweepWs w;
  size_t off = 0;
  w.sig = (uint32_t *)(ws + off);
  off += align_up((size_t)m.S * 4, 256);
  w.staytab = (float *)(ws + off);
  off += align_up((size_t)m.A * 256 * 4, 256);
  for (int i = 0; i < 2; ++i) {
    w.x[i] = (float *)(ws + off);
    off += align_up((size_t)vals * 4, 256);
  }
  w.c.res = (unsigned long long *)(ws + off);
  off += align_up((size_t)(max_sweeps + 2) * 8, 256);
  w.c.vmax = (unsigned long long *)(ws + off);
  off += align_up((size_t)(max_sweeps + 2) * 8, 256);
  w.c.bar = (unsigned long long *)(ws + off);
  w.c.out_res = (double *)(ws + off + 8);
  w.c.out_k = (int *)(ws + off + 16);
  w.c.abort = (unsigned int *)(ws + off + 20);
  w.c.arrive = (unsigned int *)(ws + off + 24);
  w.c.stop = (unsigned int *)(ws + off + 28);
  off += 256;
  w.err = (int32_t *)(ws + off);
  off += 256;
  w.c.part = (double *)(ws + off);
  w.c.max_sweeps = max_sweeps;
  w.c.tol = (double)tol;
  return w;
}

// Map signature, stay table, cleared records and both value buffers 0 (x_0,
// and the blocked cells' values, which a FIB sweep does not write).
static hipError_t sweep_setup(const DevModel &m, const SweepWs &w, long long vals,
                              hipStream_t st) {
  hipError_t e = launch_prep(m, w.sig, w.staytab, w.err, st);
  if (e != hipSuccess) return e;
  const long long n = std::max<long long>(w.c.max_sweeps + 2, vals);
  QV_LAUNCH(k_sweep_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, w.c.res,
            w.c.vmax, w.c.max_sweeps + 2, w.c.bar, w.x[0], w.x[1], vals);
  return hipGetLastError();
}

// Blind bound: grids up to this many cells take the one-launch form; larger
// ones the per-sweep launches.  Measured (a sweep, one launch vs per sweep):
// 262144 cells 162 vs 46 us -- at that size the coherent loads of the gathered
// values (past the L2) cost more than the launches they save; 40 sweeps of
// 16384 cells 750 us in one launch, of 16512 by sweep 665.
constexpr long long kCoopMaxCells = 16384;
// FIB, by cells times actions, a solve, one launch / per sweep: 64x64x8 1.11 /
// 1.31 ms, 100x40x9 2.50 / 3.24, 512x30x8 3.28 / 2.83, 128x128x8 2.62 / 2.38;
// and by cells, since the barrier waits for a workgroup per 64 of them: 40
// sweeps of 110x110, 2 and 4 actions, 0.61 / 0.61 and 0.64 / 0.61 ms, of 140x140
// 0.75 / 0.63 and 0.81 / 0.63.
constexpr long long kFibCoopMaxValues = 65536, kFibCoopMaxCells = 12288;

// Workgroups of a cooperative launch of `kernel`: at most `want`, and no
// more than can be resident at once; 0 for the per-sweep form: a `size`
// (cells, or values) above `most`, no cooperative launch on this device, or
// QVTS_SWEEP_LAUNCHES=1.  QVTS_SWEEP_COOP=1 takes the one-launch form at
// any size.
static int coop_grid(const void *kernel, int threads, size_t lds, int want, long long size,
                     long long most) {
  const char *e = std::getenv("QVTS_SWEEP_LAUNCHES");
  if (e && std::atoi(e) == 1) return 0;
  const char *f = std::getenv("QVTS_SWEEP_COOP");
  if (!(f && std::atoi(f) == 1) && size > most) return 0;
  int dev = 0, coop = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess ||
      !coop)
    return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, lds) != hipSuccess ||
      per < 1)
    return 0;
  return std::max(1, std::min(std::min(want, per * cus), kMaxCoopGrid));
}

// Workgroups of `kernel` that are resident at once on the device.
static int resident_grid(const void *kernel, int threads, size_t lds) {
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, lds) != hipSuccess)
    return kSweepGrid;
  return std::max(1, per * cus);
}

// Residual and sweep count of a cooperative solve (one wait); a barrier
// wait that gave up is reported as a launch time-out.
static hipError_t read_result(const SweepWs &w, double *residual, int *sweeps,
                              hipStream_t st) {
  unsigned char buf[16];
  hipError_t e = hipMemcpyAsync(buf, w.c.out_res, 16, hipMemcpyDeviceToHost, st);
  if (e != hipSuccess) return e;
  e = hipStreamSynchronize(st);
  if (e != hipSuccess) return e;
  unsigned int aborted;
  memcpy(residual, buf, 8);
  memcpy(sweeps, buf + 8, 4);
  memcpy(&aborted, buf + 12, 4);
  return aborted ? hipErrorLaunchTimeOut : hipSuccess;
}

// Per-sweep form: `launch(k, in, out)` enqueues sweep k on g workgroups; every
// kViChunk sweeps the host reads the chunk's residuals and stops at the first sweep
// that meets the rule.  Returns the last sweep in *sweeps.
template <class F>
static hipError_t sweep_chunks(const SweepWs &w, int g, F launch, double *residual, int *sweeps,
                               hipStream_t st) {
  std::vector<unsigned long long> hres(kViChunk), hvm(kViChunk);
  const int max_sweeps = w.c.max_sweeps;
  int done = 0;
  hipError_t e;
  for (int k0 = 1; k0 <= max_sweeps && !done; k0 += kViChunk) {
    const int k1 = std::min(max_sweeps, k0 + kViChunk - 1);
    for (int k = k0; k <= k1; ++k) launch(k, w.x[(k - 1) & 1], w.x[k & 1]);
    QV_LAUNCH(k_sweep_close, dim3(1), dim3(kBlock), 0, st, w.c, k1, g);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int cnt = k1 - k0 + 1;
    e = hipMemcpyAsync(hres.data(), w.c.res + k0, cnt * 8, hipMemcpyDeviceToHost, st);
    if (e != hipSuccess) return e;
    e = hipMemcpyAsync(hvm.data(), w.c.vmax + k0, cnt * 8, hipMemcpyDeviceToHost, st);
    if (e != hipSuccess) return e;
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return e;
    for (int i = 0; i < cnt; ++i) {
      double r, vm;
      memcpy(&r, &hres[i], 8);
      memcpy(&vm, &hvm[i], 8);
      *residual = r;
      *sweeps = k0 + i;
      if (r == 0.0 || r <= w.c.tol * std::max(1.0, vm)) {
        done = 1;
        break;
      }
    }
  }
  return hipSuccess;
}

template <int AM>
static hipError_t run_vi_am(const DevModel &m, const SweepWs &w, double *slots, float *Q,
                            double *residual, int *sweeps, hipStream_t st) {
  const int max_sweeps = w.c.max_sweeps;
  // the environment's switch to single sweeps, as in the other solves
  const char *e1 = std::getenv("QVTS_SWEEP_LAUNCHES");
  const bool single = e1 && std::atoi(e1) == 1;
  if (!single && m.W <= kViX && m.H <= kViY) {
    QV_LAUNCH((k_vi<AM, kViSolveMode>), dim3(1), dim3(kViBlock), 0, st, m, w.sig, w.staytab, 1,
              w.x[0], w.x[1], Q, 0, max_sweeps, slots, w.c);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : read_result(w, residual, sweeps, st);
  }
  const int rx = vi_regions_x(m.W), G = vi_regions(m.W, m.H), step = single ? 1 : kViRim;
  std::vector<unsigned long long> hres(kViChunk), hvm(kViChunk);
  hipError_t e;
  bool done = false;
  int kc = 0;
  for (int k0 = 0; k0 < max_sweeps && !done; k0 += kViChunk) {
    const int k1 = std::min(max_sweeps, k0 + kViChunk);
    for (int k = k0; k < k1; k += step)   // block b reads x[b & 1] and writes the other
      QV_LAUNCH((k_vi<AM, kViBlockMode>), dim3(G), dim3(kViBlock), 0, st, m, w.sig, w.staytab, rx,
                w.x[(k / step) & 1], w.x[(k / step + 1) & 1], Q, k, std::min(step, k1 - k), slots,
                w.c);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int cnt = k1 - k0;
    e = hipMemcpyAsync(hres.data(), w.c.res + k0 + 1, cnt * 8, hipMemcpyDeviceToHost, st);
    if (e != hipSuccess) return e;
    e = hipMemcpyAsync(hvm.data(), w.c.vmax + k0 + 1, cnt * 8, hipMemcpyDeviceToHost, st);
    if (e != hipSuccess) return e;
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return e;
    for (int i = 0; i < cnt && !done; ++i) {
      double r, vm;
      memcpy(&r, &hres[i], 8);
      memcpy(&vm, &hvm[i], 8);
      *residual = r;
      kc = k0 + i + 1;
      done = r == 0.0 || r <= w.c.tol * std::max(1.0, vm);
    }
  }
  *sweeps = kc;
  // Q of sweep kc, from the start of its block
  const int b = (kc - 1) / step;
  QV_LAUNCH((k_vi<AM, kViTableMode>), dim3(G), dim3(kViBlock), 0, st, m, w.sig, w.staytab, rx,
            w.x[b & 1], w.x[(b + 1) & 1], Q, b * step, kc - 1 - b * step, slots, w.c);
  e = hipGetLastError();
  return e != hipSuccess ? e : hipStreamSynchronize(st);
}

hipError_t run_value_iteration(const DevModel &m, float tol, int max_sweeps, float *Q,
                               double *residual, int *sweeps, char *ws, hipStream_t st) {
  const SweepWs w = carve(m, m.S, max_sweeps, tol, ws);
  const hipError_t e = sweep_setup(m, w, m.S, st);
  if (e != hipSuccess) return e;
  double *slots = (double *)(ws + sweep_ws(m.S, m.A, m.S, max_sweeps));
  if (m.A <= 4) return run_vi_am<4>(m, w, slots, Q, residual, sweeps, st);
  if (m.A <= 8) return run_vi_am<8>(m, w, slots, Q, residual, sweeps, st);
  return run_vi_am<9>(m, w, slots, Q, residual, sweeps, st);
}

template <class F>
static hipError_t coop_solve(const SweepWs &w, const char *name, const void *kernel, int G,
                             int threads, F args_of, double *residual, int *sweeps,
                             hipStream_t st) {
  hipError_t e;
  {
    TimingScope ts(name, st);
    e = args_of([&](void **args) {
      return hipLaunchCooperativeKernel(kernel, dim3(G), dim3(threads), args, 0u, st);
    });
  }
  if (e != hipSuccess) return e;
  return read_result(w, residual, sweeps, st);
}

// alpha after a per-sweep solve.
static hipError_t sweep_copy(const SweepWs &w, float *alpha, long long vals, int sweeps,
                             hipStream_t st) {
  const hipError_t e =
      hipMemcpyAsync(alpha, w.x[sweeps & 1], (size_t)vals * 4, hipMemcpyDeviceToDevice, st);
  return e != hipSuccess ? e : hipStreamSynchronize(st);
}

template <int AM, int NJ, bool FULL>
static hipError_t run_fib_am(const DevModel &m, const SweepWs &w, FibCells fc, float *alpha,
                             double *residual, int *sweeps, hipStream_t st) {
  const int nb = fib_blocks(m.S);
  QV_LAUNCH(k_fib_count, dim3(nb), dim3(kBlock), 0, st, m, w.sig, fc.counts);
  QV_LAUNCH(k_fib_scan, dim3(1), dim3(1024), 0, st, fc.counts, kFibClasses * nb, fc.ctl);
  QV_LAUNCH(k_fib_scatter, dim3(nb), dim3(kBlock), 0, st, m, w.sig, fc.counts, fc.cells, fc.recs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the count as a launch argument: a sweep then starts with its cells
  e = hipMemcpyAsync(&fc.nfree, fc.ctl, 4, hipMemcpyDeviceToHost, st);
  if (e != hipSuccess) return e;
  e = hipStreamSynchronize(st);
  if (e != hipSuccess) return e;
  const int threads = m.A * kWave;
  const int want = std::max(1, (fc.nfree + kWave - 1) / kWave);
  const void *coop = reinterpret_cast<const void *>(&k_fib_coop<AM, NJ, FULL>);
  const long long size = (long long)m.S * std::max<long long>(
      m.A, m.S > kFibCoopMaxCells ? kFibCoopMaxValues : 0);
  const int G = coop_grid(coop, threads, 0, want, size, kFibCoopMaxValues);
  if (G > 0) {
    DevModel mm = m;
    const float *stay = w.staytab;
    float *a0 = w.x[0], *a1 = w.x[1];
    SweepCtl c = w.c;
    return coop_solve(
        w, "k_fib_coop", coop, G, threads,
        [&](auto launch) {
          void *args[] = {&mm, &fc, &stay, &a0, &a1, &alpha, &c};
          return launch(args);
        },
        residual, sweeps, st);
  }
  // as many workgroups as are resident at once: they take the groups in turn,
  // and a part-filled second round would cost as much as the first (512x512,
  // a sweep: 1024 workgroups 34.9 us, 768 32.2, the resident 512 25.7)
  const int g = std::min(want, std::min(kFibGrid, resident_grid(
      reinterpret_cast<const void *>(&k_fib_sweep<AM, NJ, FULL>), threads, 0)));
  e = sweep_chunks(
      w, g,
      [&](int k, float *in, float *out) {
        QV_LAUNCH((k_fib_sweep<AM, NJ, FULL>), dim3(g), dim3(threads), 0, st, m, fc, w.staytab, in, out,
                  k, w.c);
      },
      residual, sweeps, st);
  if (e != hipSuccess) return e;
  return sweep_copy(w, alpha, (long long)m.S * m.A, *sweeps, st);
}

template <int AM>
static hipError_t run_blind_am(const DevModel &m, const SweepWs &w, float *alpha,
                               double *residual, int *sweeps, hipStream_t st) {
  const int want = fib_blocks(m.S);
  const void *coop = reinterpret_cast<const void *>(&k_blind_coop<AM>);
  const int G = coop_grid(coop, kBlock, 0, want, m.S, kCoopMaxCells);
  if (G > 0) {
    DevModel mm = m;
    const uint32_t *sig = w.sig;
    const float *stay = w.staytab;
    float *a0 = w.x[0], *a1 = w.x[1];
    SweepCtl c = w.c;
    return coop_solve(
        w, "k_blind_coop", coop, G, kBlock,
        [&](auto launch) {
          void *args[] = {&mm, &sig, &stay, &a0, &a1, &alpha, &c};
          return launch(args);
        },
        residual, sweeps, st);
  }
  const int g = std::min(want, kSweepGrid);
  const hipError_t e = sweep_chunks(
      w, g,
      [&](int k, float *in, float *out) {
        QV_LAUNCH((k_blind_sweep<AM>), dim3(g), dim3(kBlock), 0, st, m, w.sig, w.staytab, in, out,
                  k, w.c);
      },
      residual, sweeps, st);
  if (e != hipSuccess) return e;
  return sweep_copy(w, alpha, (long long)m.S * m.A, *sweeps, st);
}

// op 0: the FIB equation; op 1: the blind-policy equation.
hipError_t run_fib(const DevModel &m, float tol, int max_sweeps, float *alpha,
                   double *residual, int *sweeps, char *ws, hipStream_t st, int op) {
  const long long vals = (long long)m.S * m.A;
  const SweepWs w = carve(m, vals, max_sweeps, tol, ws);
  const FibCells fc = fib_cells(ws + sweep_ws(m.S, m.A, vals, max_sweeps), m.S, nullptr);
  hipError_t e = sweep_setup(m, w, vals, st);
  if (e != hipSuccess) return e;
  // (with one action there is no maximum to take, and the FIB equation is the
  // blind one; 300x300, 40 sweeps: 1.06 ms by the FIB kernels, 0.40 so)
  if (op == 1 || m.A == 1) {
    if (m.A <= 4) return run_blind_am<4>(m, w, alpha, residual, sweeps, st);
    if (m.A <= 8) return run_blind_am<8>(m, w, alpha, residual, sweeps, st);
    return run_blind_am<9>(m, w, alpha, residual, sweeps, st);
  }
  // the rows a wavefront holds: its own cell's and one per move with a
  // probability, by the action with most (three in the package's slip tables)
  int most = 0, least = 8;
  for (int a = 0; a < m.A; ++a) {
    int n = 0;
    for (int k = 0; k < 9; ++k) n += k != 4 && m.slip[a * 9 + k] != 0.f;
    most = std::max(most, n);
    least = std::min(least, n);
  }
  const bool few = most <= 4, full = least == 8;
  if (m.A <= 4)
    return few    ? run_fib_am<4, 4, false>(m, w, fc, alpha, residual, sweeps, st)
           : full ? run_fib_am<4, 8, true>(m, w, fc, alpha, residual, sweeps, st)
                  : run_fib_am<4, 8, false>(m, w, fc, alpha, residual, sweeps, st);
  if (m.A <= 8)
    return few    ? run_fib_am<8, 4, false>(m, w, fc, alpha, residual, sweeps, st)
           : full ? run_fib_am<8, 8, true>(m, w, fc, alpha, residual, sweeps, st)
                  : run_fib_am<8, 8, false>(m, w, fc, alpha, residual, sweeps, st);
  return few    ? run_fib_am<9, 4, false>(m, w, fc, alpha, residual, sweeps, st)
         : full ? run_fib_am<9, 8, true>(m, w, fc, alpha, residual, sweeps, st)
                : run_fib_am<9, 8, false>(m, w, fc, alpha, residual, sweeps, st);
}

}  // namespace qv
