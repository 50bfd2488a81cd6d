// qv_filter.hip -- batched Bayes filter step on gfx950 (Sec. III, posterior
// belief update): prediction through the slip stencil, the likelihood of
// the given observation, and normalisation.  Two passes over bands of rows:
// the first reduces P(z|b,a) per (belief, band) into the workspace, the
// second sums those partials in band order and writes the posterior.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "qv_internal.h"

namespace qv {

// Rows y0-1 .. y0+th of b into LDS; off-grid, blocked and goal cells are zero
// (none of them sends mass to a neighbour).
__device__ __forceinline__ void load_fband(const DevModel &m, const uint32_t *sig,
                                           const float *b, int y0, int th, float *band,
                                           int BW) {
  const int n = (th + 2) * BW;
  const float rBW = 1.0f / (float)BW;
  for (int i = threadIdx.x; i < n; i += kBlock) {
    const int r = fdiv(i, BW, rBW);
    const int gy = y0 - 1 + r, gx = i - r * BW - 1;
    float v = 0.f;
    if (gy >= 0 && gy < m.H && gx >= 0 && gx < m.W) {
      const int s = gy * m.W + gx;
      if ((sig[s] & (kSigFree | kSigGoal)) == kSigFree) v = b[s];
    }
    band[i] = v;
  }
}

__device__ __forceinline__ float fpredict(const DevModel &m, const float *band, int BW, int ly,
                                          int lx, uint32_t sg, const float *sl,
                                          const float *stay_a, const float *b, int t) {
  if (!(sg & kSigFree)) return 0.f;
  const float *c = band + (ly + 1) * BW + lx + 1;
  if (sg & kSigGoal) return stencil(c, BW, sl, 1.f, b[t]);
  return stencil(c, BW, sl, stay_a[sig_out8(sg)], c[0]);
}

__device__ __forceinline__ bool bu_item_ok(const DevModel &m, int a, int z) {
  return a >= 0 && a < m.A && z >= 0 && z < 16 * (m.L + 1);
}

__global__ __launch_bounds__(kBlock) void k_bu_lik(DevModel m, const uint32_t *sig,
                                                   const float *staytab, int TH, int tiles,
                                                   const float *b, const int32_t *acts,
                                                   const int32_t *obs, float *part,
                                                   int32_t *err) {
  extern __shared__ float smem[];
  __shared__ float red[kBlock / kWave];
  const int item = blockIdx.x / tiles, tile = blockIdx.x - item * tiles;
  const int a = acts[item], z = obs[item];
  if (!bu_item_ok(m, a, z)) {
    if (tile == 0 && threadIdx.x == 0) atomicOr(err, 4);
    return;
  }
  const int W = m.W, BW = W + 2;
  const int y0 = tile * TH, th = min(TH, m.H - y0);
  const float *bi = b + (size_t)item * m.S;
  float *band = smem;
  load_fband(m, sig, bi, y0, th, band, BW);
  __syncthreads();
  const float rW = 1.0f / (float)W;
  const float *sl = &m.slip[a * 9];
  const float *stay_a = staytab + a * 256;
  const uint32_t zw = (uint32_t)(z & 15), zl = (uint32_t)(z >> 4);
  float acc = 0.f;
  for (int i = threadIdx.x; i < th * W; i += kBlock) {
    const int ly = fdiv(i, W, rW), lx = i - ly * W;
    const int t = (y0 + ly) * W + lx;
    const uint32_t sg = sig[t];
    const float bp = fpredict(m, band, BW, ly, lx, sg, sl, stay_a, bi, t);
    const float o = wall_lik(m.flip, zw, sig_wall(sg)) * lm_lik(m.lm_p, zl, sig_lm(sg));
    acc = fmaf(o, bp, acc);
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    float s = 0.f;
    for (int w = 0; w < kBlock / kWave; ++w) s += red[w];
    part[(size_t)item * tiles + tile] = s;
  }
}

__global__ __launch_bounds__(kBlock) void k_bu_write(DevModel m, const uint32_t *sig,
                                                     const float *staytab, int TH, int tiles,
                                                     const float *b, const int32_t *acts,
                                                     const int32_t *obs, const float *part,
                                                     float *b_out, float *p_out,
                                                     int32_t *err) {
  extern __shared__ float smem[];
  const int item = blockIdx.x / tiles, tile = blockIdx.x - item * tiles;
  const int a = acts[item], z = obs[item];
  if (!bu_item_ok(m, a, z)) {
    if (tile == 0 && threadIdx.x == 0) p_out[item] = 0.f;
    return;
  }
  float p = 0.f;
  for (int t = 0; t < tiles; ++t) p += part[(size_t)item * tiles + t];
  if (tile == 0 && threadIdx.x == 0) {
    p_out[item] = p;
    if (!(p > 0.f)) atomicOr(err, 8);
  }
  if (!(p > 0.f)) return;
  const float inv = 1.0f / p;
  const int W = m.W, BW = W + 2;
  const int y0 = tile * TH, th = min(TH, m.H - y0);
  const float *bi = b + (size_t)item * m.S;
  float *band = smem;
  load_fband(m, sig, bi, y0, th, band, BW);
  __syncthreads();
  const float rW = 1.0f / (float)W;
  const float *sl = &m.slip[a * 9];
  const float *stay_a = staytab + a * 256;
  const uint32_t zw = (uint32_t)(z & 15), zl = (uint32_t)(z >> 4);
  float *bo = b_out + (size_t)item * m.S;
  for (int i = threadIdx.x; i < th * W; i += kBlock) {
    const int ly = fdiv(i, W, rW), lx = i - ly * W;
    const int t = (y0 + ly) * W + lx;
    const uint32_t sg = sig[t];
    const float bp = fpredict(m, band, BW, ly, lx, sg, sl, stay_a, bi, t);
    const float o = wall_lik(m.flip, zw, sig_wall(sg)) * lm_lik(m.lm_p, zl, sig_lm(sg));
    bo[t] = o * bp * inv;
  }
}

size_t belief_update_ws(const qv_model *m, int batch) {
  const size_t S = (size_t)m->W * m->H;
  const int TH = tile_rows(m->W, m->H);
  const int tiles = (m->H + TH - 1) / TH;
  size_t off = 0;
  off += align_up(S * 4, 256);                        // sig
  off += align_up((size_t)m->A * 256 * 4, 256);       // staytab
  off += align_up((size_t)batch * tiles * 4, 256);    // partial likelihoods
  off += 256;                                         // err
  return off;
}

hipError_t launch_belief_update(const DevModel &m, int batch, const float *b,
                                const int32_t *a, const int32_t *z, float *b_out,
                                float *p_out, char *ws, hipStream_t st) {
  const size_t S = (size_t)m.S;
  const int TH = tile_rows(m.W, m.H);
  const int tiles = (m.H + TH - 1) / TH;
  size_t off = 0;
  uint32_t *sig = (uint32_t *)(ws + off);
  off += align_up(S * 4, 256);
  float *staytab = (float *)(ws + off);
  off += align_up((size_t)m.A * 256 * 4, 256);
  float *part = (float *)(ws + off);
  off += align_up((size_t)batch * tiles * 4, 256);
  int32_t *err = (int32_t *)(ws + off);
  hipError_t e = launch_prep(m, sig, staytab, err, st);
  if (e != hipSuccess) return e;
  if (batch == 0) return hipSuccess;
  const size_t lds = (size_t)(TH + 2) * (m.W + 2) * sizeof(float);
  const dim3 grid((unsigned)((size_t)batch * tiles));
  QV_LAUNCH(k_bu_lik, grid, dim3(kBlock), lds, st, m, sig, staytab, TH, tiles, b, a, z,
                     part, err);
  QV_LAUNCH(k_bu_write, grid, dim3(kBlock), lds, st, m, sig, staytab, TH, tiles, b, a,
                     z, part, b_out, p_out, err);
  return hipGetLastError();
}

int32_t belief_update_args(const qv_model *m, int batch, const float *b, const int32_t *a,
                           const int32_t *z, const float *b_out, const float *p_out) {
  const int32_t st = check_model(m);
  if (st != QV_OK) return st;
  if (batch < 0) return QV_ERR_INVALID_ARG;
  if (batch > 0 && (!b || !a || !z || !b_out || !p_out)) return QV_ERR_INVALID_ARG;
  const size_t S = (size_t)m->W * m->H;
  if (batch > 0 && (const void *)b < (const void *)(b_out + (size_t)batch * S) &&
      (const void *)b_out < (const void *)(b + (size_t)batch * S))
    return QV_ERR_INVALID_ARG;
  return QV_OK;
}

int32_t belief_update_run(const qv_model *m, int batch, const float *b, const int32_t *a,
                          const int32_t *z, float *b_out, float *p_out, int check, char *ws,
                          hipStream_t hs) {
  const DevModel dm = make_dev_model(m);
  int32_t st = hip_status(launch_belief_update(dm, batch, b, a, z, b_out, p_out, ws, hs));
  if (st != QV_OK || !check) return st;
  const size_t S = (size_t)m->W * m->H;
  const size_t TH = tile_rows(m->W, m->H);
  const size_t tiles = (m->H + TH - 1) / TH;
  const size_t off = align_up(S * 4, 256) + align_up((size_t)m->A * 256 * 4, 256) +
                     align_up((size_t)batch * tiles * 4, 256);
  int32_t herr = 0;
  st = hip_status(hipMemcpyAsync(&herr, ws + off, 4, hipMemcpyDeviceToHost, hs));
  if (st != QV_OK) return st;
  st = hip_status(hipStreamSynchronize(hs));
  if (st != QV_OK) return st;
  if (herr & (4 | 8)) return QV_ERR_ZERO_LIKELIHOOD;
  if (herr) return QV_ERR_INVALID_ARG;
  return QV_OK;
}

// ---------------------------------------------------------------------------
// Belief update without allocation: the same kernels on a scratch region in
// the library's own device memory instead of a caller workspace.  Each GPU
// holds its own copy of `scratch` for the life of the process; host code
// uses the device address that hipGetSymbolAddress returns for the current
// device, never the array's name (a host-side stand-in).
// ---------------------------------------------------------------------------
constexpr int kBuMaxCells = 1 << 20;     // S = W*H at most
constexpr int kBuMaxParts = 1 << 14;     // batch * bands at most
constexpr size_t kBuScratchBytes =
    ((size_t)kBuMaxCells * 4) + ((size_t)QV_MAX_ACTIONS * 256 * 4 + 256) +
    ((size_t)kBuMaxParts * 4) + 256;
static __device__ __align__(256) char scratch[kBuScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch[kMaxDevices];

// The current device's copy of `scratch` (looked up once per device).
static hipError_t scratch_ptr(char **out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch[dev] = p;
  }
  *out = (char *)g_scratch[dev];
  return hipSuccess;
}

}  // namespace qv

extern "C" int32_t qv_belief_update_noalloc(const qv_model *m, int32_t batch, const float *b,
                                            const int32_t *a, const int32_t *z, float *b_out,
                                            float *p_out, int32_t check, void *stream) {
  using namespace qv;
  const int32_t st = belief_update_args(m, batch, b, a, z, b_out, p_out);
  if (st != QV_OK) return st;
  const long long S = (long long)m->W * m->H;
  const long long TH = tile_rows(m->W, m->H);
  const long long tiles = (m->H + TH - 1) / TH;
  if (S > kBuMaxCells || (long long)batch * tiles > kBuMaxParts) return QV_ERR_UNSUPPORTED;
  if (belief_update_ws(m, batch) > kBuScratchBytes) return QV_ERR_UNSUPPORTED;
  char *ws = nullptr;
  const int32_t hs = hip_status(scratch_ptr(&ws));
  if (hs != QV_OK) return hs;
  return belief_update_run(m, batch, b, a, z, b_out, p_out, check, ws, (hipStream_t)stream);
}

namespace qv {

// ===========================================================================
// Differentiable filter: negative log-likelihood of logged observations under
// the filter above and its adjoint with respect to the slip logits theta
// (T'(a,.) = softmax(theta[a,.])) and the wall-bit flip logits phi
// (f_j = logistic(phi_j)).  For each trajectory
//   c_t = T_{a_t}^T b_{t-1},  eta_t = sum O(z_t|.) c_t,  b_t = O(z_t|.) c_t / eta_t,
//   NLL = -sum_t log eta_t,
// and in reverse, with beta_T = 1 (the adjoint of b_t is -beta_t up to a
// constant that the normalisation takes out, and <beta_t, b_t> = 1):
//   v_t = O(z_t|.) beta_t / eta_t,  beta_{t-1}(s) = sum_k T'(a_t,k) v_t(dest(s,k)),
//   dNLL/dT'(a_t,k) -= sum_s b_{t-1}(s) v_t(dest(s,k)),
//   dNLL/df_j -= sum_s gamma_t(s) (bit j misread ? 1/f_j : -1/(1-f_j)),
//   gamma_t = b_t beta_t.
// All terms of the recursions are non-negative, so they lose no digits.
//
// One persistent workgroup per trajectory at a time.  What bounds it: the
// vector ALU (about 28 instructions per cell and filter step, 57 per reverse
// step) and, on small grids, the barrier and reduction of each step.  Hence:
//  * every thread owns a vertical strip of R cells and keeps their map
//    bits in registers; the 3x3 neighbourhood rolls down the strip, so a
//    cell costs 3 LDS reads instead of 9, and lanes sit side by side in x
//    (no bank conflicts).  The strips run along the longer side of the grid.
//  * beliefs stay unnormalised, u_t = b_t U_t with U_t = sum u_t, rescaled by
//    an exact power of two, and the bands are double-buffered (DB): a step
//    reads one band, writes the other and has one barrier.  (Without room
//    for two bands, DB = false: one band and a second barrier.)  A subnormal
//    U_t (an observation of probability below 1e-38) takes a pass of its own
//    over the band, so that the next step again has all its bits.
//  * the reverse step is one pass over the cells: gather beta_{t-1} and the
//    slip sums from band v_t, the flip sums from gamma_{t-1}, and v_{t-1}
//    into the other band.  A failed move reads the cell itself: blocked and
//    off-grid entries of v hold -1 (v is never negative).
//  * the last segment's beliefs are stored by the forward pass itself; the
//    earlier segments are recomputed from their stored start.
// Stored beliefs are in strip order [row of strip][thread], so their accesses
// are coalesced whatever the strips' direction.  Every sum runs in a fixed
// order that depends on the grid alone.  Measured, NLL + gradient of 1024
// runs x 50 steps on 128x128: 11.6 -> 3.4 ms (one thread per cell,
// two band reads and three barriers a step, before).
// ===========================================================================
constexpr int kFMaxBlock = 1024;
constexpr int kFWaves = kFMaxBlock / kWave;
constexpr int kFGrad = 85;   // 81 slip entries (A*9 used) + 4 flip entries
constexpr int kFSums = 14;   // reverse step: 9 slip sums, gamma by wall bit's rarer reading (4), gamma
constexpr int kFChunk = 256;   // steps whose inputs and sums are held in LDS
constexpr int kFLik = 33;    // likelihood row: wall reading, the same on a landmark, blocked

struct FilterArgs {
  int ntraj, T, k, nseg, G;
  int n1, n2, ng;     // cells across and along the strips, strips along
  int pitch;          // floats from one row of a band to the next, n1 + 2 at least
  int along_x;         // strips run along x (lanes along y)
  const float *theta, *phi;
  const float *b0;
  int b0_per_traj;
  const int32_t *acts, *obs;
  float *nll;         // [ntraj]
  double *gpart;      // [ntraj][kFGrad]
  float *ckpt;        // [G][nseg][R][threads] (entry 0 unused: the start belief)
  float *seg;         // [G][k+1][R][threads]
  float *usum;        // [G][T] U_1, U_2, ..
  const uint32_t *sig;
  int32_t *err;
  int want_grad;
};

// Map bits of a strip's cell: 0..9 byte offset of its stay entry, 10..15 its
// entry of a likelihood row (wall reading in 10..13), 16..24 landmark id,
// 30 free, 31 goal.
constexpr uint32_t kFiFree = 1u << 30, kFiGoal = 1u << 31;
constexpr uint32_t kFiBlocked = 32u << 10;
__device__ __forceinline__ uint32_t filter_info(uint32_t sg) {
  if (!(sg & kSigFree)) return kFiBlocked;
  const uint32_t lm = sig_lm(sg);
  return (sig_out8(sg) << 2) | ((sig_wall(sg) | (lm ? 16u : 0u)) << 10) | (lm << 16) | kFiFree |
         ((sg & kSigGoal) ? kFiGoal : 0u);
}

// Keeps the fields of v packed: without it the compiler unpacks every cell's
// fields once, outside the loop over steps, and spills them.
__device__ __forceinline__ void keep_packed(uint32_t &v) { asm volatile("" : "+v"(v)); }
// Likewise for a running LDS index (not one register per row of the strip).
__device__ __forceinline__ void keep_running(int &v) { asm volatile("" : "+v"(v)); }

struct FilterShared {
  // (the two read as 4-vectors come first, aligned)
  alignas(16) float upart[2][kFWaves];          // per-wavefront sums of u_t, by step parity
  alignas(16) float gpart[2][kFSums][kFWaves];  // per-wavefront reverse sums, by step parity
  float slip[81], flip[4];
  float lik[2][16][kFLik];          // [a landmark id observed][zw][entry]
  double g[81], mis[4], ok[4];
  double red[kFWaves];
  int32_t az[kFChunk];              // action + 256 observation of a chunk of steps
  float u[kFChunk];                 // U of a chunk of steps
};
static_assert(offsetof(FilterShared, upart) % 16 == 0 && offsetof(FilterShared, gpart) % 16 == 0 &&
                  kFWaves % 4 == 0,
              "rows read as 4-vectors");

// O(z|.) of a cell from the step's likelihood row (lk, zl uniform).
template <bool PLAIN>
__device__ __forceinline__ float filter_lik(const float *lk, uint32_t info, uint32_t zl) {
  const float o = lk[(info >> 10) & 63u];
  if constexpr (PLAIN) return o;
  // (bit operations: a short-circuit test became a branch per row of the
  // strip, between which the compiler spilled 200 registers at R = 16; NLL and
  // gradient of 256 runs x 50 steps on 64x64 with landmarks and a goal took
  // 1.28 ms, not 0.50)
  const uint32_t zm = zl ? 0x1FF0000u : 0u;
  return ((info ^ (zl << 16)) & zm) == 0u ? o : 0.f;
}

// Sum of the wavefronts' partials (absent ones are 0), in a fixed order;
// small: at most four wavefronts.
__device__ __forceinline__ float filter_sum_waves(const float *p, bool small) {
  const float4 *q = reinterpret_cast<const float4 *>(p);
  const float4 a = q[0];
  const float sa = (a.x + a.y) + (a.z + a.w);
  if (small) return sa;
  const float4 b = q[1], c = q[2], d = q[3];
  return (sa + ((b.x + b.y) + (b.z + b.w))) +
         (((c.x + c.y) + (c.z + c.w)) + ((d.x + d.y) + (d.z + d.w)));
}

// A step sees the sum U before it as U 2^-k in [1, 2), k = filter_exp(U) (U = 0,
// infinite or NaN: any k).  Below -126, U is subnormal and 2^-k may not be a
// float: the band is lifted by 2^23 first, which takes kFLift off k.
constexpr int kFLift = 23;
__device__ __forceinline__ int filter_exp(float U) {
  return min(__builtin_amdgcn_frexp_expf(U) - 1, 126);
}
__device__ __forceinline__ float filter_scaled(float U) { return ldexpf(U, -filter_exp(U)); }
__device__ __forceinline__ float filter_scale(int k) {
  return __int_as_float((127 - (k < -126 ? k + kFLift : k)) << 23);
}

// Workgroup barrier for LDS alone: stores to global memory stay in flight
// (__syncthreads waits for them; each thread reads back only its own).
// Also where an LDS write of the loop's end meets a barrier at its top: there
// the compiler has left the wait of __syncthreads out.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// PLAIN: the map has neither landmarks nor an absorbing goal.
template <int R, bool DB, bool PLAIN>
__global__ __launch_bounds__(kFMaxBlock) void k_filter(DevModel m, FilterArgs fa) {
  extern __shared__ float smem[];
  __shared__ FilterShared sh;
  const int A = m.A, n1 = fa.n1, n2 = fa.n2, P = fa.pitch;
  const int NT = blockDim.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int band_floats = (fa.ng * R + 2) * P;
  float *band0 = smem, *band1 = DB ? smem + band_floats : smem;
  float *stay = smem + (DB ? 2 : 1) * band_floats;   // [A][256] stay probability of T'
  const int strip = tid / n1, i1 = tid - strip * n1;
  const bool act = strip < fa.ng, small = NT <= 4 * kWave;
  const int j0 = strip * R;
  const int pos = act ? j0 * P + i1 : 0;   // band entry above and left of the strip's first cell
  const size_t SL = (size_t)R * NT;        // floats of a stored belief

  // ---- tables of the evaluation point, and the strip's map bits
  if (tid < A) {
    float mx = -INFINITY;
    for (int k = 0; k < 9; ++k) mx = fmaxf(mx, fa.theta[tid * 9 + k]);
    float e[9], sum = 0.f;
    for (int k = 0; k < 9; ++k) {
      e[k] = expf(fa.theta[tid * 9 + k] - mx);
      sum += e[k];
    }
    for (int k = 0; k < 9; ++k) sh.slip[tid * 9 + k] = e[k] / sum;
  }
  if (tid < 4) sh.flip[tid] = 1.f / (1.f + expf(-fa.phi[tid]));
  if (tid < kFWaves) sh.upart[0][tid] = sh.upart[1][tid] = 0.f;
  for (int i = tid; i < 2 * kFSums * kFWaves; i += NT) (&sh.gpart[0][0][0])[i] = 0.f;
  __syncthreads();
  for (int i = tid; i < A * 256; i += NT) {
    const int a = i >> 8, pat = i & 255;
    float st = sh.slip[a * 9 + 4];
    int bit = 0;
    for (int k = 0; k < 9; ++k) {
      if (k == 4) continue;
      if (!((pat >> bit) & 1)) st += sh.slip[a * 9 + k];
      ++bit;
    }
    stay[i] = st;
  }
  for (int i = tid; i < 2 * 16 * kFLik; i += NT) {
    const int j = i % kFLik, zw = (i / kFLik) & 15, l = i / (16 * kFLik);
    float o = 0.f;
    if (j < 32) {
      o = wall_lik(sh.flip, (uint32_t)zw, (uint32_t)(j & 15));
      o *= l ? ((j & 16) ? m.lm_p : 0.f) : ((j & 16) ? 1.f - m.lm_p : 1.f);
    }
    sh.lik[l][zw][j] = o;
  }
  uint32_t info[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    info[r] = kFiBlocked;
    if (act && j0 + r < n2)
      info[r] = filter_info(fa.sig[fa.along_x ? i1 * m.W + j0 + r : (j0 + r) * m.W + i1]);
  }
  // the goal cell, in its thread: its row of the strip and its own mass (its
  // entry of a belief band is 0: it sends none to its neighbours)
  int rgoal = -1;
  float gown = 0.f;
  if constexpr (!PLAIN) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (info[r] & kFiGoal) rgoal = r;
  }
  __syncthreads();

  float *ckpt = fa.ckpt + (size_t)blockIdx.x * fa.nseg * SL;
  float *segb = fa.seg + (size_t)blockIdx.x * (fa.k + 1) * SL;
  float *usum = fa.usum + (size_t)blockIdx.x * fa.T;

  // Flip sums: per wall bit gamma is summed over the cells with the rarer
  // reading (misread, or with f_j > 1/2 rightly read: bits of `rare`); the other
  // reading has the rest.  The other way round, the rare one would be a
  // difference of two sums, with their rounding and not its own.
  uint32_t rare = 0u;
#pragma unroll
  for (int i = 0; i < 4; ++i) rare |= sh.flip[i] > 0.5f ? 1u << i : 0u;
  rare = __builtin_amdgcn_readfirstlane(rare);

  // slip weight of the move by d2 along and d1 across the strips: lane
  // 3 a + d1 + 1 of register d2 + 1 holds it
  float slr[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int la = min(lane / 3, A - 1), j = lane % 3;
    slr[i] = sh.slip[la * 9 + (fa.along_x ? j * 3 + i : i * 3 + j)];
  }
  auto slip_at = [&](int a, int d2, int d1) {
    return __int_as_float(
        __builtin_amdgcn_readlane(__float_as_int(slr[d2 + 1]), a * 3 + d1 + 1));
  };
  auto fill = [&](float v) {   // every entry of both bands
    for (int i = tid; i < band_floats; i += NT) {
      band0[i] = v;
      if (DB) band1[i] = v;
    }
  };
  // One filter step from band x to band y: u_t = O c(u_{t-1}) s, stored to dst
  // too with STORE.  Leaves the wavefronts' sums in upart[par]; a barrier
  // follows in the caller.
  auto fstep = [&](auto STORE, const float *x, float *y, int a, int z, float s, float *dst,
                   int par) {
    // gather form: mass from the neighbour at (d2, d1) moved by (-d2, -d1)
    float w[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) w[q] = slip_at(a, 1 - q / 3, 1 - q % 3);
    const char *sa = reinterpret_cast<const char *>(stay + a * 256);
    const uint32_t zl = (uint32_t)(z >> 4);
    const float *lk = sh.lik[zl ? 1 : 0][z & 15];
    float tot = 0.f;
    float ub[DB ? 1 : R];
    if (act) {
      int o = pos;   // left neighbour in the row above
      float a0 = x[o], a1 = x[o + 1], a2 = x[o + 2];
      o += P;
      float b0 = x[o], b1 = x[o + 1], b2 = x[o + 2];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        keep_packed(info[r]);
        keep_running(o);
        const float d0 = x[o + P], d1 = x[o + P + 1], d2 = x[o + P + 2];
        float v = w[0] * a0;
        v = fmaf(w[1], a1, v);
        v = fmaf(w[2], a2, v);
        v = fmaf(w[3], b0, v);
        v = fmaf(w[5], b2, v);
        v = fmaf(w[6], d0, v);
        v = fmaf(w[7], d1, v);
        v = fmaf(w[8], d2, v);
        v = fmaf(*reinterpret_cast<const float *>(sa + (info[r] & 0x3FCu)), b1, v);
        const float u = filter_lik<PLAIN>(lk, info[r], zl) * s * v;
        tot += u;
        if constexpr (decltype(STORE)::value) (dst + (size_t)r * NT)[tid] = u;
        if constexpr (DB)
          y[o + 1] = u;
        else
          ub[r] = u;
        a0 = b0; a1 = b1; a2 = b2;
        b0 = d0; b1 = d1; b2 = d2;
        o += P;
      }
    }
    if constexpr (!DB) {
      lds_barrier();   // every read of the band is done
      if (act) {
#pragma unroll
        for (int r = 0; r < R; ++r) y[pos + (r + 1) * P + 1] = ub[r];
      }
    }
    if constexpr (!PLAIN) {
      if (rgoal >= 0) {
        // the goal's inflow is in the band; its own mass stays on it
        const uint32_t gi = filter_info(fa.sig[m.goal]);
        float *yg = y + pos + (rgoal + 1) * P + 1;
        const float add = filter_lik<PLAIN>(lk, gi, zl) * s * gown;
        gown = *yg + add;
        tot += add;
        *yg = 0.f;
        if constexpr (decltype(STORE)::value) (dst + (size_t)rgoal * NT)[tid] = gown;
      }
    }
    tot = wave_total_lane63(tot);
    if (lane == kWave - 1) sh.upart[par][wave] = tot;
  };

  for (int tr = blockIdx.x; tr < fa.ntraj; tr += fa.G) {
    const int32_t *at = fa.acts + (size_t)tr * fa.T;
    const int32_t *zt = fa.obs + (size_t)tr * fa.T;
    const float *b0 = fa.b0 + (fa.b0_per_traj ? (size_t)tr * m.S : 0);
    // step i + 1's action and observation, U_{i+1}: chunk by chunk through LDS
    // (a global load in the loop over steps would wait for its stores too)
    int azc = -1, uc = (fa.T - 1) / kFChunk;
    auto az_at = [&](int i) {
      if (i / kFChunk != azc) {
        azc = i / kFChunk;
        lds_barrier();   // (its wait is its own: see lds_barrier)
        for (int j = tid; j < kFChunk; j += NT) {
          const int g = azc * kFChunk + j;
          sh.az[j] = g < fa.T ? at[g] + 256 * zt[g] : 0;
        }
        __syncthreads();
      }
      return sh.az[i % kFChunk];
    };
    auto u_at = [&](int i) {
      if (i / kFChunk != uc) {
        uc = i / kFChunk;
        lds_barrier();
        for (int j = tid; j < kFChunk; j += NT) sh.u[j] = usum[min(uc * kFChunk + j, fa.T - 1)];
        __syncthreads();
      }
      return sh.u[i % kFChunk];
    };
    bool bad = false;
    for (int t = tid; t < fa.T; t += NT) {
      const int a = at[t], z = zt[t];
      bad |= a < 0 || a >= A || z < 0 || z >= 16 * (m.L + 1);
    }
    if (__syncthreads_or(bad)) {
      if (tid == 0) {
        atomicOr(fa.err, 4);
        fa.nll[tr] = NAN;
      }
      if (fa.want_grad)
        for (int i = tid; i < kFGrad; i += NT) fa.gpart[(size_t)tr * kFGrad + i] = 0.0;
      continue;
    }
    for (int i = tid; i < 81; i += NT) sh.g[i] = 0.0;
    if (tid < 4) sh.mis[tid] = sh.ok[tid] = 0.0;
    float beta[R];
#pragma unroll
    for (int r = 0; r < R; ++r) beta[r] = 1.f;   // beta_T
    // First the forward pass over all steps, which stores the start of every
    // segment but the last, and all of the last; then, segment by segment
    // from the last, the segment's beliefs (recomputed from its start, except
    // for the last) and its reverse steps.
    const int tlast = (fa.nseg - 1) * fa.k;
    for (int sg = fa.nseg - 1; sg >= 0; --sg) {
      const bool whole = sg == fa.nseg - 1;
      const int t0 = sg * fa.k, t1 = min(fa.T, t0 + fa.k);
      const int tb = whole ? 0 : t0;   // first step of this forward pass
      const bool grad = fa.want_grad != 0;
      __syncthreads();
      fill(0.f);
      __syncthreads();
      float *x = band0, *y = band1;
      const int kb = tb == 0 ? 0 : __builtin_amdgcn_readfirstlane(filter_exp(u_at(tb - 1)));
      {
        const bool strips = tb != 0;
        const float lift = kb < -126 ? 0x1p23f : 1.f;
        const float *src = strips ? ckpt + (size_t)sg * SL : b0;
        float *dst = grad && (!whole || tlast == 0) ? segb : nullptr;
        int o = pos + 1;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          keep_packed(info[r]);
          keep_running(o);
          o += P;
          float v = 0.f;
          if (info[r] & kFiFree)
            v = strips ? (src + (size_t)r * NT)[tid]
                       : src[fa.along_x ? i1 * m.W + j0 + r : (j0 + r) * m.W + i1];
          if (dst) (dst + (size_t)r * NT)[tid] = v;
          v *= lift;
          if (!PLAIN && (info[r] & kFiGoal)) {
            gown = v;
            v = 0.f;
          }
          if (act) x[o] = v;
        }
      }
      __syncthreads();
      float s = filter_scale(kb);
      int az = az_at(tb);
      int tk = fa.k;   // next step whose belief starts a segment
      for (int t = tb + 1; t <= t1; ++t) {
        float *dst = nullptr;
        if (grad) {
          if (t > t0 || t == tlast) {
            dst = segb + (size_t)(t - t0) * SL;
          } else if (t == tk) {
            dst = ckpt + (size_t)(t / fa.k) * SL;
            tk += fa.k;
          }
        }
        const int uz = __builtin_amdgcn_readfirstlane(az), a = uz & 255, z = uz >> 8;
        az = az_at(min(t, t1 - 1));   // of the next step
        if (dst)
          fstep(std::true_type{}, x, y, a, z, s, dst, t & 1);
        else
          fstep(std::false_type{}, x, y, a, z, s, dst, t & 1);
        lds_barrier();
        const float U = filter_sum_waves(sh.upart[t & 1], small);
        if (whole && wave == 0) {   // (wavefront 0 reads what its lane 0 wrote)
          const int i = t - 1, j = i % kFChunk;
          if (lane == 0) sh.u[j] = U;
          if (j == kFChunk - 1 || t == fa.T)
            for (int l = lane; l <= j; l += kWave) usum[i - j + l] = sh.u[l];
        }
        s = filter_scale(filter_exp(U));
        if (__builtin_amdgcn_readfirstlane(__float_as_int(U)) - 1u < 0x7FFFFFu) {   // subnormal, rare: a pass over the band, own cells
          if (act) {
#pragma unroll 1
            for (int r = 0, o = pos + P + 1; r < R; ++r, o += P) y[o] *= 0x1p23f;
          }
          gown *= 0x1p23f;
          lds_barrier();
        }
        float *o = x;
        x = y;
        y = o;
      }
      if (whole) {
        // NLL = -sum log(U_t / U_{t-1} as step t saw it), in FP64
        __syncthreads();
        double nll = 0.0;
        for (int t = 1 + tid; t <= fa.T; t += NT) {
          const float up = t > 1 ? usum[t - 2] : 1.f;
          nll -= log((double)usum[t - 1] / (double)filter_scaled(up));
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) nll += __shfl_xor(nll, o, kWave);
        if (lane == 0) sh.red[wave] = nll;
        __syncthreads();
        if (tid == 0) {
          nll = 0.0;
          for (int w = 0; w < NT / kWave; ++w) nll += sh.red[w];
          fa.nll[tr] = (float)nll;
          if (!(nll < INFINITY)) atomicOr(fa.err, 8);
        }
      }
      if (!grad) break;

      // ---- the segment's reverse steps
      __syncthreads();
      fill(-1.f);   // blocked and off-grid entries of v
      __syncthreads();
      x = band0;
      y = band1;
      az = __builtin_amdgcn_readfirstlane(az_at(t1 - 1));
      int a = az & 255, z = az >> 8;
      float U = u_at(t1 - 1), Up = t1 > 1 ? u_at(t1 - 2) : 1.f;
      float gs[9], gm[5];   // slip sums; gamma by wall bit's rarer reading and in all
#pragma unroll
      for (int i = 0; i < 5; ++i) gm[i] = 0.f;
      {
        // v_{t1} from beta_{t1}, and gamma_{t1}
        const float ie = filter_scaled(Up) / U;   // 1 / eta_t
        const uint32_t zl = (uint32_t)(z >> 4), zx = ((uint32_t)z ^ rare) << 10;
        const float *lk = sh.lik[zl ? 1 : 0][z & 15];
        const float *ut = segb + (size_t)(t1 - t0) * SL;
        int o = pos + 1;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          keep_packed(info[r]);
          keep_running(o);
          o += P;
          if (info[r] & kFiFree) {
            x[o] = filter_lik<PLAIN>(lk, info[r], zl) * beta[r] * ie;
            const float ga = (ut + (size_t)r * NT)[tid] * beta[r];
#pragma unroll
            for (int i = 0; i < 4; ++i) gm[i] += (((info[r] ^ zx) >> (10 + i)) & 1u) ? ga : 0.f;
            gm[4] += ga;
          }
        }
      }
      __syncthreads();
      for (int t = t1; t > t0; --t) {
        // the step before (at the segment's start: none): its action,
        // observation, sum and belief, read ahead
        const int tn = max(t - 1, 1);
        az = __builtin_amdgcn_readfirstlane(az_at(tn - 1));
        const int an = az & 255, zn = az >> 8;
        const float Upp = t > 2 ? u_at(t - 3) : 1.f;
        const float *up = segb + (size_t)(t - 1 - t0) * SL;
        float bp[R];
#pragma unroll
        for (int r = 0; r < R; ++r) bp[r] = (up + (size_t)r * NT)[tid];
        float w[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) w[q] = slip_at(a, q / 3 - 1, q % 3 - 1);
        const float ie = filter_scaled(Upp) / Up;   // 1 / eta_{t-1}
        const uint32_t zl = (uint32_t)(zn >> 4), zx = ((uint32_t)zn ^ rare) << 10;
        const float *lk = sh.lik[zl ? 1 : 0][zn & 15];
        float gn[5];
#pragma unroll
        for (int i = 0; i < 9; ++i) gs[i] = 0.f;
#pragma unroll
        for (int i = 0; i < 5; ++i) gn[i] = 0.f;
        if (act) {
          int o = pos;
          float a0 = x[o], a1 = x[o + 1], a2 = x[o + 2];
          o += P;
          float b0_ = x[o], b1 = x[o + 1], b2 = x[o + 2];
#pragma unroll
          for (int r = 0; r < R; ++r) {
            keep_packed(info[r]);
            keep_running(o);
            const float d0 = x[o + P], d1 = x[o + P + 1], d2 = x[o + P + 2];
            const float n[9] = {a0, a1, a2, b0_, b1, b2, d0, d1, d2};
            const float ub = bp[r];
            // the goal moves no mass (nor does a blocked cell, whose u is 0)
            const bool at_goal = !PLAIN && (info[r] & kFiGoal);
            const float bv = at_goal ? 0.f : ub;
            float acc = w[4] * b1;
            gs[4] = fmaf(bv, b1, gs[4]);
#pragma unroll
            for (int q = 0; q < 9; ++q) {
              if (q == 4) continue;
              const float cd = n[q] < 0.f ? b1 : n[q];
              acc = fmaf(w[q], cd, acc);
              gs[q] = fmaf(bv, cd, gs[q]);
            }
            if (at_goal) acc = b1;   // the goal keeps its own mass
            beta[r] = acc;
            const float ga = ub * acc;
#pragma unroll
            for (int i = 0; i < 4; ++i) gn[i] += (((info[r] ^ zx) >> (10 + i)) & 1u) ? ga : 0.f;
            gn[4] += ga;
            if constexpr (DB) {
              const float v = filter_lik<PLAIN>(lk, info[r], zl) * acc * ie;
              y[o + 1] = (info[r] & kFiFree) ? v : -1.f;
            }
            a0 = b0_; a1 = b1; a2 = b2;
            b0_ = d0; b1 = d1; b2 = d2;
            o += P;
          }
        }
        // the wavefronts' sums: slip of step t, gamma_t from the pass before
#pragma unroll
        for (int i = 0; i < kFSums; ++i) {
          const float v = wave_total_lane63(i < 9 ? gs[i < 9 ? i : 0] : gm[i < 9 ? 0 : i - 9]);
          if (lane == kWave - 1) sh.gpart[t & 1][i][wave] = v;
        }
        lds_barrier();
        if constexpr (!DB) {
          if (act) {
#pragma unroll
            for (int r = 0; r < R; ++r)
              if (info[r] & kFiFree)
                y[pos + (r + 1) * P + 1] = filter_lik<PLAIN>(lk, info[r], zl) * beta[r] * ie;
          }
          lds_barrier();
        }
        if (tid < 13) {
          const float *p = &sh.gpart[t & 1][0][0];
          const double v = filter_sum_waves(p + tid * kFWaves, small);
          const double all = filter_sum_waves(p + 13 * kFWaves, small);
          // <beta_t, b_t> = all / U_t is 1 but for the steps' roundings, which
          // would add up over the run: it is divided out of every step's terms
          if (tid < 9) {
            const int k = fa.along_x ? tid % 3 * 3 + tid / 3 : tid;
            // b_{t-1} = u_{t-1} / U_{t-1} (the start belief itself at t = 1)
            sh.g[a * 9 + k] -= v * (double)U / (t > 1 ? (double)Up * all : all);
          } else {
            const int i = tid - 9;
            const double few = v / all, rest = (all - v) / all;
            sh.mis[i] += ((rare >> i) & 1) ? rest : few;
            sh.ok[i] += ((rare >> i) & 1) ? few : rest;
          }
        }
#pragma unroll
        for (int i = 0; i < 5; ++i) gm[i] = gn[i];
        float *o = x;
        x = y;
        y = o;
        a = an;
        z = zn;
        U = Up;
        Up = Upp;
      }
    }
    if (!fa.want_grad) continue;
    __syncthreads();
    for (int i = tid; i < 81; i += NT)
      fa.gpart[(size_t)tr * kFGrad + i] = i < A * 9 ? sh.g[i] : 0.0;
    if (tid < 4) {
      // where a factor is 0 the step's likelihood is 0 too and adds nothing
      const double f = (double)sh.flip[tid], g = (double)(1.f - sh.flip[tid]);
      fa.gpart[(size_t)tr * kFGrad + 81 + tid] =
          (g > 0.0 ? sh.ok[tid] / g : 0.0) - (f > 0.0 ? sh.mis[tid] / f : 0.0);
    }
  }
}

// Sum of the per-trajectory partials (FP64, fixed order: kFGradParts
// interleaved running sums, then those in order), then the chain rule through
// the softmax and the logistic.  Latency-bound: one running sum over 1024
// trajectories took 325 us, twelve take 24 us.
constexpr int kFGradParts = 12;
__global__ __launch_bounds__(1024) void k_filter_grad(int ntraj, int A, const float *theta,
                                                      const float *phi, const double *gpart,
                                                      float *g_slip, float *g_flip) {
  __shared__ double part[kFGradParts * kFGrad];
  __shared__ double g[kFGrad];
  __shared__ double sl[81];
  const int tid = threadIdx.x;
  if (tid < kFGradParts * kFGrad) {
    const int j = tid / kFGrad, i = tid - j * kFGrad;
    double s = 0.0;
#pragma unroll 8
    for (int t = j; t < ntraj; t += kFGradParts) s += gpart[(size_t)t * kFGrad + i];
    part[tid] = s;
  }
  __syncthreads();
  if (tid < kFGrad) {
    double s = 0.0;
    for (int j = 0; j < kFGradParts; ++j) s += part[j * kFGrad + tid];
    g[tid] = s;
  }
  if (tid < A) {
    double mx = -INFINITY, sum = 0.0;
    for (int k = 0; k < 9; ++k) mx = fmax(mx, (double)theta[tid * 9 + k]);
    for (int k = 0; k < 9; ++k) sum += exp((double)theta[tid * 9 + k] - mx);
    for (int k = 0; k < 9; ++k) sl[tid * 9 + k] = exp((double)theta[tid * 9 + k] - mx) / sum;
  }
  __syncthreads();
  if (tid < A * 9) {
    const int a = tid / 9, j = tid - a * 9;
    double s = 0.0;
    for (int k = 0; k < 9; ++k)
      s += g[a * 9 + k] * sl[a * 9 + k] * ((k == j ? 1.0 : 0.0) - sl[a * 9 + j]);
    g_slip[tid] = (float)s;
  }
  if (tid < 4) {
    const double f = 1.0 / (1.0 + exp(-(double)phi[tid]));
    g_flip[tid] = (float)(g[81 + tid] * f * (1.0 - f));
  }
}

size_t filter_lds_bytes(const qv_model *m) {
  return ((size_t)(m->H + 2) * (m->W + 2) + (size_t)m->W * m->H + (size_t)m->A * 256) *
         sizeof(float);
}

bool filter_supported(const qv_model *m) { return filter_lds_bytes(m) <= 150 * 1024; }

// How a grid is cut into strips, and how many trajectories run at once.  It
// depends on the grid alone (and so do all sums), except for G.
struct FilterPlan {
  int n1, n2, along_x, rr, ng, pitch, threads, G;
  bool db;
  size_t lds;
};

// Bytes that the stored beliefs of several workgroups a CU may take.  Measured,
// 4096 runs on 24x24: 2000 steps, every 10th stored, 36 ms in 804 MiB, 49 in
// 515, 82 in 259 and 162 in 123 (one a CU); 200 steps, every 14th, 3.6 ms in
// 116 MiB.
constexpr size_t kFilterStore = (size_t)512 << 20;

// Strip length: the one of least estimated time of a step on the busiest
// SIMD, in cycles: each of its wavefronts takes about 800 for the step itself
// (inputs, reduction, barrier) and 110 per cell, so a small grid is better
// cut into few wavefronts of longer strips.  Measured on 24x24, 8 runs x 200
// steps, NLL: 9 wavefronts of 1 cell 343 us, 3 of 4 cells 208 us.  From 8 cells on
// a strip spills registers (9 at 8, 31 at 12, 57 at 16, 91 at 22 cells, up to
// six more with landmarks or a goal); those of 22 count double, so that they are
// taken only where nothing shorter covers the grid.
static FilterPlan filter_plan(int W, int H, int A, int ntraj, int T, int k) {
  FilterPlan p;
  p.along_x = W > H ? 1 : 0;
  p.n1 = p.along_x ? H : W;
  p.n2 = p.along_x ? W : H;
  int best = 1 << 30;
  p.rr = p.ng = p.threads = 0;
  for (const int rr : {1, 2, 4, 6, 8, 12, 16, 22}) {   // the lengths of k_filter's instances
    const int ng = (p.n2 + rr - 1) / rr;
    if (p.n1 * ng > kFMaxBlock) continue;
    const int waves = (p.n1 * ng + kWave - 1) / kWave;
    const int cost = ((waves + 3) / 4) * (800 + 110 * rr) * (rr > 16 ? 2 : 1);
    if (cost < best) {
      best = cost;
      p.rr = rr;
      p.ng = ng;
      p.threads = waves * kWave;
    }
  }
  const size_t rest = (size_t)A * 256 * sizeof(float);
  const size_t room = 160 * 1024 - sizeof(FilterShared);
  auto band_bytes = [&](int pitch) { return (size_t)(p.ng * p.rr + 2) * pitch * sizeof(float); };
  // On narrow grids a wavefront holds many strips; where their starts would
  // all fall on one or two banks of the LDS, rows are a float apart more (2000x2, 64
  // runs x 20 steps, NLL: 121 us without, 86 with).
  p.pitch = p.n1 + 2;
  if (p.n1 < kWave && p.rr * p.pitch % 32 == 0 && 2 * band_bytes(p.pitch + 1) + rest <= room)
    ++p.pitch;
  const size_t band = band_bytes(p.pitch);
  p.db = 2 * band + rest <= room;
  p.lds = (p.db ? 2 : 1) * band + rest;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus <= 0)
    cus = 256;
  const int per = std::max<int>(1, std::min<int>(16 / (p.threads / kWave),
                                                 (int)(160 * 1024 / (p.lds + sizeof(FilterShared)))));
  // Several workgroups a CU as long as their stored beliefs take no more than
  // one a CU would for the bare cells, or than kFilterStore.
  const size_t nseg = (T + k - 1) / k;
  const size_t each = (nseg + k + 1) * p.rr * p.threads * 4 + (size_t)T * 4;
  const size_t bare = (nseg + k + 2) * W * H * 4 + (size_t)(T + 1) * 4;
  const size_t limit = std::max((size_t)std::min(ntraj, cus) * bare, kFilterStore);
  p.G = std::max(1, (int)std::min<size_t>(std::min(ntraj, cus * per), limit / each));
  return p;
}

// Byte offsets of the filter workspace.
struct FilterWs {
  size_t sig, staytab, ckpt, seg, usum, gpart, err, total;
};

static FilterWs filter_layout(const FilterPlan &p, int W, int H, int A, int ntraj, int T, int k) {
  const size_t S = (size_t)W * H, SL = (size_t)p.rr * p.threads;
  const int nseg = (T + k - 1) / k;
  FilterWs w;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off += align_up(bytes, 256);
    return at;
  };
  w.sig = take(S * 4);
  w.staytab = take((size_t)A * 256 * 4);          // (prep)
  w.ckpt = take((size_t)p.G * nseg * SL * 4);     // stored beliefs
  w.seg = take((size_t)p.G * (k + 1) * SL * 4);   // segment buffers
  w.usum = take((size_t)p.G * T * 4);           // U_t
  w.gpart = take((size_t)ntraj * kFGrad * 8);     // per-trajectory partials
  w.err = take(4);                                // the last 256 bytes
  w.total = off;
  return w;
}

size_t filter_ws(const qv_model *m, int ntraj, int T, int k) {
  const FilterPlan p = filter_plan(m->W, m->H, m->A, ntraj, T, k);
  return filter_layout(p, m->W, m->H, m->A, ntraj, T, k).total;
}

template <int R, bool DB, bool PLAIN>
static hipError_t launch_filter_r(const DevModel &m, const FilterArgs &fa, const FilterPlan &p,
                                  hipStream_t st) {
  const hipError_t e =
      hipFuncSetAttribute(reinterpret_cast<const void *>(&k_filter<R, DB, PLAIN>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds);
  if (e != hipSuccess) return e;
  QV_LAUNCH((k_filter<R, DB, PLAIN>), dim3(p.G), dim3(p.threads), p.lds, st, m, fa);
  return hipGetLastError();
}

template <bool PLAIN>
static hipError_t launch_filter_p(const DevModel &m, const FilterArgs &fa, const FilterPlan &p,
                                  hipStream_t st) {
  switch (p.rr) {
    case 1: return launch_filter_r<1, true, PLAIN>(m, fa, p, st);
    case 2: return launch_filter_r<2, true, PLAIN>(m, fa, p, st);
    case 4: return launch_filter_r<4, true, PLAIN>(m, fa, p, st);
    case 6: return launch_filter_r<6, true, PLAIN>(m, fa, p, st);
    case 8: return launch_filter_r<8, true, PLAIN>(m, fa, p, st);
    case 12: return launch_filter_r<12, true, PLAIN>(m, fa, p, st);
    // only the longest strips' grids can lack room for two bands
    case 16:
      return p.db ? launch_filter_r<16, true, PLAIN>(m, fa, p, st)
                  : launch_filter_r<16, false, PLAIN>(m, fa, p, st);
    case 22:
      return p.db ? launch_filter_r<22, true, PLAIN>(m, fa, p, st)
                  : launch_filter_r<22, false, PLAIN>(m, fa, p, st);
    default: return hipErrorInvalidValue;   // no accepted grid comes here
  }
}

hipError_t launch_filter(const DevModel &m, const float *theta, const float *phi, int ntraj,
                         int T, const float *b0, int b0_per_traj, const int32_t *acts,
                         const int32_t *obs, int k, float *nll, float *g_slip, float *g_flip,
                         char *ws, hipStream_t st) {
  const FilterPlan p = filter_plan(m.W, m.H, m.A, ntraj, T, k);
  const FilterWs w = filter_layout(p, m.W, m.H, m.A, ntraj, T, k);
  uint32_t *sig = (uint32_t *)(ws + w.sig);
  hipError_t e = launch_prep(m, sig, (float *)(ws + w.staytab), (int32_t *)(ws + w.err), st);
  if (e != hipSuccess) return e;
  FilterArgs fa;
  fa.ntraj = ntraj;
  fa.T = T;
  fa.k = k;
  fa.nseg = (T + k - 1) / k;
  fa.G = p.G;
  fa.n1 = p.n1;
  fa.n2 = p.n2;
  fa.ng = p.ng;
  fa.pitch = p.pitch;
  fa.along_x = p.along_x;
  fa.theta = theta;
  fa.phi = phi;
  fa.b0 = b0;
  fa.b0_per_traj = b0_per_traj;
  fa.acts = acts;
  fa.obs = obs;
  fa.nll = nll;
  fa.gpart = (double *)(ws + w.gpart);
  fa.ckpt = (float *)(ws + w.ckpt);
  fa.seg = (float *)(ws + w.seg);
  fa.usum = (float *)(ws + w.usum);
  fa.sig = sig;
  fa.err = (int32_t *)(ws + w.err);
  fa.want_grad = (g_slip && g_flip) ? 1 : 0;
  if (ntraj > 0) {
    e = m.L == 0 && m.goal < 0 ? launch_filter_p<true>(m, fa, p, st)
                               : launch_filter_p<false>(m, fa, p, st);
    if (e != hipSuccess) return e;
  }
  // with no trajectories the gradient kernel writes zeros
  if (fa.want_grad)
    QV_LAUNCH(k_filter_grad, dim3(1), dim3(1024), 0, st, ntraj, m.A, theta, phi, fa.gpart, g_slip,
              g_flip);
  return hipGetLastError();
}

}  // namespace qv
