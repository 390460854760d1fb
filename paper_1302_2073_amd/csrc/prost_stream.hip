// Frames too large for a resident gang of register tiles (Sec. 3.3, Steps
// 1-3, with the step-size rule of Sec. 3.4): the same per-frame arithmetic as
// the frame kernel, but every dependent pass streams U and the frame from
// HBM.  Per frame and CG step (Step 1):
//   gradient pass: r = x - U y, phi, c; partials of U^T (w phi'(r)),
//                  sum w phi(r) and the upper triangle of
//                  H = U^T diag(w c) U
//   step:          fixed-order sums of the partials, PR+ direction d,
//                  d^T H d, alpha = -g.d / d^T H d, y += alpha d
// then (Step 2) the eta pass (eta = -w phi'(r) stored per entry, partials of
// U^T eta, ||eta||^2 and the final cost), the geodesic scalars, and one pass
// that updates U and labels every pixel (Step 3).  A thread takes one pixel
// (all channels), or two adjacent ones in bfloat16 storage with even P and
// aligned planes (32-bit accesses).  Reductions: float32 over the pixels that a
// wavefront takes at a time, float64 over those and across wavefronts and
// workgroups, H in float64 throughout; the order is fixed, so results are
// deterministic.
//
// A step reads U once: H (a contraction over the rows with both operands U) is
// formed on the matrix cores beside the gradient, where a second pass for
// sum w c (u.d)^2 took 26 us of a 1280x720x3, k = 15 float32 step and
// k (k + 1) / 2 products per entry in the vector unit 38.
// The sums of a step's partials run one workgroup per value, and the last of
// them to finish takes the k-space step: two launches per CG step instead of
// four, and none around the frame.  A 1280x720x3, k = 15 frame takes 359 us in
// float32 (482 with the two-pass step) and 309 in bfloat16 (315).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "../../include/prost.h"
#include "prost_frame.hpp"
#include "prost_host.hpp"

namespace prost {

constexpr int kStBlock = 256;           // threads per workgroup of a pass (one pixel or pixel pair each)
constexpr int kStWaves = kStBlock / 64;
constexpr int kStWide = 160;            // values of a gradient pass: g (K), f and H's upper triangle (<= 153)
template <int KC>
constexpr int st_nh() { return KC + 1 + KC * (KC + 1) / 2; }
static_assert(st_nh<kMaxK>() <= kStWide && kStWide <= kStBlock, "one thread per value");
constexpr int kStPad = 68;              // floats per column of a wavefront's 64 rows in LDS (16-byte aligned, spreads banks)

// Workgroups of a reducing pass over nchunk groups of kStBlock threads' pixels:
// five per compute unit, what both storage types hold at once, each taking
// groups kStResident apart.  A pass leaves 1280 partials per value of a
// 1280x720 frame instead of 3600 to sum, and every compute unit gets the same
// share.
constexpr int kStResident = 1280;
static int st_blocks(int nchunk) { return std::min(nchunk, kStResident); }

// k-space state of the frame being streamed (device memory, one per handle).
struct StreamKS {
  double y[kMaxK], gp[kMaxK], d[kMaxK], dp[kMaxK];   // y, previous gradient, direction, previous direction
  double gd;
  float yf[kMaxK], yl[kMaxK];   // y as float32 plus its float32 remainder: r = x - U yf - U yl
  float df[kMaxK], vf[kMaxK], af[kMaxK];
  float cm1, sz, nu;
  int stop, bad, upd, steps, restarts;
  unsigned ticket;        // workgroups of a summing launch that are done
  double tot[kStWide];    // reduced values of the latest pass
};

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// One value per workgroup of a summing launch: value v = blockIdx.x's partials
// of the nblk workgroups of a pass (contiguous) in a fixed order, to ks->tot.
// True in the workgroup that finishes last, which then sees all totals: they
// go out as device-coherent stores, complete before the ticket is taken.
__device__ __forceinline__ bool st_sum_value(StreamKS* ks, const double* __restrict__ part, int nblk, double* red,
                                             int* last, double* tot) {
  const int v = blockIdx.x, t = threadIdx.x;
  const double* row = part + (size_t)v * nblk;
  double s = 0.0;
#pragma unroll 4
  for (int b = t; b < nblk; b += kStBlock) s += row[b];
  s = wave_sum(s);
  if ((t & 63) == 0) red[t >> 6] = s;
  __syncthreads();
  if (t == 0) {
    __hip_atomic_store(&ks->tot[v], (red[0] + red[1]) + (red[2] + red[3]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the total is out
    *last = __hip_atomic_fetch_add(&ks->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x;
    if (*last) ks->ticket = 0;
  }
  __syncthreads();
  if (!*last) return false;
  if (t < (int)gridDim.x) tot[t] = __hip_atomic_load(&ks->tot[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  return true;
}

__device__ __forceinline__ float st_weight(const FrameArgs& a, int p) {
  const uint8_t* src = a.weights_from_filtered ? a.mask : a.lab;
  return src[p] ? a.omega : 1.0f;
}

// Pixels per thread of a pass: one, or (PAIR, bfloat16 with even P and
// 4-byte aligned planes) two adjacent pixels whose entries are one aligned
// 32-bit word in every plane of U and of the frame: half the load and store
// instructions for the same bytes.
template <typename TS, bool PAIR>
struct StPix {
  static_assert(!PAIR || sizeof(TS) == 2, "pairs of bfloat16 entries");
  static constexpr int N = PAIR ? 2 : 1;
};

// The entries of channel c of this thread's pixels p0 (.. p0 + 1): U rows
// (columns >= k are 0) and frame values.
template <int KC, typename TS, bool PAIR>
__device__ __forceinline__ void st_load(const FrameArgs& a, int c, int p0, float (&u)[StPix<TS, PAIR>::N][KC],
                                        float (&x)[StPix<TS, PAIR>::N]) {
  const long long e = (long long)c * a.P + p0;
  if constexpr (PAIR) {
    const uint32_t* __restrict__ U = (const uint32_t*)a.U;
    const uint32_t xw = ((const uint32_t*)a.x)[e >> 1];
    x[0] = bf_lo(xw);
    x[1] = bf_hi(xw);
#pragma unroll
    for (int j = 0; j < KC; ++j) {
      const uint32_t w = (j < a.k) ? U[((long long)j * a.ldU + e) >> 1] : 0u;
      u[0][j] = bf_lo(w);
      u[1][j] = bf_hi(w);
    }
  } else {
    const TS* __restrict__ U = (const TS*)a.U;
    x[0] = ld_elem((const TS*)a.x, e);
#pragma unroll
    for (int j = 0; j < KC; ++j) u[0][j] = (j < a.k) ? ld_elem(U, (long long)j * a.ldU + e) : 0.f;
  }
}

// r = x - U y with y as the float32 pair (value, remainder).
template <int KC>
__device__ __forceinline__ float st_residual(float x, const float (&u)[KC], const float* ys, const float* yl) {
  float r = x, rl = 0.f;
#pragma unroll
  for (int j = 0; j < KC; ++j) {
    r = fmaf(-u[j], ys[j], r);
    rl = fmaf(-u[j], yl[j], rl);
  }
  return r + rl;
}

// y (float64) as the float32 pair the passes use: every pass recomputes
// r = x - U y from the frame, and the remainder keeps that residual as
// accurate as the float64 y (near a fit the gradient is small and a
// float32-rounded y would dominate its error).
__device__ __forceinline__ void st_set_y(StreamKS* ks, int j, double yv) {
  ks->y[j] = yv;
  const float hi = (float)yv;
  ks->yf[j] = hi;
  ks->yl[j] = (float)(yv - (double)hi);
}

// y of the passes: the handle's at the frame's first step (nothing is prepared
// before it), the k-space state's after that.
__device__ __forceinline__ void st_get_y(const FrameArgs& a, const StreamKS* ks, bool first, int j, float* ys,
                                         float* yl) {
  if (first) {
    const double yv = (j < a.k) ? a.y[j] : 0.0;
    ys[j] = (float)yv;
    yl[j] = (float)(yv - (double)(float)yv);
  } else {
    ys[j] = ks->yf[j];
    yl[j] = ks->yl[j];
  }
}

// Step 1 gradient pass at the current y (float32 per thread, as the frame
// kernel): partials of g, f and H's upper triangle row by row, value-major
// (part[v * gridDim.x + workgroup]).  H: a wavefront leaves 64 rows of U,
// times the root of their w c, in LDS (its own, no barrier) and multiplies them
// in 16 steps of v_mfma_f64_16x16x4: lane l holds column l % 16 of rows
// 16 (l / 16) + step, as both operands, and one 16 x 16 tile accumulates over
// all rows of the wavefront.  In float64: along a direction that foreground
// pixels carry (weight omega, far from the fit) d^T H d is what is left of
// entries 10^7 times larger, and a float32 tile lost it (a step 30 times too
// short, or an early end of the steps).  The products of the rounded rows are
// exact, so the tile is the square of a matrix, and what their rounding adds to
// the form is a square too: as much as rounding u.d adds to sum w c (u.d)^2.
// These matrix instructions and the vector work share the SIMD's time (each
// alone 905 and 972 us, together 1832), so they cost 64 cycles per 4 rows of a
// wavefront even behind the read.  Up to 8 columns two groups of 32 rows lie
// side by side in the tile, up to 4 four of 16 (their products with each other
// are not used): half and a quarter of the steps.  Below 16 columns the tile has
// room for r beside U, and its column of products is g: no separate sums (at 8,
// where r would take the second group's room, they cost less than it).  f, and g
// where it is not in the tile, are float32 over a thread's pixels of one group, as the frame kernel
// has them over a tile, and float64 over the groups: a float32 sum over all of a
// workgroup's groups would lose more with every group of a larger frame.
template <int KC, typename TS, bool PAIR>
__global__ __launch_bounds__(kStBlock) void st_grad(FrameArgs a, const StreamKS* __restrict__ ks,
                                                    double* __restrict__ part, int nchunk, bool first) {
  constexpr int N = StPix<TS, PAIR>::N;
  constexpr int NV = st_nh<KC>();
  constexpr bool kGradInTile = KC != 8 && KC < 16;   // column KC of the tile is r
  constexpr int LG = kGradInTile ? 1 : KC + 1;
  constexpr int kCols = kGradInTile ? KC + 1 : KC;
  constexpr int PK = kCols <= 4 ? 4 : kCols <= 8 ? 2 : 1;   // row groups side by side in the tile
  constexpr int GC = 16 / PK, GR = 64 / PK;                 // columns and rows of a group
  if (!first && (ks->stop || ks->bad)) return;
  __shared__ float ys[KC], yl[KC];
  __shared__ __align__(16) float us[kStWaves][16][kStPad];
  __shared__ double red[kStWaves][LG];
  const int tid = thread_index(), lane = tid & 63, wv = tid >> 6;
  const int i16 = lane & 15, k4 = lane >> 4;
  float (*const row)[kStPad] = &us[wv][lane / GR * GC];   // this lane's row: row[column][lane % GR]
  if (tid < KC) st_get_y(a, ks, first, tid, ys, yl);
#pragma unroll
  for (int j = kCols; j < GC; ++j) row[j][lane % GR] = 0.f;
  __syncthreads();
  double sum = 0.0;   // f of this thread, or component comp of (g, f) of the wavefront
  int comp = 0;
  f64x4_t h = {0.0, 0.0, 0.0, 0.0};
  for (int ch = blockIdx.x; ch < nchunk; ch += gridDim.x) {
    const int p0 = (ch * kStBlock + tid) * N;
    const bool valid = p0 < a.P;   // with pairs P is even, so both pixels are
    float wt[N], acc[LG];
#pragma unroll
    for (int j = 0; j < LG; ++j) acc[j] = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) wt[i] = valid ? st_weight(a, p0 + i) : 0.f;
    for (int c = 0; c < a.C; ++c) {
      float u[N][KC], x[N];
      if (valid) {
        st_load<KC, TS, PAIR>(a, c, p0, u, x);
      } else {
#pragma unroll
        for (int i = 0; i < N; ++i) {
          x[i] = 0.f;
#pragma unroll
          for (int j = 0; j < KC; ++j) u[i][j] = 0.f;
        }
      }
#pragma unroll
      for (int i = 0; i < N; ++i) {
        float sw = 0.f, r = 0.f;
        if (valid) {
          r = st_residual<KC>(x[i], u[i], ys, yl);
          float phi, cc;
          cost_eval(r, a.cp, phi, cc);
          const float w_c = wt[i] * cc;
          acc[LG - 1] = fmaf(wt[i], phi, acc[LG - 1]);
          if constexpr (!kGradInTile) {
            const float wd = w_c * r;                 // w phi'(r)
#pragma unroll
            for (int j = 0; j < KC; ++j) acc[j] = fmaf(wd, u[i][j], acc[j]);
          }
          sw = sqrtf(w_c);
        }
        wave_order();   // the rows before these have been read
#pragma unroll
        for (int j = 0; j < KC; ++j) row[j][lane % GR] = sw * u[i][j];
        if constexpr (kGradInTile) row[KC][lane % GR] = sw * r;
        wave_order();
#pragma unroll
        for (int q = 0; q < GR / 16; ++q) {
          const float4 uq = *(const float4*)&us[wv][i16][k4 * (GR / 4) + 4 * q];
          h = __builtin_amdgcn_mfma_f64_16x16x4f64((double)uq.x, (double)uq.x, h, 0, 0, 0);
          h = __builtin_amdgcn_mfma_f64_16x16x4f64((double)uq.y, (double)uq.y, h, 0, 0, 0);
          h = __builtin_amdgcn_mfma_f64_16x16x4f64((double)uq.z, (double)uq.z, h, 0, 0, 0);
          h = __builtin_amdgcn_mfma_f64_16x16x4f64((double)uq.w, (double)uq.w, h, 0, 0, 0);
        }
      }
    }
    if constexpr (kGradInTile)
      sum += (double)acc[0];
    else
      sum += (double)wave_reduce_scatter<LG>(acc, comp);
  }
  if constexpr (kGradInTile) {
    sum = wave_sum(sum);
    if (lane == 0) red[wv][0] = sum;
  } else {
    if (wave_rs_owner<LG>(lane) && comp < LG) red[wv][comp] = sum;
  }
  wave_order();
#pragma unroll
  for (int v = 0; v < 4; ++v) ((double*)us[wv])[(4 * v + k4) * 16 + i16] = h[v];   // H[row][column]
  __syncthreads();
  if (tid < NV) {
    double s = 0.0;
    if (tid == KC || (!kGradInTile && tid < KC)) {
#pragma unroll
      for (int w = 0; w < kStWaves; ++w) s += red[w][kGradInTile ? 0 : tid];
    } else {
      int i = tid, t = KC - tid;   // g: row tid, column KC
      if (tid > KC) {
        i = 0;
        t = tid - (KC + 1);
        while (t >= KC - i) {
          t -= KC - i;
          ++i;
        }
      }
#pragma unroll
      for (int w = 0; w < kStWaves; ++w) {
#pragma unroll
        for (int p = 0; p < PK; ++p) s += ((const double*)us[w])[(p * GC + i) * 16 + p * GC + i + t];
      }
    }
    part[(size_t)tid * gridDim.x + blockIdx.x] = s;
  }
}

// PR+ direction from the reduced gradient and cost tot[0..KC] (the frame
// kernel's k-space step), by the first wavefront; d, its float32 copy, the
// previous gradient, g.d and the stop / bad flags land in ks.
template <int KC>
__device__ __forceinline__ void st_dir_core(const FrameArgs& a, StreamKS* ks, const double* tot, int it) {
  const int lane = threadIdx.x;
  const double g = (lane < a.k) ? -tot[lane] : 0.0;
  const double f = tot[KC];
  const double gg = row16_sum(g * g);
  int stop = 0, bad = 0;
  if (it == 0 && !(isfinite(f) && isfinite(gg))) stop = bad = 1;
  if (gg == 0.0) stop = 1;
  double beta = 0.0, dj = -g;
  if (!stop && it > 0 && a.ysolve == 0) {
    const double gpv = (lane < a.k) ? ks->gp[lane] : 0.0;
    const double num = row16_sum(g * (g - gpv));
    const double den = row16_sum(gpv * gpv);
    beta = fmax(0.0, num / den);
    const double dpv = (lane < a.k) ? ks->dp[lane] : 0.0;
    dj = -g + beta * dpv;
    if (row16_sum(g * dj) >= 0.0) {
      dj = -g;
      if (lane == 0) ++ks->restarts;
    }
  }
  const double gd = row16_sum(g * dj);
  if (lane < kMaxK) {
    ks->d[lane] = (lane < a.k) ? dj : 0.0;
    ks->df[lane] = (lane < a.k) ? (float)dj : 0.f;
    ks->gp[lane] = (lane < a.k) ? g : 0.0;
  }
  if (lane == 0) {
    a.stats->f[it] = f;
    a.stats->beta[it] = beta;
    ks->gd = gd;
    ks->stop = stop;
    if (bad) {
      ks->bad = 1;
      __hip_atomic_fetch_or(&a.sync[2], kErrBadFrame, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// Majoriser step alpha = -g.d / d^T H d, y += alpha d (stop if d^T H d <= 0).
__device__ __forceinline__ void st_adv_core(const FrameArgs& a, StreamKS* ks, double dHd, int it) {
  const int t = threadIdx.x;
  if (!(dHd > 0.0)) {
    if (t == 0) ks->stop = 1;
    return;
  }
  const double alpha = -ks->gd / dHd;
  if (t < kMaxK) {
    st_set_y(ks, t, ks->y[t] + alpha * ks->d[t]);
    ks->dp[t] = ks->d[t];
  }
  if (t == 0) {
    a.stats->alpha[it] = alpha;
    ks->steps = it + 1;
  }
}

// Sums of a gradient pass, then direction and majoriser step from them
// (d^T H d: lane i row i of the triangle, rows added in order).  H is
// positive semidefinite, and the form is known to about 2^-48 of the
// magnitudes of its terms (the square of a float32 rounding, which is what a
// sum of w c (u.d)^2 with u.d in float32 resolves too): anything below is that.
// A larger curvature majorises as well, so the step stays one of descent, and
// rounding does not end the steps: only H d = 0 does.
template <int KC>
__global__ __launch_bounds__(kStBlock) void st_step(FrameArgs a, StreamKS* ks, const double* __restrict__ part,
                                                    int nblk, int it) {
  if (it > 0 && (ks->stop || ks->bad)) return;
  __shared__ double red[kStWaves];
  __shared__ int last;
  __shared__ double tot[kStWide];
  __shared__ double rowsum[KC], rowabs[KC];
  if (!st_sum_value(ks, part, nblk, red, &last, tot)) return;
  const int t = threadIdx.x;
  if (it == 0) {   // frame start: y from the handle, flags cleared
    if (t < kMaxK) st_set_y(ks, t, (t < a.k) ? a.y[t] : 0.0);
    if (t == 0) {
      ks->stop = ks->bad = ks->upd = ks->steps = ks->restarts = 0;
      a.stats->frame = *a.nframe;
    }
    __syncthreads();
  }
  if (t < 64) st_dir_core<KC>(a, ks, tot, it);
  __syncthreads();
  if (ks->stop || ks->bad) return;
  if (t < KC) {
    int q = KC + 1 + t * KC - t * (t - 1) / 2;   // H[t][t]
    double s = tot[q] * ks->d[t] * ks->d[t], b = fabs(s);
    for (int l = t + 1; l < KC; ++l) {
      const double v = 2.0 * tot[++q] * ks->d[t] * ks->d[l];
      s += v;
      b += fabs(v);
    }
    rowsum[t] = s;
    rowabs[t] = b;
  }
  __syncthreads();
  double dHd = 0.0, mag = 0.0;
  for (int r = 0; r < KC; ++r) {
    dHd += rowsum[r];
    mag += rowabs[r];
  }
  if (dHd < 0x1p-48 * mag) dHd = 0x1p-48 * mag;
  st_adv_core(a, ks, dHd, it);
}

// Step 2 eta pass at the final y: eta = -w phi'(r) stored per entry;
// partials of U^T eta, ||eta||^2 and the final cost: float32 over the pixels of
// one group, float64 over the groups.
template <int KC, typename TS, bool PAIR>
__global__ __launch_bounds__(kStBlock) void st_eta(FrameArgs a, const StreamKS* __restrict__ ks, float* __restrict__ eta,
                                                   double* __restrict__ part, int nchunk) {
  constexpr int N = StPix<TS, PAIR>::N;
  constexpr int L = KC + 2;
  if (ks->bad) return;
  __shared__ float ys[KC], yl[KC];
  __shared__ double red[kStWaves][L];
  const int tid = thread_index(), lane = tid & 63, wv = tid >> 6;
  if (tid < KC) st_get_y(a, ks, false, tid, ys, yl);
  __syncthreads();
  double sum = 0.0;
  int comp = 0;
  for (int ch = blockIdx.x; ch < nchunk; ch += gridDim.x) {
    const int p0 = (ch * kStBlock + tid) * N;
    const bool valid = p0 < a.P;
    float wt[N], acc[L];
#pragma unroll
    for (int j = 0; j < L; ++j) acc[j] = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) wt[i] = valid ? st_weight(a, p0 + i) : 0.f;
    for (int c = 0; valid && c < a.C; ++c) {
      float u[N][KC], x[N];
      st_load<KC, TS, PAIR>(a, c, p0, u, x);
      const long long e = (long long)c * a.P + p0;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const float r = st_residual<KC>(x[i], u[i], ys, yl);
        float phi, cc;
        cost_eval(r, a.cp, phi, cc);
        const float et = -wt[i] * cc * r;
        eta[e + i] = et;
        acc[KC] = fmaf(et, et, acc[KC]);
        acc[KC + 1] = fmaf(wt[i], phi, acc[KC + 1]);
#pragma unroll
        for (int j = 0; j < KC; ++j) acc[j] = fmaf(et, u[i][j], acc[j]);
      }
    }
    sum += (double)wave_reduce_scatter<L>(acc, comp);
  }
  if (wave_rs_owner<L>(lane) && comp < L) red[wv][comp] = sum;
  __syncthreads();
  if (tid < L) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kStWaves; ++w) s += red[w][tid];
    part[(size_t)tid * gridDim.x + blockIdx.x] = s;
  }
}

// Sums of the eta pass, then the geodesic scalars (Sec. 3.3 Step 2, Sec. 3.4
// step size) as geodesic_setup forms them, and the end of the frame: y and the
// frame counter (an accepted frame only; the update pass needs neither).
template <int KC>
__global__ __launch_bounds__(kStBlock) void st_geodesic(FrameArgs a, StreamKS* ks, const double* __restrict__ part,
                                                        int nblk) {
  if (ks->bad) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      a.stats->bad_frame = 1;
      a.sync[4] = 0;
    }
    return;
  }
  __shared__ double red[kStWaves];
  __shared__ int last;
  __shared__ double tot[kStWide];
  if (!st_sum_value(ks, part, nblk, red, &last, tot)) return;
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    const double av = (lane < a.k) ? tot[lane] : 0.0;
    const double yv = (lane < a.k) ? ks->y[lane] : 0.0;
    const double aa = row16_sum(av * av);
    const double yy = row16_sum(yv * yv);
    const double ee = tot[KC];
    const double zeta = sqrt(fmax(ee - aa, 0.0));
    const double nu = sqrt(yy);
    const double sigma = zeta * nu;
    const int upd = (zeta > 0.0 && nu > 0.0) ? 1 : 0;
    if (lane < kMaxK) {
      ks->af[lane] = (float)av;
      ks->vf[lane] = upd ? (float)(yv / nu) : 0.f;
    }
    if (lane < a.k) a.y[lane] = yv;
    if (lane == 0) {
      const long long n = *a.nframe;
      const double t = step_size(a.tau * (double)n, a.t_init, a.t_min);
      const GeoScalars g = geodesic_scalars(t, sigma, zeta);
      ks->cm1 = upd ? (float)g.cm1 : 0.f;
      ks->sz = upd ? (float)g.sz : 0.f;
      ks->nu = (float)nu;
      ks->upd = upd;
      const int steps = ks->steps;
      a.stats->f[steps] = tot[KC + 1];
      a.stats->cg_steps = steps;
      a.stats->restarts = ks->restarts;
      a.stats->t = t;
      a.stats->sigma = sigma;
      a.stats->theta = g.theta;
      a.stats->zeta = zeta;
      a.stats->nu = nu;
      a.stats->updated = upd;
      a.stats->bad_frame = 0;
      *a.nframe = n + 1;
      a.sync[4] = 0;   // the mask is no longer the labels' median
    }
  }
}

// Rank-one geodesic update of every row and the pixel labels (Step 3), one
// pass: u <- u + coef v with coef = (cos theta - 1)(u.v) - (sin theta / zeta)
// (eta - u.a); r' = r - coef nu (r' = x - U' y); label = any channel with
// |r'| >= delta.
template <int KC, typename TS, bool PAIR>
__global__ __launch_bounds__(kStBlock) void st_update(FrameArgs a, const StreamKS* __restrict__ ks,
                                                      const float* __restrict__ eta) {
  constexpr int N = StPix<TS, PAIR>::N;
  if (ks->bad) return;
  __shared__ float ys[KC], yl[KC], vs[KC], as[KC];
  const int tid = thread_index();
  if (tid < KC) {
    ys[tid] = ks->yf[tid];
    yl[tid] = ks->yl[tid];
    vs[tid] = ks->vf[tid];
    as[tid] = ks->af[tid];
  }
  __syncthreads();
  const int p0 = (blockIdx.x * kStBlock + tid) * N;
  if (p0 >= a.P) return;
  const float cm1 = ks->cm1, sz = ks->sz, nu = ks->nu;
  const bool upd = ks->upd != 0;
  uint8_t label[N];
#pragma unroll
  for (int i = 0; i < N; ++i) label[i] = 0;
  for (int c = 0; c < a.C; ++c) {
    float u[N][KC], x[N];
    st_load<KC, TS, PAIR>(a, c, p0, u, x);
    const long long e = (long long)c * a.P + p0;
    float un[N][KC];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      float r = st_residual<KC>(x[i], u[i], ys, yl);
      if (upd) {
        float uv = 0.f, ua = 0.f;
#pragma unroll
        for (int j = 0; j < KC; ++j) {
          uv = fmaf(u[i][j], vs[j], uv);
          ua = fmaf(u[i][j], as[j], ua);
        }
        const float coef = fmaf(cm1, uv, -sz * (eta[e + i] - ua));
#pragma unroll
        for (int j = 0; j < KC; ++j) un[i][j] = fmaf(coef, vs[j], u[i][j]);
        if (a.labels_after_update) r = fmaf(-coef, nu, r);
      }
      if (fabsf(r) >= a.delta) label[i] = 1;
    }
    if (upd) {
      if constexpr (PAIR) {
        uint32_t* __restrict__ U = (uint32_t*)a.U;
#pragma unroll
        for (int j = 0; j < KC; ++j)
          if (j < a.k) U[((long long)j * a.ldU + e) >> 1] = pack_bf16_rne(un[0][j], un[1][j]);
      } else {
        TS* __restrict__ U = (TS*)a.U;
#pragma unroll
        for (int j = 0; j < KC; ++j)
          if (j < a.k) st_elem(U, (long long)j * a.ldU + e, un[0][j]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i) a.lab[p0 + i] = label[i];
}

// One frame: nchunk groups of kStBlock threads, each thread one pixel (or one
// pixel pair with PAIR).
template <int KC, typename TS, bool PAIR>
static void st_frame_launch(const FrameArgs& a, StreamKS* ks, float* eta, double* part, int nchunk, hipStream_t s) {
  const int nblk = st_blocks(nchunk);
  for (int it = 0; it < a.J; ++it) {
    hipLaunchKernelGGL((st_grad<KC, TS, PAIR>), dim3(nblk), dim3(kStBlock), 0, s, a, (const StreamKS*)ks, part, nchunk,
                       it == 0);
    hipLaunchKernelGGL((st_step<KC>), dim3(st_nh<KC>()), dim3(kStBlock), 0, s, a, ks, (const double*)part, nblk, it);
  }
  hipLaunchKernelGGL((st_eta<KC, TS, PAIR>), dim3(nblk), dim3(kStBlock), 0, s, a, (const StreamKS*)ks, eta, part,
                     nchunk);
  hipLaunchKernelGGL((st_geodesic<KC>), dim3(KC + 2), dim3(kStBlock), 0, s, a, ks, (const double*)part, nblk);
  hipLaunchKernelGGL((st_update<KC, TS, PAIR>), dim3(nchunk), dim3(kStBlock), 0, s, a, (const StreamKS*)ks,
                     (const float*)eta);
}

template <typename TS, bool PAIR>
static void st_frame_class(int kc, const FrameArgs& a, StreamKS* ks, float* eta, double* part, int nchunk,
                           hipStream_t s) {
  switch (kc) {
    case 2: st_frame_launch<2, TS, PAIR>(a, ks, eta, part, nchunk, s); break;
    case 4: st_frame_launch<4, TS, PAIR>(a, ks, eta, part, nchunk, s); break;
    case 5: st_frame_launch<5, TS, PAIR>(a, ks, eta, part, nchunk, s); break;
    case 8: st_frame_launch<8, TS, PAIR>(a, ks, eta, part, nchunk, s); break;
    case 10: st_frame_launch<10, TS, PAIR>(a, ks, eta, part, nchunk, s); break;
    case 12: st_frame_launch<12, TS, PAIR>(a, ks, eta, part, nchunk, s); break;
    case 15: st_frame_launch<15, TS, PAIR>(a, ks, eta, part, nchunk, s); break;
    default: st_frame_launch<16, TS, PAIR>(a, ks, eta, part, nchunk, s); break;
  }
}

static int st_class(int k) {
  return k <= 2 ? 2 : k <= 4 ? 4 : k <= 5 ? 5 : k <= 8 ? 8 : k <= 10 ? 10 : k <= 12 ? 12 : k <= 15 ? 15 : 16;
}

}  // namespace prost

// Device buffers of the streamed path: k-space state, per-entry eta,
// per-workgroup partials.
pros_status prost_stream_alloc(pros_handle* h) {
  using namespace prost;
  const int nchunk = (h->P + kStBlock - 1) / kStBlock;   // one pixel per thread; pairs need half
  const int nblk = std::min(nchunk, kStResident);
  const size_t bytes = sizeof(StreamKS) + sizeof(float) * (size_t)h->m + sizeof(double) * (size_t)nblk * kStWide + 1024;
  hipError_t e = hipMalloc(&h->stream_ws, bytes);
  if (e != hipSuccess) return prost_host::set_error(PROS_ENOMEM, "streamed-frame buffers: %s", hipGetErrorString(e));
  e = hipMemsetAsync(h->stream_ws, 0, bytes, h->stream);
  if (e != hipSuccess) return prost_host::set_error(PROS_EHIP, "streamed-frame buffers: %s", hipGetErrorString(e));
  h->stream_groups = nchunk;
  return PROS_OK;
}

pros_status prost_stream_frame(pros_handle* h, const prost::FrameArgs& a) {
  using namespace prost;
  char* base = (char*)h->stream_ws;
  StreamKS* ks = (StreamKS*)base;
  float* eta = (float*)(base + ((sizeof(StreamKS) + 255) / 256) * 256);
  double* part = (double*)(((uintptr_t)(eta + h->m) + 255) / 256 * 256);
  const int kc = st_class(h->k);
  if (h->prm.storage == PROS_BF16) {
    // pixel pairs: even P and every plane start 4-byte aligned (U's planes
    // are ldU apart with ldU a multiple of 64; the frame is the caller's)
    const bool pair = h->P % 2 == 0 && h->ldU % 2 == 0 && ((uintptr_t)a.x & 3u) == 0 && ((uintptr_t)a.U & 3u) == 0;
    if (pair)
      st_frame_class<uint16_t, true>(kc, a, ks, eta, part, (h->P / 2 + kStBlock - 1) / kStBlock, h->stream);
    else
      st_frame_class<uint16_t, false>(kc, a, ks, eta, part, h->stream_groups, h->stream);
  } else {
    st_frame_class<float, false>(kc, a, ks, eta, part, h->stream_groups, h->stream);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    h->broken = true;
    h->broken_status = PROS_EHIP;
    return prost_host::set_error(PROS_EHIP, "streamed frame launch failed: %s", hipGetErrorString(e));
  }
  return PROS_OK;
}
