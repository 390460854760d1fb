// Re-orthonormalisation of U in float64 on the GPU (precision form).
//
// U drifts off the Stiefel manifold (Sec. 2.1, eq. stiefeldef) when it is
// stored in float32 or bfloat16.  Since only span(U) matters (Sec. 3.2), U is
// replaced by its nearest orthonormal matrix, the polar factor
//   U <- U G^{-1/2},  G = U^T U,
// and y <- G^{1/2} y keeps U y unchanged to first order.  Three kernels:
//   gram_partial: per-workgroup float64 partial sums of the upper triangle of G
//   gram_solve:   fixed-order sum, Jacobi eigensolver of G in one wavefront
//                 (float64), G^{-1/2}, G^{1/2} y
//   gram_apply:   u_e <- u_e G^{-1/2} in float64, rounded to storage
// Both passes over U run their products on the float64 matrix instruction.
#include <hip/hip_runtime.h>

#include "prost_device.hpp"
#include "prost_host.hpp"

namespace prost {

constexpr int kGramPairs = kMaxK * (kMaxK + 1) / 2;
constexpr int kGramBlocks = 256;      // one workgroup of 8 wavefronts per compute unit
constexpr int kGramThreads = 512;
constexpr int kGramWaves = kGramThreads / 64;
constexpr int kSolveThreads = 1024;

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// Elements of one column that a lane takes at a time: 16 bytes of the storage
// types (their planes are 16-byte aligned), one of the float64 initialization
// matrix (its planes are m apart, m arbitrary).
template <typename TS>
constexpr int gram_vec() { return sizeof(TS) == 8 ? 1 : 16 / (int)sizeof(TS); }

template <typename TS>
__device__ __forceinline__ void gram_load(const TS* __restrict__ col, long long r, long long m, bool on,
                                          double (&v)[gram_vec<TS>()]) {
  constexpr int V = gram_vec<TS>();
  if constexpr (V > 1) {
    if (on && r + V <= m) {
      const uint4 w = *(const uint4*)(col + r);
      const uint32_t q[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int i = 0; i < V; ++i)
        v[i] = (double)(sizeof(TS) == 4 ? __uint_as_float(q[i & 3])
                                        : __uint_as_float((i & 1) ? (q[i >> 1] & 0xFFFF0000u) : (q[i >> 1] << 16)));
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < V; ++i) v[i] = (on && r + i < m) ? (double)ld_elem(col, r + i) : 0.0;
}

// Partial sums of the upper triangle of G = U^T U, pair (i, j) at
// part[block * kGramPairs + ...], row by row.  G is a contraction over the rows
// with both operands U: lane l holds column l % 16 of some rows in float64, and
// v_mfma_f64_16x16x4 with that one register as both operands adds the products
// of its four lane groups' rows (the order of rows within the sum is free, so a
// lane's rows can be the 16 contiguous bytes that it loads).  Products are
// exact in float64 and accumulation is float64, as before; the order is fixed.
// Bound by the latency of the reads of U.  With a float64 LDS tile and one pair
// per thread it was bound by LDS reads (640x480x3, k = 15, bfloat16: 63 us;
// this form 18, and 22 in float32: 2.5 TB/s).
template <typename TS>
__global__ __launch_bounds__(kGramThreads) void gram_partial(const TS* __restrict__ U, long long ldU, long long m,
                                                             int k, double* __restrict__ part) {
  constexpr int V = gram_vec<TS>();
  __shared__ double red[kGramWaves][256];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int j = lane & 15;
  const bool on = j < k;
  const TS* col = U + (long long)(on ? j : 0) * ldU;
  f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
  const long long step = (long long)gridDim.x * kGramWaves * 4 * V;
  for (long long r0 = ((long long)blockIdx.x * kGramWaves + wv) * 4 * V; r0 < m; r0 += 2 * step) {
    const long long r = r0 + (lane >> 4) * V;
    double v0[V], v1[V];
    gram_load(col, r, m, on, v0);
    gram_load(col, r + step, m, on, v1);   // all zero past the end
#pragma unroll
    for (int i = 0; i < V; ++i) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v0[i], v0[i], acc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < V; ++i) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v1[i], v1[i], acc, 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) red[wv][(4 * i + (lane >> 4)) * 16 + j] = acc[i];   // row 4 i + lane / 16, column lane % 16
  __syncthreads();
  if (threadIdx.x < 256) {
    const int row = threadIdx.x >> 4, cl = threadIdx.x & 15;
    if (row <= cl && cl < k) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < kGramWaves; ++w) s += red[w][threadIdx.x];
      part[(size_t)blockIdx.x * kGramPairs + row * k - row * (row - 1) / 2 + (cl - row)] = s;
    }
  }
}

// Fixed-order sum of the workgroups' partials into the symmetric G (LDS), by
// kSolveThreads threads: seven per pair, each every seventh workgroup, their
// sums added in order.  (One wavefront with a pair per lane read 512 partials
// one after the other: most of 0.1 ms.)
__device__ __forceinline__ void gram_sum(const double* __restrict__ part, int nblocks, int k,
                                         double (*G)[kMaxK], double* __restrict__ buf) {
  constexpr int kGroups = kSolveThreads / kGramPairs;
  const int np = k * (k + 1) / 2;
  const int q = threadIdx.x % kGramPairs, g = threadIdx.x / kGramPairs;
  if (g < kGroups && q < np) {
    double s = 0.0;
#pragma unroll 8
    for (int b = g; b < nblocks; b += kGroups) s += part[(size_t)b * kGramPairs + q];
    buf[g * kGramPairs + q] = s;
  }
  __syncthreads();
  if (threadIdx.x < (unsigned)np) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kGroups; ++i) s += buf[i * kGramPairs + threadIdx.x];
    int t = threadIdx.x, i = 0;
    while (t >= k - i) { t -= k - i; ++i; }
    G[i][i + t] = s;
    G[i + t][i] = s;
  }
  __syncthreads();
}

// Orders the LDS accesses of one wavefront (they execute in order; this keeps
// the compiler from moving them).
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// G^{-1/2} into ws (row-major k x k, stride 16) and y <- G^{1/2} y, from an
// eigendecomposition of G by Jacobi rotations in float64, one wavefront after
// the sum of the partials.  The rotations of a sweep go in the round-robin
// order: n / 2 disjoint pairs at a time (n: k rounded up to even), whose angles
// n / 2 lanes form together and whose two-sided update is one 2 x 2 block per
// lane.  The chain of divisions and roots is what bounds it, and it is paid
// n - 1 times per sweep instead of k (k - 1) / 2 times: at k = 15 the kernel
// took 825 us with one pair at a time and takes 57-72.
__global__ __launch_bounds__(kSolveThreads) void gram_solve(const double* __restrict__ part, int nblocks, int k,
                                                            double* __restrict__ y, double* __restrict__ ws) {
  __shared__ double A[kMaxK][kMaxK];
  __shared__ double Vm[kMaxK][kMaxK];
  __shared__ double cs[kMaxK / 2][2];
  __shared__ double buf[(kSolveThreads / kGramPairs) * kGramPairs];
  if (threadIdx.x < kMaxK * kMaxK) {
    const int i = threadIdx.x / kMaxK, j = threadIdx.x % kMaxK;
    Vm[i][j] = (i == j) ? 1.0 : 0.0;
    if (i >= k || j >= k) A[i][j] = (i == j) ? 1.0 : 0.0;   // pads an odd k: never rotated
  }
  gram_sum(part, nblocks, k, A, buf);
  if (threadIdx.x >= 64) return;
  const int l = threadIdx.x;
  const int n = (k + 1) & ~1, half = n / 2;
  const int bi = l >> 3, bj = l & 7;
  for (int sweep = 0; sweep < 30 && k > 1; ++sweep) {
    double off = 0.0, dia = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = l >> 2, j = 4 * (l & 3) + c;
      const double v = (i < k && j < k) ? A[i][j] * A[i][j] : 0.0;
      if (i == j) dia += v;
      else off += v;
    }
    off = wave_sum(off);
    dia = wave_sum(dia);
    if (!(off > 1e-32 * dia)) break;
    for (int s = 0; s < n - 1; ++s) {
      // pair i of step s: (n - 1, s) for i = 0, ((s + i) mod (n - 1), (s - i) mod (n - 1)) else
      auto first = [&](int i) { return i == 0 ? n - 1 : s + i >= n - 1 ? s + i - (n - 1) : s + i; };
      auto second = [&](int i) { return s - i < 0 ? s - i + n - 1 : s - i; };
      if (l < half) {
        const int p = first(l), q = second(l);
        const double apq = A[p][q], th = A[q][q] - A[p][p], d = 2.0 * apq;
        double c = 1.0, sn = 0.0;
        const double den = fabs(th) + sqrt(fma(th, th, d * d));
        // den is 0 where th is 0 and d^2 underflows (|apq| below 2^-538): as good as
        // rotated, and 0 / 0 would spoil the whole decomposition
        if (apq != 0.0 && den > 0.0) {   // t = sgn(tau) / (|tau| + sqrt(1 + tau^2)), tau = th / d
          const double t = (th >= 0.0 ? d : -d) / den;
          c = rsqrt(fma(t, t, 1.0));
          sn = t * c;
        }
        cs[l][0] = c;
        cs[l][1] = sn;
      }
      wave_fence();
      if (bi < half && bj < half) {   // A <- J^T A J, the 2 x 2 block of pairs bi (rows) and bj (columns)
        const int p = first(bi), q = second(bi), u = first(bj), v = second(bj);
        const double ci = cs[bi][0], si = cs[bi][1], cj = cs[bj][0], sj = cs[bj][1];
        const double a = A[p][u], b = A[p][v], c = A[q][u], d = A[q][v];
        const double a1 = cj * a - sj * b, b1 = sj * a + cj * b;
        const double c1 = cj * c - sj * d, d1 = sj * c + cj * d;
        // a pair's own off-diagonal is 0 by the choice of its angle; as computed it
        // would keep rounding of the diagonal (2^-53 of it), above the bound of the
        // sweeps, all 30 of which would then run
        A[p][u] = ci * a1 - si * c1;
        A[p][v] = bi == bj ? 0.0 : ci * b1 - si * d1;
        A[q][u] = bi == bj ? 0.0 : si * a1 + ci * c1;
        A[q][v] = si * b1 + ci * d1;
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {   // V <- V J, row l % 16, pairs l / 16 and l / 16 + 4
        const int i = (l >> 4) + 4 * h, r = l & 15;
        if (i < half) {
          const int p = first(i), q = second(i);
          const double c = cs[i][0], sn = cs[i][1];
          const double vp = Vm[r][p], vq = Vm[r][q];
          Vm[r][p] = c * vp - sn * vq;
          Vm[r][q] = sn * vp + c * vq;
        }
      }
      wave_fence();
    }
  }
  // G^{-1/2} = V diag(lam^{-1/2}) V^T, G^{1/2} y = V diag(lam^{1/2}) V^T y
  const double lam = (l < k) ? A[l][l] : 1.0;
  if (__any(!(lam > 1e-300))) {   // rank-deficient U: leave U and y unchanged
    if (l < k)
      for (int j = 0; j < k; ++j) ws[l * kMaxK + j] = (l == j) ? 1.0 : 0.0;
    return;
  }
  double* root = buf;              // sqrt(lam), then its reciprocal at 16, V^T y scaled at 32
  if (l < kMaxK) {
    root[l] = sqrt(lam);
    root[kMaxK + l] = 1.0 / sqrt(lam);
  }
  wave_fence();
  if (l < k) {
    double t = 0.0;
    for (int i = 0; i < k; ++i) t = fma(Vm[i][l], y[i], t);
    root[2 * kMaxK + l] = root[l] * t;
  }
  wave_fence();
  for (int q = l; q < k * k; q += 64) {
    const int i = q / k, j = q - i * k;
    double t = 0.0;
    for (int c = 0; c < k; ++c) t = fma(Vm[i][c] * root[kMaxK + c], Vm[j][c], t);
    ws[i * kMaxK + j] = t;
  }
  if (l < k) {
    double t = 0.0;
    for (int c = 0; c < k; ++c) t = fma(Vm[l][c], root[2 * kMaxK + c], t);
    y[l] = t;
  }
}

// u_e <- u_e G^{-1/2} for every row, in float64, rounded to the storage type.
// The transposed product M^T U^T goes through v_mfma_f64_16x16x4: M (symmetric)
// stays in four registers, and the result has lane l % 16 = row, so a lane
// that takes two adjacent rows stores them as one word into each plane.  Bound
// by the read and the write of U; with one row per thread it was bound by the
// K^2 reads of M from LDS per row (640x480x3, k = 15, bfloat16: 31 us; now 21).
template <typename TS>
__global__ __launch_bounds__(256) void gram_apply(TS* __restrict__ U, long long ldU, int m, int k,
                                                  const double* __restrict__ ws) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int lo = lane & 15, hi = lane >> 4;
  double M[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) M[s] = (4 * s + hi < k && lo < k) ? ws[(4 * s + hi) * kMaxK + lo] : 0.0;
  for (long long r0 = ((long long)blockIdx.x * 4 + wv) * 32; r0 < m; r0 += (long long)gridDim.x * 128) {
    const long long r = r0 + 2 * lo;   // rows r, r + 1 (one word of every plane: ldU is a multiple of 64)
    const bool in = r < m;
    double u[4][2];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      float a = 0.f, b = 0.f;
      if (in && 4 * s + hi < k) {
        const TS* p = U + (long long)(4 * s + hi) * ldU + r;
        if constexpr (sizeof(TS) == 2) {
          const uint32_t w = *(const uint32_t*)p;
          a = __uint_as_float(w << 16);
          b = __uint_as_float(w & 0xFFFF0000u);
        } else {
          const float2 w = *(const float2*)p;
          a = w.x;
          b = w.y;
        }
      }
      u[s][0] = (double)a;
      u[s][1] = (double)b;
    }
    f64x4_t d0 = {0.0, 0.0, 0.0, 0.0}, d1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      d0 = __builtin_amdgcn_mfma_f64_16x16x4f64(M[s], u[s][0], d0, 0, 0, 0);
      d1 = __builtin_amdgcn_mfma_f64_16x16x4f64(M[s], u[s][1], d1, 0, 0, 0);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {      // column 4 c + lane / 16 of rows r, r + 1
      const int j = 4 * c + hi;
      if (!in || j >= k) continue;
      TS* p = U + (long long)j * ldU + r;
      if (r + 1 < m) {
        if constexpr (sizeof(TS) == 2)
          *(uint32_t*)p = (uint32_t)f32_to_bf16_rne((float)d0[c]) | ((uint32_t)f32_to_bf16_rne((float)d1[c]) << 16);
        else
          *(float2*)p = make_float2((float)d0[c], (float)d1[c]);
      } else {
        st_elem(p, 0, (float)d0[c]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Initialization of U (Sec. 3.4): the orthonormal factor of the reduced QR
// decomposition of a random m x k matrix A.  A is drawn on the device from a
// counter-based generator (Philox4x32-10, Salmon et al., SC'11) with
// Box-Muller, so that the draw is reproducible per (seed, stream) and
// independent of the launch; Q = A R^{-1} comes from CholeskyQR2 in float64
// (two passes of G = A^T A, G = R^T R, A <- A R^{-1}), whose R has a
// positive diagonal, i.e. the QR factor with diag(R) > 0.
// ---------------------------------------------------------------------------

__device__ __forceinline__ void philox_round10(uint32_t (&c)[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int rnd = 0; rnd < 10; ++rnd) {
    if (rnd) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const unsigned long long a = (unsigned long long)c[0] * 0xD2511F53ull;
    const unsigned long long b = (unsigned long long)c[2] * 0xCD9E8D57ull;
    const uint32_t w0 = (uint32_t)(b >> 32) ^ c[1] ^ k0;
    const uint32_t w2 = (uint32_t)(a >> 32) ^ c[3] ^ k1;
    c[1] = (uint32_t)b;
    c[3] = (uint32_t)a;
    c[0] = w0;
    c[2] = w2;
  }
}

// Entry e = j m + i of the column-major m x k matrix: pair q = e / 2 is one
// generator call with counter (q lo, q hi, stream, 0) and key (seed lo, seed
// hi); its two 64-bit words give uniforms (z / 2^11 + 1/2) 2^-53 in (0, 1),
// and Box-Muller gives the cosine (even e) and sine (odd e) normal variates.
__global__ __launch_bounds__(256) void gauss_fill(double* __restrict__ A, long long n, unsigned long long seed,
                                                  uint32_t stream_index) {
  const long long npair = (n + 1) / 2;
  for (long long q = (long long)blockIdx.x * 256 + threadIdx.x; q < npair; q += (long long)gridDim.x * 256) {
    uint32_t c[4] = {(uint32_t)q, (uint32_t)((unsigned long long)q >> 32), stream_index, 0u};
    philox_round10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    const unsigned long long za = (((unsigned long long)c[0] << 32) | c[1]) >> 11;
    const unsigned long long zb = (((unsigned long long)c[2] << 32) | c[3]) >> 11;
    const double ua = ((double)za + 0.5) * 0x1p-53;
    const double ub = ((double)zb + 0.5) * 0x1p-53;
    const double rad = sqrt(-2.0 * log(ua));
    const double ang = 2.0 * 3.141592653589793 * ub;
    A[2 * q] = rad * cos(ang);
    if (2 * q + 1 < n) A[2 * q + 1] = rad * sin(ang);
  }
}

// G from the partials (fixed order), Cholesky G = R^T R (R
// upper, by lane 0 in float64), R^{-1} (upper) into ws (k x k, stride 16).
// A non-positive pivot (rank-deficient A) sets *bad and leaves ws = I.
__global__ __launch_bounds__(kSolveThreads) void qr_chol_inv(const double* __restrict__ part, int nblocks, int k,
                                                  double* __restrict__ ws, int* __restrict__ bad) {
  __shared__ double G[kMaxK][kMaxK];
  __shared__ double R[kMaxK][kMaxK];
  __shared__ double Ri[kMaxK][kMaxK];
  __shared__ double buf[(kSolveThreads / kGramPairs) * kGramPairs];
  const int l = threadIdx.x;
  gram_sum(part, nblocks, k, G, buf);
  if (l == 0) {
    int ok = 1;
    for (int i = 0; i < k && ok; ++i) {
      for (int j = 0; j < k; ++j) R[i][j] = 0.0;
      double d = G[i][i];
      for (int r = 0; r < i; ++r) d -= R[r][i] * R[r][i];
      if (!(d > 0.0)) { ok = 0; break; }
      const double rii = sqrt(d);
      R[i][i] = rii;
      for (int j = i + 1; j < k; ++j) {
        double v = G[i][j];
        for (int r = 0; r < i; ++r) v -= R[r][i] * R[r][j];
        R[i][j] = v / rii;
      }
    }
    // R^{-1} by back substitution, column by column
    for (int j = k - 1; ok && j >= 0; --j) {
      for (int i = 0; i < k; ++i) Ri[i][j] = 0.0;
      Ri[j][j] = 1.0 / R[j][j];
      for (int i = j - 1; i >= 0; --i) {
        double v = 0.0;
        for (int r = i + 1; r <= j; ++r) v += R[i][r] * Ri[r][j];
        Ri[i][j] = -v / R[i][i];
      }
    }
    for (int i = 0; i < kMaxK; ++i)
      for (int j = 0; j < kMaxK; ++j)
        ws[i * kMaxK + j] = (i < k && j < k) ? (ok ? Ri[i][j] : (i == j ? 1.0 : 0.0)) : 0.0;
    if (!ok) *bad = 1;
  }
}

// a_e <- a_e R^{-1} for every row of the float64 m x k matrix (in place).
template <int K>
__global__ __launch_bounds__(256) void qr_apply_f64(double* __restrict__ A, long long m,
                                                    const double* __restrict__ ws) {
  __shared__ double M[K][K];
  for (int q = threadIdx.x; q < K * K; q += 256) M[q / K][q % K] = ws[(q / K) * kMaxK + (q % K)];
  __syncthreads();
  for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < m; e += (long long)gridDim.x * 256) {
    int z = 0;
    asm volatile("" : "+v"(z));   // keeps the reads of M in the loop (K K / 2 doubles would not fit the registers)
    const double* Ml = &M[0][0] + z;
    double a[K];
#pragma unroll
    for (int i = 0; i < K; ++i) a[i] = A[(long long)i * m + e];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      double s = 0.0;
#pragma unroll
      for (int i = 0; i <= j; ++i) s = fma(a[i], Ml[i * K + j], s);   // R^{-1} is upper triangular
      A[(long long)j * m + e] = s;
    }
  }
}

// U (storage type, leading dimension ldU) <- A rounded to nearest.
template <typename TS>
__global__ __launch_bounds__(256) void store_subspace(TS* __restrict__ U, long long ldU, const double* __restrict__ A,
                                                      long long m, int k) {
  for (long long q = (long long)blockIdx.x * 256 + threadIdx.x; q < m * k; q += (long long)gridDim.x * 256) {
    const long long j = q / m, e = q - j * m;
    st_elem(U, j * ldU + e, (float)A[q]);
  }
}

static hipError_t qr_apply_launch(int k, double* A, long long m, const double* ws, int blocks, hipStream_t st) {
#define PROST_QR_CASE(KK) \
  case KK: hipLaunchKernelGGL((qr_apply_f64<KK>), dim3(blocks), dim3(256), 0, st, A, m, ws); break;
  switch (k) {
    PROST_QR_CASE(1) PROST_QR_CASE(2) PROST_QR_CASE(3) PROST_QR_CASE(4)
    PROST_QR_CASE(5) PROST_QR_CASE(6) PROST_QR_CASE(7) PROST_QR_CASE(8)
    PROST_QR_CASE(9) PROST_QR_CASE(10) PROST_QR_CASE(11) PROST_QR_CASE(12)
    PROST_QR_CASE(13) PROST_QR_CASE(14) PROST_QR_CASE(15) PROST_QR_CASE(16)
    default: return hipErrorInvalidValue;
  }
#undef PROST_QR_CASE
  return hipGetLastError();
}

}  // namespace prost

// The seeded orthonormal m x k matrix into A (device, float64, column-major,
// leading dimension m), on `st`; synchronises.  Scratch is allocated here.
pros_status prost_random_subspace(unsigned long long seed, uint32_t stream_index, long long m, int k, double* A,
                                  hipStream_t st) {
  using namespace prost;
  if (m < k || k < 1 || k > PROS_MAX_K) return prost_host::set_error(PROS_EINVAL, "need 1 <= k <= min(m, %d)", PROS_MAX_K);
  const int nb = (int)std::min<long long>(kGramBlocks, (m + 255) / 256);
  double* part = nullptr;
  hipError_t e = hipMalloc((void**)&part, sizeof(double) * ((size_t)kGramBlocks * kGramPairs + 256) + 64);
  if (e != hipSuccess) return prost_host::set_error(PROS_ENOMEM, "initialization scratch: %s", hipGetErrorString(e));
  double* ws = part + (size_t)kGramBlocks * kGramPairs;
  int* bad = (int*)(ws + 256);
  const long long n = m * k;
  const int fb = (int)std::min<long long>(4096, ((n + 1) / 2 + 255) / 256);
  const int ab = (int)std::min<long long>(2048, (m + 255) / 256);
  e = hipMemsetAsync(bad, 0, sizeof(int), st);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(gauss_fill, dim3(fb), dim3(256), 0, st, A, n, seed, stream_index);
    for (int pass = 0; pass < 2 && e == hipSuccess; ++pass) {
      hipLaunchKernelGGL((gram_partial<double>), dim3(nb), dim3(kGramThreads), 0, st, (const double*)A, m, m, k, part);
      hipLaunchKernelGGL(qr_chol_inv, dim3(1), dim3(kSolveThreads), 0, st, (const double*)part, nb, k, ws, bad);
      e = qr_apply_launch(k, A, m, ws, ab, st);
    }
  }
  int hbad = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  (void)hipFree(part);
  if (e != hipSuccess) return prost_host::set_error(PROS_EHIP, "initialization of U: %s", hipGetErrorString(e));
  if (hbad) return prost_host::set_error(PROS_EINVAL, "random matrix is rank-deficient (m=%lld, k=%d)", m, k);
  return PROS_OK;
}

// U of a handle <- the seeded orthonormal matrix rounded to the storage type.
pros_status prost_init_subspace(pros_handle* h, unsigned long long seed, uint32_t stream_index) {
  using namespace prost;
  double* A = nullptr;
  hipError_t e = hipMalloc((void**)&A, sizeof(double) * (size_t)h->m * h->k);
  if (e != hipSuccess) return prost_host::set_error(PROS_ENOMEM, "initialization buffer: %s", hipGetErrorString(e));
  pros_status st = prost_random_subspace(seed, stream_index, h->m, h->k, A, h->stream);
  if (st == PROS_OK) {
    const int sb = (int)std::min<long long>(4096, ((long long)h->m * h->k + 255) / 256);
    if (h->prm.storage == PROS_BF16)
      hipLaunchKernelGGL((store_subspace<uint16_t>), dim3(sb), dim3(256), 0, h->stream, (uint16_t*)h->U, h->ldU,
                         (const double*)A, (long long)h->m, h->k);
    else
      hipLaunchKernelGGL((store_subspace<float>), dim3(sb), dim3(256), 0, h->stream, (float*)h->U, h->ldU,
                         (const double*)A, (long long)h->m, h->k);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) st = prost_host::set_error(PROS_EHIP, "initialization store: %s", hipGetErrorString(e));
  }
  (void)hipFree(A);
  return st;
}

pros_status prost_reorth_launch(pros_handle* h) {
  using namespace prost;
  const int nb = (int)std::min<long long>(kGramBlocks, ((long long)h->m + 255) / 256);
  if (!h->reorth_ws) {
    hipError_t e = hipMalloc(&h->reorth_ws, sizeof(double) * ((size_t)kGramBlocks * kGramPairs + 256));
    if (e != hipSuccess) return prost_host::set_error(PROS_ENOMEM, "re-orthonormalisation workspace: %s", hipGetErrorString(e));
  }
  double* part = (double*)h->reorth_ws;
  double* ws = part + (size_t)kGramBlocks * kGramPairs;
  const bool bf = h->prm.storage == PROS_BF16;
  if (bf)
    hipLaunchKernelGGL((gram_partial<uint16_t>), dim3(nb), dim3(kGramThreads), 0, h->stream, (const uint16_t*)h->U, h->ldU,
                       (long long)h->m, h->k, part);
  else
    hipLaunchKernelGGL((gram_partial<float>), dim3(nb), dim3(kGramThreads), 0, h->stream, (const float*)h->U, h->ldU,
                       (long long)h->m, h->k, part);
  hipLaunchKernelGGL(gram_solve, dim3(1), dim3(kSolveThreads), 0, h->stream, (const double*)part, nb, h->k, h->y, ws);
  const int ab = (int)std::min<long long>(2048, ((long long)h->m + 127) / 128);
  if (bf)
    hipLaunchKernelGGL((gram_apply<uint16_t>), dim3(ab), dim3(256), 0, h->stream, (uint16_t*)h->U, h->ldU, h->m, h->k,
                       (const double*)ws);
  else
    hipLaunchKernelGGL((gram_apply<float>), dim3(ab), dim3(256), 0, h->stream, (float*)h->U, h->ldU, h->m, h->k,
                       (const double*)ws);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    h->broken = true;
    h->broken_status = PROS_EHIP;
    return prost_host::set_error(PROS_EHIP, "re-orthonormalisation launch failed: %s", hipGetErrorString(e));
  }
  return PROS_OK;
}
