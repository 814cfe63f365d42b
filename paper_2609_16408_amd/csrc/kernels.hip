// Kernels around the Sternheimer solve: Galerkin initial guess, density
// accumulation, Lanczos recurrence with full reorthogonalisation,
// tridiagonal Gauss quadrature and frequency integration.
#include "internal.h"

#include <algorithm>

namespace rpa {

namespace {

// ---------------------------------------------------------------------------
__global__ void k_fill_d(double* p, double v, long long n) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    p[i] = v;
}
__global__ void k_fill_i(int* p, int v, long long n) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    p[i] = v;
}
__global__ void k_d2f(const double* __restrict__ a, float* __restrict__ b, long long n) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    b[i] = (float)a[i];
}
__global__ void k_set_onehot(double* q, long long stride, const long long* idx, int B) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) q[(size_t)b * stride + idx[b]] = 1.0;
}

// ---------------------------------------------------------------------------
// Galerkin projection, part 1: part[b][c][m][n] = sum_{r in chunk c} psi_m psi_n u_b,
// a contraction over grid points on the FP64 matrix cores (v_mfma_f64_16x16x4:
// A lane l = row l%16, k l/16; B lane l = column l%16, k l/16; D register v of
// lane l = row l/16 + 4v, column l%16).  Each wave owns a tile of 16 TM x 16 TN
// outputs of one chunk and takes its operands straight from global memory: per
// step of 16 points a lane loads the four points 4 l/16 .. + 3 of its row (32
// contiguous bytes, 128 per row and four lanes), and product q contracts
// points q, q + 4, q + 8, q + 12 of all lanes, the same ones in A and B.
// Tiles follow the orbital counts: four orbitals cost one 16-wide tile.
// The workgroups of a chunk are dealt to one XCD, whose L2 then serves its
// psi rows to all start vectors and tiles.
// Bound by the matrix cores at 512 x 128 states; 48^3, 16 start vectors:
// 8.6 -> 4.0 ms (58 TFLOP/s) against 128 x 128 tiles through LDS; 12^3, 4 states:
// 332 -> 6 us, 24^3, 16 states, 64 vectors: 694 -> 36 us.
typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
constexpr int kXcds = 8;

// index of this workgroup's chunk (possibly past the last one) and its rank in the chunk
__device__ __forceinline__ void xcd_chunk(int per_chunk, int& chunk, int& rank) {
  const int x = blockIdx.x % kXcds, k = blockIdx.x / kXcds;
  chunk = x + kXcds * (k / per_chunk);
  rank = k % per_chunk;
}
inline unsigned xcd_grid(int chunks, int per_chunk) {
  return (unsigned)((chunks + kXcds - 1) / kXcds * kXcds * per_chunk);
}

template <int TM, int TN>
__global__ void __launch_bounds__(256, 2) k_gram(const double* __restrict__ psi,
                                                 const double* __restrict__ u, int B, int n_occ, int ng,
                                                 long long N, int n_chunks, double* __restrict__ part) {
  const int ntm = (ng + 16 * TM - 1) / (16 * TM), ntn = (n_occ + 16 * TN - 1) / (16 * TN);
  const int jobs = B * ntm * ntn;
  int c, rank;
  xcd_chunk((jobs + 3) / 4, c, rank);
  const int job = rank * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (c >= n_chunks || job >= jobs) return;
  const int b = job / (ntm * ntn), tile = job - b * ntm * ntn;
  const int m0 = tile / ntn * 16 * TM, n0 = tile % ntn * 16 * TN;
  const long long clen = ((N + n_chunks - 1) / n_chunks + 15) & ~15LL;
  const long long r0 = c * clen, r1 = r0 + clen < N ? r0 + clen : N;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const double* ub = u + (size_t)b * N;
  const double* pm[TM];
  const double* pn[TN];
#pragma unroll
  for (int t = 0; t < TM; ++t) {
    const int m = m0 + 16 * t + li;
    pm[t] = psi + (size_t)(m < ng ? m : ng - 1) * N;       // repeated rows are not stored
  }
#pragma unroll
  for (int t = 0; t < TN; ++t) {
    const int n = n0 + 16 * t + li;
    pn[t] = psi + (size_t)(n < n_occ ? n : n_occ - 1) * N;
  }
  d4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  auto load = [&](const double* p, long long r, bool full) {
    d4 v;
    if (full) {
      const d2u x = *reinterpret_cast<const d2u*>(p + r), y = *reinterpret_cast<const d2u*>(p + r + 2);
      v = d4{x[0], x[1], y[0], y[1]};
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = r + q < r1 ? p[r + q] : 0.0;
    }
    return v;
  };
  auto step = [&](long long rb, bool full) {
    const long long r = rb + 4 * lk;
    const d4 uu = load(ub, r, full);
    d4 a[TM], bb[TN];
#pragma unroll
    for (int t = 0; t < TM; ++t) a[t] = load(pm[t], r, full);
#pragma unroll
    for (int t = 0; t < TN; ++t) bb[t] = load(pn[t], r, full);
#pragma unroll
    for (int t = 0; t < TM; ++t) a[t] *= uu;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][q], bb[j][q], acc[i][j], 0, 0, 0);
  };
  long long rb = r0;
  for (; rb + 16 <= r1; rb += 16) step(rb, true);
  if (rb < r1) step(rb, false);
  double* out = part + ((size_t)b * n_chunks + c) * ng * n_occ;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + 16 * j + li;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + 16 * i + lk + 4 * v;
        if (m < ng && n < n_occ) out[(size_t)m * n_occ + n] = acc[i][j][v];
      }
    }
  }
}

// part 2: G[b][m][n] = (-dV sum_c part) / (eps_m - eps_n - i omega_b), m over the
// ng Galerkin states (occupied first), n over the occupied ones
__global__ void k_gram_finish(const double* __restrict__ part, int B, int n_occ, int ng, int n_chunks,
                              double dV, const double* __restrict__ eps,
                              const double* __restrict__ omega, double2* __restrict__ G) {
  const long long total = (long long)B * ng * n_occ;
  for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < total;
       t += (long long)gridDim.x * blockDim.x) {
    const int b = (int)(t / ((long long)ng * n_occ));
    const long long mn = t - (long long)b * ng * n_occ;
    const int m = (int)(mn / n_occ), n = (int)(mn % n_occ);
    double s = 0.0;
    for (int c = 0; c < n_chunks; ++c) s += part[((size_t)b * n_chunks + c) * ng * n_occ + mn];
    const double cm = -dV * s;
    const double dr = eps[m] - eps[n];
    const double di = -omega[b];
    const double den = dr * dr + di * di;
    G[t] = make_double2(cm * dr / den, -cm * di / den);
  }
}

// part 3: x64[(b*n_occ + n)][r] = sum_m psi_m(r) G[b][m][n], m over the ng states,
// on the FP64 matrix cores with rows n, columns r and the real and imaginary
// parts of G as two A operands that share psi.  Each wave owns 16 TN orbitals
// x 64 grid points; the workgroups of a point range are dealt to one XCD.
// Bound by the matrix cores at 512 x 128 states: 48^3, 16 start vectors,
// 13.3 -> 10.2 ms (46 TFLOP/s) against vector FP64 tiles through LDS.
constexpr int kExpandPoints = 64;        // grid points of a k_expand workgroup
template <int TN>
__global__ void __launch_bounds__(256, 2) k_expand(const double* __restrict__ psi,
                                                   const double2* __restrict__ G, int B, int n_occ, int ng,
                                                   long long N, long long c0, double2* __restrict__ x64) {
  constexpr int TR = kExpandPoints / 16;
  const int ntn = (n_occ + 16 * TN - 1) / (16 * TN);
  const int jobs = B * ntn;
  int c, rank;
  xcd_chunk((jobs + 3) / 4, c, rank);
  const int job = rank * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const long long r0 = (c0 + c) * kExpandPoints;
  if (r0 >= N || job >= jobs) return;
  const int b = job / ntn, n0 = job % ntn * 16 * TN;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const double2* Gb = G + (size_t)b * ng * n_occ;
  d4 re[TN][TR], im[TN][TR];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TR; ++j) re[i][j] = im[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  long long rc[TR];
  int nc[TN];
#pragma unroll
  for (int j = 0; j < TR; ++j) rc[j] = r0 + 16 * j + li < N ? r0 + 16 * j + li : N - 1;   // not stored
#pragma unroll
  for (int i = 0; i < TN; ++i) nc[i] = n0 + 16 * i + li < n_occ ? n0 + 16 * i + li : n_occ - 1;
#pragma unroll 2
  for (int m0 = 0; m0 < ng; m0 += 4) {
    const int m = m0 + lk, mc = m < ng ? m : ng - 1;
    double2 g[TN];
    double p[TR];
#pragma unroll
    for (int i = 0; i < TN; ++i) g[i] = Gb[(size_t)mc * n_occ + nc[i]];
#pragma unroll
    for (int j = 0; j < TR; ++j) p[j] = psi[(size_t)mc * N + rc[j]];
    if (m >= ng) {
#pragma unroll
      for (int i = 0; i < TN; ++i) g[i] = make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TR; ++j) {
        re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(g[i].x, p[j], re[i][j], 0, 0, 0);
        im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(g[i].y, p[j], im[i][j], 0, 0, 0);
      }
  }
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int n = n0 + 16 * i + lk + 4 * v;
      if (n >= n_occ) continue;
      double2* dst = x64 + ((size_t)b * n_occ + n) * N;
#pragma unroll
      for (int j = 0; j < TR; ++j) {
        const long long r = r0 + 16 * j + li;
        if (r < N) dst[r] = make_double2(re[i][j][v], im[i][j][v]);
      }
    }
}

// racc[b][r] = 4 sum_n psi_n(r) Re x64[b][n][r]
__global__ void k_accumulate(const double* __restrict__ psi, const double2* __restrict__ x64,
                             int B, int n_occ, long long N, const int* __restrict__ active,
                             double* __restrict__ racc) {
  const long long total = (long long)B * N;
  for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < total;
       t += (long long)gridDim.x * blockDim.x) {
    const int b = (int)(t / N);
    const long long r = t - (long long)b * N;
    double s = 0.0;
    if (active == nullptr || active[b]) {
      const double2* xb = x64 + (size_t)b * n_occ * N;
      for (int n = 0; n < n_occ; ++n) s += psi[(size_t)n * N + r] * xb[(size_t)n * N + r].x;
    }
    racc[t] = 4.0 * s;
  }
}

// ---------------------------------------------------------------------------
// Lanczos step k for start vector b = blockIdx.x (one workgroup each):
//   alpha_k = q_k^T v;  v -= alpha_k q_k + beta_{k-1} q_{k-1};
//   two classical Gram-Schmidt passes against q_0..q_k;
//   if k < m-1: beta_k = ||v||, breakdown if beta_k <= brk * max|alpha|,
//   else q_{k+1} = v / beta_k.
// lane-0 broadcast into scalar registers: wave-uniform control flow around barriers
__device__ __forceinline__ int uni_i(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double uni_d(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffLL));
  const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

__device__ double lz_block_sum(double x, double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  if (lane == 0) red[wave] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += red[w];
    red[64] = s;
  }
  __syncthreads();
  const double r = uni_d(red[64]);
  __syncthreads();
  return r;
}

__global__ void __launch_bounds__(1024) k_lanczos_step(int k, int m_total, int B, long long N,
                                                       double* __restrict__ Q,
                                                       double* __restrict__ v,
                                                       double* __restrict__ alpha,
                                                       double* __restrict__ beta,
                                                       int* __restrict__ mlen,
                                                       int* __restrict__ active, double brk) {
  __shared__ double red[72];
  __shared__ double coef[kMaxLanczos];
  const int b = blockIdx.x;
  if (!uni_i(active[b])) return;
  // Q layout [m_total][B][N]: q_j of start vector b at Q + (j*B + b)*N
  const size_t qs = (size_t)B * N;
  double* Qb = Q + (size_t)b * N;
  double* vb = v + (size_t)b * N;
  const double* qk = Qb + (size_t)k * qs;
  double s = 0.0;
  for (long long i = threadIdx.x; i < N; i += blockDim.x) s += qk[i] * vb[i];
  const double a = lz_block_sum(s, red);
  const double bprev = k > 0 ? beta[(size_t)b * m_total + k - 1] : 0.0;
  const double* qkm = k > 0 ? Qb + (size_t)(k - 1) * qs : nullptr;
  for (long long i = threadIdx.x; i < N; i += blockDim.x) {
    double t = vb[i] - a * qk[i];
    if (k > 0) t -= bprev * qkm[i];
    vb[i] = t;
  }
  __syncthreads();
  for (int pass = 0; pass < 2; ++pass) {
    for (int j = 0; j <= k; ++j) {
      const double* qj = Qb + (size_t)j * qs;
      double sj = 0.0;
      for (long long i = threadIdx.x; i < N; i += blockDim.x) sj += qj[i] * vb[i];
      const double cj = lz_block_sum(sj, red);
      if (threadIdx.x == 0) coef[j] = cj;
    }
    __syncthreads();
    for (long long i = threadIdx.x; i < N; i += blockDim.x) {
      double t = vb[i];
      for (int j = 0; j <= k; ++j) t -= coef[j] * Qb[(size_t)j * qs + i];
      vb[i] = t;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) alpha[(size_t)b * m_total + k] = a;
  if (k < m_total - 1) {
    double s2 = 0.0;
    for (long long i = threadIdx.x; i < N; i += blockDim.x) s2 += vb[i] * vb[i];
    const double bk = sqrt(lz_block_sum(s2, red));
    double amax = 0.0;
    for (int j = 0; j < k; ++j) amax = fmax(amax, fabs(alpha[(size_t)b * m_total + j]));
    amax = uni_d(fmax(amax, fabs(a)));
    if (bk <= brk * amax) {
      if (threadIdx.x == 0) { mlen[b] = k + 1; active[b] = 0; }
      return;
    }
    const double inv = 1.0 / bk;
    double* qn = Qb + (size_t)(k + 1) * qs;
    for (long long i = threadIdx.x; i < N; i += blockDim.x) qn[i] = vb[i] * inv;
    if (threadIdx.x == 0) { beta[(size_t)b * m_total + k] = bk; mlen[b] = k + 2; }
  } else {
    if (threadIdx.x == 0) mlen[b] = k + 1;
  }
}

// ---------------------------------------------------------------------------
// Symmetric tridiagonal eigenproblem by the implicit-shift QL iteration
// (Bowdler, Martin, Reinsch and Wilkinson, 1968), tracking only the first
// row of the eigenvector matrix; then [f(T)]_11 = sum_i z_i^2 f(lambda_i).
__device__ __host__ inline int ql_first_row(int n, double* d, double* e, double* z) {
  for (int i = 0; i < n; ++i) z[i] = (i == 0) ? 1.0 : 0.0;
  if (n == 1) return 0;
  e[n - 1] = 0.0;
  for (int l = 0; l < n; ++l) {
    int iter = 0;
    int m;
    for (;;) {
      for (m = l; m < n - 1; ++m) {
        const double dd = fabs(d[m]) + fabs(d[m + 1]);
        if (fabs(e[m]) <= 2.2e-16 * dd) break;
      }
      if (m == l) break;
      if (++iter > 100) return 1;
      double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
      double r = hypot(g, 1.0);
      g = d[m] - d[l] + e[l] / (g + (g >= 0.0 ? fabs(r) : -fabs(r)));
      double s = 1.0, c = 1.0, p = 0.0;
      int i;
      bool underflow = false;
      for (i = m - 1; i >= l; --i) {
        double f = s * e[i];
        const double bb = c * e[i];
        r = hypot(f, g);
        e[i + 1] = r;
        if (r == 0.0) {
          d[i + 1] -= p;
          e[m] = 0.0;
          underflow = true;
          break;
        }
        s = f / r;
        c = g / r;
        g = d[i + 1] - p;
        r = (d[i] - g) * s + 2.0 * c * bb;
        p = s * r;
        d[i + 1] = g + p;
        g = c * r - bb;
        f = z[i + 1];
        z[i + 1] = s * z[i] + c * f;
        z[i] = c * z[i] - s * f;
      }
      if (underflow) continue;
      d[l] -= p;
      e[l] = g;
      e[m] = 0.0;
    }
  }
  return 0;
}

__global__ void k_tridiag_quad(int B, int m_total, const double* __restrict__ alpha,
                               const double* __restrict__ beta, const int* __restrict__ mlen,
                               const long long* __restrict__ out_pos, double* __restrict__ dout,
                               int* __restrict__ fail) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  double d[kMaxLanczos], e[kMaxLanczos], z[kMaxLanczos];
  const int m = mlen[b];
  for (int i = 0; i < m; ++i) d[i] = alpha[(size_t)b * m_total + i];
  for (int i = 0; i + 1 < m; ++i) e[i] = beta[(size_t)b * m_total + i];
  const int bad = ql_first_row(m, d, e, z);
  double acc = 0.0;
  for (int i = 0; i < m; ++i) acc += z[i] * z[i] * (log1p(-d[i]) + d[i]);
  dout[out_pos ? out_pos[b] : b] = acc;
  if (bad) atomicAdd(&fail[0], 1);
  if (m < m_total) atomicAdd(&fail[1], 1);
}

__global__ void k_scatter(const double* __restrict__ src, const long long* __restrict__ pos, int n,
                          double* __restrict__ dst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[pos[i]] = src[i];
}

// ---------------------------------------------------------------------------
// e_fine[j] = scale_fine * sum_k w_k dhat_k[j];  partials[block] = sum_j sum_k w_k dhat_k[j]
__global__ void __launch_bounds__(256) k_weighted_sum(const double* __restrict__ dhat,
                                                     const double* __restrict__ w, int n_omega,
                                                     long long N, double scale_fine,
                                                     double* __restrict__ e_fine,
                                                     double* __restrict__ partials) {
  __shared__ double red[8];
  const long long per = (N + gridDim.x - 1) / gridDim.x;
  const long long j0 = blockIdx.x * per;
  const long long j1 = j0 + per < N ? j0 + per : N;
  double s = 0.0;
  for (long long j = j0 + threadIdx.x; j < j1; j += blockDim.x) {
    double t = 0.0;
    for (int k = 0; k < n_omega; ++k) t += w[k] * dhat[(size_t)k * N + j];
    s += t;
    if (e_fine) e_fine[j] = scale_fine * t;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += red[i];
    partials[blockIdx.x] = t;
  }
}

int grid_for(long long n, int block) {
  long long g = (n + block - 1) / block;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (int)g;
}

}  // namespace

hipError_t launch_fill_d(double* p, double v, long long n, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_d, dim3(grid_for(n, 256)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}
hipError_t launch_fill_i(int* p, int v, long long n, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_i, dim3(grid_for(n, 256)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}
hipError_t launch_d2f(const double* a, float* b, long long n, hipStream_t s) {
  hipLaunchKernelGGL(k_d2f, dim3(grid_for(n, 256)), dim3(256), 0, s, a, b, n);
  return hipGetLastError();
}
hipError_t launch_set_onehot(double* q, long long stride, const long long* idx, int B, hipStream_t s) {
  hipLaunchKernelGGL(k_set_onehot, dim3((B + 63) / 64), dim3(64), 0, s, q, stride, idx, B);
  return hipGetLastError();
}

int gram_chunks(long long N, int n_occ, int ng) {
  // enough chunks to fill the chip at any batch size (the sums must not depend
  // on the batch): at least 2048 points each, or 128 where the partial sums
  // then stay below one vector per start vector
  const long long few = std::max<long long>(1, N / 2048);
  const long long many = std::min<long long>(N / 128, N / ((long long)ng * n_occ));
  return (int)std::min<long long>(64, std::max(few, many));
}
hipError_t launch_gram(const double* psi, const double* u, int B, int n_occ, int ng, long long N,
                       int n_chunks, double* part, hipStream_t s) {
  const int tm = ng <= 16 ? 1 : (ng <= 32 ? 2 : 4), tn = n_occ <= 16 ? 1 : (n_occ <= 32 ? 2 : 4);
  const long long jobs = (long long)B * ((ng + 16 * tm - 1) / (16 * tm)) * ((n_occ + 16 * tn - 1) / (16 * tn));
  const dim3 grid(xcd_grid(n_chunks, (int)((jobs + 3) / 4)));
#define RPA_GRAM(TM, TN)                                                                             \
  if (tm == TM && tn == TN)                                                                          \
    hipLaunchKernelGGL((k_gram<TM, TN>), grid, dim3(256), 0, s, psi, u, B, n_occ, ng, N, n_chunks, part);
  RPA_GRAM(1, 1) RPA_GRAM(1, 2) RPA_GRAM(1, 4) RPA_GRAM(2, 1) RPA_GRAM(2, 2) RPA_GRAM(2, 4) RPA_GRAM(4, 1)
  RPA_GRAM(4, 2) RPA_GRAM(4, 4)
#undef RPA_GRAM
  return hipGetLastError();
}
hipError_t launch_gram_finish(const double* part, int B, int n_occ, int ng, int n_chunks, double dV,
                              const double* eps, const double* omega, double2* G, hipStream_t s) {
  const long long total = (long long)B * ng * n_occ;
  hipLaunchKernelGGL(k_gram_finish, dim3(grid_for(total, 256)), dim3(256), 0, s, part, B, n_occ, ng,
                     n_chunks, dV, eps, omega, G);
  return hipGetLastError();
}
hipError_t launch_expand(const double* psi, const double2* G, int B, int n_occ, int ng, long long N,
                         double2* x64, hipStream_t s) {
  const int tn = n_occ <= 16 ? 1 : 2;
  const long long ntn = (n_occ + 16 * tn - 1) / (16 * tn), chunks = (N + kExpandPoints - 1) / kExpandPoints;
  // a grid's threads are counted in 32 bits: ranges of start vectors, then of
  // points in whole rounds of the XCDs, of at most kMost workgroups
  constexpr long long kMost = 1LL << 23;
  const int nb = (int)std::min<long long>(B, std::max(1LL, kMost / kXcds * 4 / ntn));
  for (int b0 = 0; b0 < B; b0 += nb) {
    const int bn = std::min(nb, B - b0);
    const long long per_chunk = (bn * ntn + 3) / 4, span = std::max(1LL, kMost / kXcds / per_chunk) * kXcds;
    const double2* Gb = G + (size_t)b0 * ng * n_occ;
    double2* xb = x64 + (size_t)b0 * n_occ * N;
    for (long long c0 = 0; c0 < chunks; c0 += span) {
      const dim3 grid(xcd_grid((int)std::min(span, chunks - c0), (int)per_chunk));
      if (tn == 1)
        hipLaunchKernelGGL((k_expand<1>), grid, dim3(256), 0, s, psi, Gb, bn, n_occ, ng, N, c0, xb);
      else
        hipLaunchKernelGGL((k_expand<2>), grid, dim3(256), 0, s, psi, Gb, bn, n_occ, ng, N, c0, xb);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}
hipError_t launch_accumulate(const double* psi, const double2* x64, int B, int n_occ, long long N,
                             const int* active, double* racc, hipStream_t s) {
  hipLaunchKernelGGL(k_accumulate, dim3(grid_for((long long)B * N, 256)), dim3(256), 0, s, psi,
                     x64, B, n_occ, N, active, racc);
  return hipGetLastError();
}
hipError_t launch_lanczos_step(int k, int m_total, int B, long long N, double* Q, double* v,
                               double* alpha, double* beta, int* mlen, int* active, double brk,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_lanczos_step, dim3(B), dim3(1024), 0, s, k, m_total, B, N, Q, v, alpha, beta,
                     mlen, active, brk);
  return hipGetLastError();
}
hipError_t launch_tridiag_quad(int B, int m_total, const double* alpha, const double* beta,
                                const int* mlen, const long long* out_pos, double* d, int* fail,
                                hipStream_t s) {
  hipLaunchKernelGGL(k_tridiag_quad, dim3((B + 63) / 64), dim3(64), 0, s, B, m_total, alpha, beta,
                     mlen, out_pos, d, fail);
  return hipGetLastError();
}

hipError_t launch_scatter(const double* src, const long long* pos, int n, double* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_scatter, dim3((n + 255) / 256), dim3(256), 0, s, src, pos, n, dst);
  return hipGetLastError();
}

hipError_t launch_weighted_sum(const double* dhat, const double* w, int n_omega, long long N,
                               double scale_fine, double* e_fine, double* partials, int nblocks,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_weighted_sum, dim3(nblocks), dim3(256), 0, s, dhat, w, n_omega, N,
                     scale_fine, e_fine, partials);
  return hipGetLastError();
}

}  // namespace rpa
