// Separable per-axis transforms of batches of real 3D arrays: the Kronecker
// form of nu^1/2 and nu, the kinetic preconditioner plan and the separable
// interpolants.
//
// Two kernels on the FP64 matrix cores (v_mfma_f64_16x16x4) cover every
// array whose dimensions are at most kMaxTransformDim: k_plane contracts the
// last two axes of one (d1, d2) plane, k_cols the first axis of a column
// block, there and back where a diagonal scale sits in between.  A full
// forward-scale-inverse transform is three launches that each read and write
// the batch once.  Larger arrays take k_axis, one axis per launch.
//
// The accumulator of this instruction holds row l/16 + 4v, column l%16 in
// lane l, register v; its B operand holds k = l/16, column l%16.  So a
// product's accumulator tile IS the B operand of the next product for
// k = 4v .. 4v+3, and both contractions of a kernel chain in registers.
// Measured against one k_axis launch per axis (which re-reads a line of
// inputs through the caches for every output): nu^1/2 of 64 vectors on 48^3
// 2226 -> 143 us, M^-1 of 16 complex vectors on 24x24x48 268 -> 44 us.
#include "internal.h"

namespace rpa {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// out[i][j] = sum_a L[a][i] (sum_b X[a][b] R[b][j]) for PL planes per
// workgroup, X a plane of na x nb values (RA = ceil(na / 16) row tiles).  R
// and L are stored k-major and zero-padded to multiples of 16.  Each wave
// owns 16 columns j of every plane of the workgroup.
//
// Bound by the matrix cores' operand supply at cell sizes (a 48^3 plane: 72
// instructions per wave and plane, each with one LDS or L1 operand), by
// launch latency below.  Two planes per workgroup share every basis operand
// read; one where that would leave compute units without a workgroup.
template <int RA, int PL, bool ENERGY>
__global__ void __launch_bounds__(512) k_plane(const double* __restrict__ in, double* __restrict__ out,
                                               long long planes, int na, int nb, int ni, int nj,
                                               const double* __restrict__ Rm,
                                               const double* __restrict__ Lm, int ld, double scale,
                                               double* __restrict__ partials) {
  extern __shared__ double sx[];
  __shared__ double red[8];
  const int kb = (nb + 15) & ~15, oj = (nj + 15) & ~15, oi = (ni + 15) & ~15;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const long long p0 = (long long)blockIdx.x * PL;
  const int np = planes - p0 < PL ? (int)(planes - p0) : PL;
  const int slab = RA * 16 * ld;
  for (int p = 0; p < np; ++p) {
    const double* src = in + (size_t)(p0 + p) * na * nb;
    double* dst = sx + p * slab;
    // four rows' loads in flight per wave
    for (int a = wave; a < RA * 16; a += 4 * nw)
      for (int b = lane; b < kb; b += 64) {
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = (a + u * nw < na && b < nb) ? src[(a + u * nw) * nb + b] : 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (a + u * nw < RA * 16) dst[(a + u * nw) * ld + b] = v[u];
      }
  }
  __syncthreads();
  double esum = 0.0;
  for (int j0 = wave * 16; j0 < oj; j0 += nw * 16) {
    d4 t[PL][RA];
#pragma unroll
    for (int p = 0; p < PL; ++p)
#pragma unroll
      for (int r = 0; r < RA; ++r) t[p][r] = d4{0.0, 0.0, 0.0, 0.0};
    const double* bp = Rm + (size_t)lk * oj + j0 + li;
    const double* ap = sx + li * ld + lk;
    for (int k0 = 0; k0 < kb; k0 += 16) {
      double b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) b[q] = bp[(size_t)(k0 + 4 * q) * oj];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int p = 0; p < PL; ++p)
#pragma unroll
          for (int r = 0; r < RA; ++r) t[p][r] = mma(ap[p * slab + r * 16 * ld + k0 + 4 * q], b[q], t[p][r]);
    }
    for (int i0 = 0; i0 < oi; i0 += 16) {
      const double* lp = Lm + (size_t)lk * oi + i0 + li;
      d4 acc[PL];
#pragma unroll
      for (int p = 0; p < PL; ++p) acc[p] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int r = 0; r < RA; ++r)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double l = lp[(size_t)(16 * r + 4 * v) * oi];
#pragma unroll
          for (int p = 0; p < PL; ++p) acc[p] = mma(l, t[p][r][v], acc[p]);
        }
#pragma unroll
      for (int p = 0; p < PL; ++p) {
        if (p >= np || j0 + li >= nj) continue;
        double* dst = out ? out + (size_t)(p0 + p) * ni * nj + j0 + li : nullptr;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = i0 + lk + 4 * v;
          if (i >= ni) continue;
          if constexpr (ENERGY) {
            esum += acc[p][v];
            if (dst) dst[(size_t)i * nj] = scale * acc[p][v];
          } else {
            dst[(size_t)i * nj] = acc[p][v];
          }
        }
      }
    }
  }
  if constexpr (ENERGY) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) esum += __shfl_xor(esum, off, 64);
    if (lane == 0) red[wave] = esum;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s = 0.0;
      for (int w = 0; w < nw; ++w) s += red[w];
      partials[blockIdx.x] = s;
    }
  }
}

// Small host values that travel with the launch: the weights of the frequency
// sum folded into an interpolation's first pass (a), or the shifts of a
// kinetic solve (a + i b).  n = 0: the shifts are in device memory.
struct ColsArgs {
  int n;
  double a[kMaxFieldWeights], b[kMaxFieldWeights];
};

enum ColsMode {
  COLS_ONCE,                   // out = A1^T X            (n_in rows -> n_out rows)
  COLS_FIELDS,                 // the same of sum_f w_f X_f
  COLS_SCALE,                  // out = A2^T (s .* (A1^T X)), real diagonal s[row][column]
  COLS_KINETIC                 // ... complex diagonal 1 / (s[row][column] + sigma_b) over the
};                             // real and imaginary fields of vector b

// One wave per 16 * NC columns of one array (COLS_KINETIC: the same 16
// columns of the real and of the imaginary field): X's whole columns are
// loaded as B operands and everything after stays in registers.  Each row
// of a load or store is a 128 B segment; the matrix operands come from L1,
// one read per NC products.
template <int RK, int NC, int MODE>
__global__ void __launch_bounds__(256) k_cols(const double* __restrict__ in, double* __restrict__ out, int n_in,
                                              int n_out, int ncol, const double* __restrict__ A1,
                                              const double* __restrict__ A2, const double* __restrict__ diag,
                                              const double* __restrict__ sig_re,
                                              const double* __restrict__ sig_im, ColsArgs fw) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  constexpr int CW = MODE == COLS_KINETIC ? 16 : 16 * NC;   // columns of a wave
  const int c0 = ((int)blockIdx.x * nw + wave) * CW;
  if (c0 >= ncol) return;
  const size_t isz = (size_t)n_in * ncol, osz = (size_t)n_out * ncol;
  const int o1 = MODE == COLS_SCALE || MODE == COLS_KINETIC ? n_in : n_out;
  const int op = (o1 + 15) & ~15;
  const size_t b = blockIdx.y;
  const double* src[NC];
  double* dst[NC];
  int col[NC];
  bool ok[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int cc = MODE == COLS_KINETIC ? c0 + li : c0 + 16 * c + li;
    ok[c] = cc < ncol;
    col[c] = ok[c] ? cc : 0;
    const size_t f = MODE == COLS_KINETIC ? 2 * b + c : b;
    src[c] = in + f * isz + col[c];
    dst[c] = out + f * osz + col[c];
  }
  double x[NC][RK * 4];
  if constexpr (MODE == COLS_FIELDS) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int q = 0; q < RK * 4; ++q) x[c][q] = 0.0;
  }
  // one field's loads are all in flight together
  for (int f = 0; f < (MODE == COLS_FIELDS ? fw.n : 1); ++f) {
#pragma unroll
    for (int q = 0; q < RK * 4; ++q) {
      const int r = 4 * q + lk;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const double v = r < n_in && ok[c] ? src[c][f * isz + (size_t)r * ncol] : 0.0;
        if constexpr (MODE == COLS_FIELDS) x[c][q] += fw.a[f] * v;
        else x[c][q] = v;
      }
    }
  }
  if constexpr (MODE == COLS_ONCE || MODE == COLS_FIELDS) {
    for (int i0 = 0; i0 < op; i0 += 16) {
      const double* ap = A1 + (size_t)lk * op + i0 + li;
      d4 acc[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[c] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < RK * 4; ++q) {
        const double a = ap[(size_t)4 * q * op];
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = mma(a, x[c][q], acc[c]);
      }
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = i0 + lk + 4 * v;
          if (i < n_out && ok[c]) dst[c][(size_t)i * ncol] = acc[c][v];
        }
    }
  } else {
    d4 t[NC][RK];
#pragma unroll
    for (int m = 0; m < RK; ++m) {
      const double* ap = A1 + (size_t)lk * op + 16 * m + li;
#pragma unroll
      for (int c = 0; c < NC; ++c) t[c][m] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < RK * 4; ++q) {
        const double a = ap[(size_t)4 * q * op];
#pragma unroll
        for (int c = 0; c < NC; ++c) t[c][m] = mma(a, x[c][q], t[c][m]);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 16 * m + lk + 4 * v;      // mode; rows past n_in are zero
        if constexpr (MODE == COLS_SCALE) {
#pragma unroll
          for (int c = 0; c < NC; ++c)
            t[c][m][v] *= r < n_in ? diag[(size_t)r * ncol + col[c]] : 0.0;
        } else {
          const double dr = (r < n_in ? diag[(size_t)r * ncol + col[0]] : 0.0) + (fw.n ? fw.a[b] : sig_re[b]);
          const double di = fw.n ? fw.b[b] : sig_im[b];
          const double den = dr * dr + di * di;
          const double xr = t[0][m][v], xi = t[1][m][v];
          t[0][m][v] = (xr * dr + xi * di) / den;
          t[1][m][v] = (xi * dr - xr * di) / den;
        }
      }
    }
    for (int i0 = 0; i0 < op; i0 += 16) {
      const double* ap = A2 + (size_t)lk * op + i0 + li;
      d4 acc[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[c] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int m = 0; m < RK; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double a = ap[(size_t)(16 * m + 4 * v) * op];
#pragma unroll
          for (int c = 0; c < NC; ++c) acc[c] = mma(a, t[c][m][v], acc[c]);
        }
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = i0 + lk + 4 * v;
          if (i < n_in && ok[c]) dst[c][(size_t)i * ncol] = acc[c][v];
        }
    }
  }
}

// ---------------------------------------------------------------------------
// Per-axis transform of arrays with a dimension beyond kMaxTransformDim:
// out[b, ..., i, ...] = sum_k M(i, k) in[b, ..., k, ...]
__global__ void k_axis(const double* __restrict__ in, double* __restrict__ out, int B, int d0,
                       int d1, int d2, int axis, int n_out, const double* __restrict__ M,
                       int trans, const double* __restrict__ scale) {
  int od0 = d0, od1 = d1, od2 = d2;
  if (axis == 0) od0 = n_out; else if (axis == 1) od1 = n_out; else od2 = n_out;
  const long long osz = (long long)od0 * od1 * od2;
  const long long isz = (long long)d0 * d1 * d2;
  const long long total = osz * B;
  const int n_in = axis == 0 ? d0 : (axis == 1 ? d1 : d2);
  for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < total;
       t += (long long)gridDim.x * blockDim.x) {
    const long long b = t / osz;
    const long long o = t - b * osz;
    const int i2 = (int)(o % od2);
    const long long o01 = o / od2;
    const int i1 = (int)(o01 % od1);
    const int i0 = (int)(o01 / od1);
    const double* src = in + b * isz;
    long long base, stride;
    int i;
    if (axis == 0) { i = i0; base = (long long)i1 * d2 + i2; stride = (long long)d1 * d2; }
    else if (axis == 1) { i = i1; base = (long long)i0 * d1 * d2 + i2; stride = d2; }
    else { i = i2; base = ((long long)i0 * d1 + i1) * d2; stride = 1; }
    double acc = 0.0;
    if (trans) {
      for (int k = 0; k < n_in; ++k) acc += M[(long long)k * n_out + i] * src[base + k * stride];
    } else {
      const double* row = M + (long long)i * n_in;
      for (int k = 0; k < n_in; ++k) acc += row[k] * src[base + k * stride];
    }
    if (scale) acc *= scale[o];
    out[t] = acc;
  }
}

// Complex diagonal solve in the eigenbasis of the FD Laplacian, the middle
// step of the shifted kinetic preconditioner: vector b is stored planar
// (N real parts, then N imaginary parts) and each mode o is divided by
// kin[o] + sigma_b, kin >= 0 the kinetic eigenvalue, Re(sigma_b) > 0.
__global__ void k_kin_scale(double* __restrict__ a, const double* __restrict__ kin,
                            const double* __restrict__ sig_re, const double* __restrict__ sig_im,
                            int B, long long N) {
  const long long total = (long long)B * N;
  for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < total;
       t += (long long)gridDim.x * blockDim.x) {
    const long long b = t / N;
    const long long o = t - b * N;
    double* re = a + b * 2 * N;
    double* im = re + N;
    const double dr = kin[o] + sig_re[b];
    const double di = sig_im[b];
    const double den = dr * dr + di * di;
    const double xr = re[o], xi = im[o];
    re[o] = (xr * dr + xi * di) / den;
    im[o] = (xi * dr - xr * di) / den;
  }
}

int grid_of(long long n) {
  const long long g = (n + 255) / 256;
  return (int)(g > 65536 ? 65536 : (g < 1 ? 1 : g));
}

// Largest row tiles of the forms that work on two planes or column blocks at
// once: beyond, their tiles need more registers than a wave has.
constexpr int kPairTiles = 5;

template <int PL, bool ENERGY>
hipError_t plane_t(const double* in, double* out, long long planes, int na, int nb, int ni, int nj,
                   const double* R, const double* L, double scale, double* partials, hipStream_t s) {
  const int ra = (na + 15) / 16;
  const int ld = ((nb + 15) & ~15) + 1;      // odd: the 16 rows of an operand fall into different banks
  const int ct = (nj + 15) / 16;
  const size_t shmem = (size_t)PL * ra * 16 * ld * sizeof(double);
  const dim3 block(64 * (ct < 8 ? ct : 8));
  constexpr long long kChunk = 1LL << 22;    // planes per launch, within the grid's thread count
  for (long long p0 = 0; p0 < planes; p0 += kChunk) {
    const long long np = planes - p0 < kChunk ? planes - p0 : kChunk;
    const dim3 grid((unsigned)((np + PL - 1) / PL));
    const double* src = in + (size_t)p0 * na * nb;
    double* dst = out ? out + (size_t)p0 * ni * nj : nullptr;
    double* par = partials ? partials + p0 / PL : nullptr;
#define RPA_PLANE(RA)                                                                               \
  case RA:                                                                                          \
    hipLaunchKernelGGL((k_plane<RA, PL, ENERGY>), grid, block, shmem, s, src, dst, np, na, nb, ni, nj, R, L, ld, \
                       scale, par);                                                                 \
    break;
    static_assert(kPairTiles == 5, "the first switch lists the row tiles of both forms");
    if (ra <= kPairTiles) {
      switch (ra) { RPA_PLANE(1) RPA_PLANE(2) RPA_PLANE(3) RPA_PLANE(4) RPA_PLANE(5) }
    } else if constexpr (PL == 1) {
      switch (ra) {
        RPA_PLANE(6) RPA_PLANE(7) RPA_PLANE(8)
        default: return hipErrorInvalidValue;
      }
    } else {
      return hipErrorInvalidValue;
    }
#undef RPA_PLANE
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int NC, int MODE>
hipError_t cols_t(const double* in, double* out, int B, int n_in, int n_out, int ncol, const double* A1,
                  const double* A2, const double* diag, const double* sr, const double* si, const ColsArgs& fw,
                  hipStream_t s) {
  const int waves = (ncol + (MODE == COLS_KINETIC ? 16 : 16 * NC) - 1) / (MODE == COLS_KINETIC ? 16 : 16 * NC);
  const int wpb = waves < 4 ? waves : 4;
  const dim3 block(64 * wpb);
  constexpr int kChunk = 1 << 15;            // arrays per launch (grid rows)
  const size_t fields = MODE == COLS_KINETIC ? 2 : 1;
  for (int b0 = 0; b0 < B; b0 += kChunk) {
    const dim3 grid((unsigned)((waves + wpb - 1) / wpb), (unsigned)(B - b0 < kChunk ? B - b0 : kChunk));
    const double* src = in + (size_t)b0 * fields * n_in * ncol;
    double* dst = out + (size_t)b0 * fields * n_out * ncol;
    const double* sr0 = sr ? sr + b0 : nullptr;
    const double* si0 = si ? si + b0 : nullptr;
#define RPA_COLS(RK)                                                                                \
  case RK:                                                                                          \
    hipLaunchKernelGGL((k_cols<RK, NC, MODE>), grid, block, 0, s, src, dst, n_in, n_out, ncol, A1, A2, diag, \
                       sr0, si0, fw);                                                               \
    break;
    const int rk = (n_in + 15) / 16;
    if (rk <= kPairTiles) {
      switch (rk) { RPA_COLS(1) RPA_COLS(2) RPA_COLS(3) RPA_COLS(4) RPA_COLS(5) }
    } else if constexpr (NC == 1 || MODE == COLS_KINETIC) {
      switch (rk) {
        RPA_COLS(6) RPA_COLS(7) RPA_COLS(8)
        default: return hipErrorInvalidValue;
      }
    } else {
      return hipErrorInvalidValue;
    }
#undef RPA_COLS
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

bool transform_fits(int d0, int d1, int d2) {
  return d0 <= kMaxTransformDim && d1 <= kMaxTransformDim && d2 <= kMaxTransformDim;
}

hipError_t launch_planes(const double* in, double* out, long long planes, int na, int nb, int ni, int nj,
                         const double* L, const double* R, hipStream_t s) {
  // two planes per workgroup need their registers and LDS, and enough planes
  // that every compute unit still gets several workgroups
  if (na <= 16 * kPairTiles && nb <= 16 * kPairTiles && planes >= 2048)
    return plane_t<2, false>(in, out, planes, na, nb, ni, nj, R, L, 1.0, nullptr, s);
  return plane_t<1, false>(in, out, planes, na, nb, ni, nj, R, L, 1.0, nullptr, s);
}

hipError_t launch_planes_energy(const double* in, double* e_fine, long long planes, int na, int nb, int ni, int nj,
                                const double* L, const double* R, double scale_fine, double* partials,
                                hipStream_t s) {
  return plane_t<1, true>(in, e_fine, planes, na, nb, ni, nj, R, L, scale_fine, partials, s);
}

hipError_t launch_cols(const double* in, double* out, int B, int n_in, int n_out, int ncol, const double* A,
                       hipStream_t s) {
  return cols_t<1, COLS_ONCE>(in, out, B, n_in, n_out, ncol, A, nullptr, nullptr, nullptr, nullptr, ColsArgs{}, s);
}

hipError_t launch_cols_fields(const double* in, double* out, int n_fields, const double* w, int n_in, int n_out,
                              int ncol, const double* A, hipStream_t s) {
  if (n_fields > kMaxFieldWeights) return hipErrorInvalidValue;
  ColsArgs fw{};
  fw.n = n_fields;
  for (int f = 0; f < n_fields; ++f) fw.a[f] = w[f];
  return cols_t<1, COLS_FIELDS>(in, out, 1, n_in, n_out, ncol, A, nullptr, nullptr, nullptr, nullptr, fw, s);
}

hipError_t launch_cols_scale(const double* in, double* out, int B, int n, int ncol, const double* fwd,
                             const double* inv, const double* diag, hipStream_t s) {
  if (n <= 16 * kPairTiles && (long long)B * ncol >= 32 * 2048)
    return cols_t<2, COLS_SCALE>(in, out, B, n, n, ncol, fwd, inv, diag, nullptr, nullptr, ColsArgs{}, s);
  return cols_t<1, COLS_SCALE>(in, out, B, n, n, ncol, fwd, inv, diag, nullptr, nullptr, ColsArgs{}, s);
}

hipError_t launch_cols_kinetic(const double* in, double* out, int nvec, int n, int ncol, const double* fwd,
                               const double* inv, const double* kin, const double* sig_re, const double* sig_im,
                               bool host_sigma, hipStream_t s) {
  ColsArgs fw{};
  if (host_sigma) {
    if (nvec > kMaxFieldWeights) return hipErrorInvalidValue;
    fw.n = nvec;
    for (int v = 0; v < nvec; ++v) {
      fw.a[v] = sig_re[v];
      fw.b[v] = sig_im[v];
    }
    sig_re = sig_im = nullptr;
  }
  return cols_t<2, COLS_KINETIC>(in, out, nvec, n, n, ncol, fwd, inv, kin, sig_re, sig_im, fw, s);
}

void pad_k_major(const double* M, int n_out, int n_in, bool trans, double* dst) {
  const int op = transform_pad(n_out);
  for (int k = 0; k < transform_pad(n_in); ++k)
    for (int o = 0; o < op; ++o)
      dst[(size_t)k * op + o] =
          k < n_in && o < n_out ? (trans ? M[(size_t)k * n_out + o] : M[(size_t)o * n_in + k]) : 0.0;
}

hipError_t launch_axis(const double* in, double* out, int B, int d0, int d1, int d2, int axis,
                       int n_out, const double* M, bool trans, const double* scale, hipStream_t s) {
  long long osz = (long long)d0 * d1 * d2;
  const int nin = axis == 0 ? d0 : (axis == 1 ? d1 : d2);
  osz = osz / nin * n_out;
  hipLaunchKernelGGL(k_axis, dim3(grid_of(osz * B)), dim3(256), 0, s, in, out, B, d0, d1,
                     d2, axis, n_out, M, trans ? 1 : 0, scale);
  return hipGetLastError();
}

hipError_t launch_kin_scale(double* a, const double* kin, const double* sig_re,
                            const double* sig_im, int B, long long N, hipStream_t s) {
  hipLaunchKernelGGL(k_kin_scale, dim3(grid_of((long long)B * N)), dim3(256), 0, s, a, kin,
                     sig_re, sig_im, B, N);
  return hipGetLastError();
}

}  // namespace rpa
