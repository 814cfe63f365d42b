// Batched Sternheimer COCG launches (kernels in cocg_impl.h, compiled by
// cocg_kernels.hip), the plain operator application and the nonlocal term of the latter.
#include "cocg_impl.h"

#include <algorithm>

namespace rpa {

namespace {

// Shifts that travel with the launch (n = 0: they are in device memory).
struct HapplyShifts {
  int n;
  double re[kMaxFieldWeights], im[kMaxFieldWeights];
};

// Tile blockIdx.x, vector blockIdx.y, planes of segment blockIdx.z.  FP32: at
// most 80 registers, so that two workgroups of a 768-thread tile share a
// compute unit and one loads while the other computes (512 vectors of 48^3:
// 305 us with one workgroup, 270 with two; 193 at the rate of a copy).
template <typename T>
constexpr int kHapplyWaves = sizeof(T) == 4 ? 6 : 4;   // per SIMD: at most 80 and 128 registers
template <typename T, int M, int PITCH>
__global__ void __launch_bounds__(kMaxBlock, kHapplyWaves<T>) k_happly(Geom g, StencilCoef<T> cf, const T* v,
                                                       const double* sr, const double* si,
                                                       const void* x, void* y, int seg, HapplyShifts sh) {
  extern __shared__ double smem_d[];
  typedef typename V2<T>::t T2;
  constexpr bool FULL = M == 0;
  constexpr int HS = M == 2 ? 2 : 1;
  const int vec = blockIdx.y;
  const size_t base = (size_t)vec * g.N;
  HPol<T> p;
  p.x = reinterpret_cast<const T2*>(x) + base;
  p.y = reinterpret_cast<T2*>(y) + base;
  p.v = v; p.c0 = cf.c0;
  p.sr = (T)(sh.n ? sh.re[vec] : sr[vec]);
  p.si = (T)(sh.n ? sh.im[vec] : si[vec]);
  const int xb = blockIdx.z * seg, xe = min(g.nx, xb + seg);
  march<T, FULL, HS, PITCH>(g, cf, p, reinterpret_cast<T2*>(smem_d), blockIdx.x, blockIdx.x + 1, xb, xe);
}

// Nonlocal term of the plain operator application: per vector, the
// projections (one workgroup each, coefficients through LDS to coef), then
// y += V_nl x point by point.
template <typename T>
__global__ void __launch_bounds__(256) k_nl_coef(NlArgs nl, const void* x, long long N,
                                                  void* coef) {
  typedef typename V2<T>::t T2;
  extern __shared__ double smem_d[];
  T2* c = reinterpret_cast<T2*>(smem_d);
  const T2* xv = reinterpret_cast<const T2*>(x) + (size_t)blockIdx.x * N;
  double d0 = 0.0, d1 = 0.0;
  nl_project<T, T>(nl, xv, c, d0, d1);
  __syncthreads();
  T2* out = reinterpret_cast<T2*>(coef) + (size_t)blockIdx.x * nl.n_proj;
  for (int p = threadIdx.x; p < nl.n_proj; p += blockDim.x) out[p] = c[p];
}

template <typename T>
__global__ void __launch_bounds__(256) k_nl_add(NlArgs nl, long long N, const void* coef,
                                                 void* y) {
  typedef typename V2<T>::t T2;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const T2* c = reinterpret_cast<const T2*>(coef) + (size_t)blockIdx.y * nl.n_proj;
  T2* yv = reinterpret_cast<T2*>(y) + (size_t)blockIdx.y * N;
  T2 o = yv[i];
  nl_point<T>(nl.pm_ptr, nl.pm_proj, nl_pick<T>(nl.pm_v32, nl.pm_v64), c, i, o.x, o.y);
  yv[i] = o;
}

}  // namespace

namespace {

int tile_mode(const Geom& g, int block) {
  if (g.ty == g.ny) return 0;
  return block >= 2 * R * g.nz ? 1 : 2;
}

// LDS row pitch.  When a wave spans several rows, a pitch that is a multiple
// of the 64 banks puts the same columns of all its rows into the same banks:
// 56 shifts each row by eight elements.  Rows of 45 to 52 points nearly fill a
// wave and take 64.
int pitch_for(const Geom& g) { return g.nz + 2 * R <= 56 ? 56 : (g.nz + 2 * R <= 64 ? 64 : 128); }

template <int V>
CocgKernel cocg_pick_v(const Geom& g, int block, bool refine) {
  const int m = tile_mode(g, block);
  switch (pitch_for(g)) {
    case 56: return cocg_kernel<V, 56>(m, refine);
    case 64: return cocg_kernel<V, 64>(m, refine);
    default: return cocg_kernel<V, 128>(m, refine);
  }
}

// The persistent kernel for a launch of `block` threads.
CocgKernel cocg_pick(const Geom& g, int block, bool refine, bool nonlocal) {
  if (g.prec) return nonlocal ? cocg_pick_v<3>(g, block, refine) : cocg_pick_v<2>(g, block, refine);
  return nonlocal ? cocg_pick_v<1>(g, block, refine) : cocg_pick_v<0>(g, block, refine);
}

}  // namespace

bool geom_supported(const Geom& g) { return g.nz + 2 * R <= 128; }

size_t cocg_shmem_bytes(const Geom& g, int block, bool fp32_refine, int n_proj) {
  return lds_plane_bytes(g, pitch_for(g), fp32_refine) + red_bytes(g.prec && g.pc_block ? g.pc_block : block) +
         (size_t)n_proj * sizeof(double2);
}

void cocg_pc_shape(Geom& g, int block, int n_proj) {
  // kPcBlock threads keep the memory pipes busy whatever the stencil tile is;
  // the tile's own workgroup only where the larger reduction buffer would not fit
  for (const int b : {kPcBlock, block}) {
    const size_t rest = red_bytes(b) + (size_t)n_proj * sizeof(double2);
    const size_t lds = 160 * 1024 > rest ? 160 * 1024 - rest : 0;
    g.pc_block = b;
    g.pc_planes32 = pc_planes<float>(g, b, lds);
    g.pc_planes64 = pc_planes<double>(g, b, lds);
    if (cocg_shmem_bytes(g, b, true, n_proj) <= 160 * 1024 && cocg_shmem_bytes(g, b, false, n_proj) <= 160 * 1024)
      return;
  }
}

int cocg_blocks_per_cu(const Geom& g, int block, bool fp32_refine, int n_proj) {
  const size_t shmem = cocg_shmem_bytes(g, block, fp32_refine, n_proj);
  if (g.prec && g.pc_block) block = g.pc_block;
  int nb = 0;
  const void* fn = reinterpret_cast<const void*>(cocg_pick(g, block, fp32_refine, n_proj > 0));
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, block, shmem);
  if (e != hipSuccess || nb < 1) return 1;
  return nb;
}

int cocg_prec_regs(const Geom& g, int block) { return prec_regs(g, block); }
int cocg_prec_regs_max() { return kPrecRegs; }

long long cocg_slot_bytes(const Geom& g, bool fp32_refine) {
  // r, q, p (+ the FP32 correction d, + the preconditioner's transform buffer)
  const long long vecs = 3 + (fp32_refine ? 1 : 0) + (g.prec ? 1 : 0);
  return vecs * g.N * (long long)(fp32_refine ? sizeof(float2) : sizeof(double2));
}

size_t cocg_slots_bytes(const Geom& g, bool fp32_refine, int grid) {
  return (size_t)std::max((long long)grid * cocg_slot_bytes(g, fp32_refine), cocg_slot_bytes(g, false));
}

namespace {
template <typename T>
using HapplyKernel = void (*)(Geom, StencilCoef<T>, const T*, const double*, const double*, const void*, void*, int,
                              HapplyShifts);

template <typename T, int P>
HapplyKernel<T> happly_kernel(int m) {
  if (m == 0) return &k_happly<T, 0, P>;
  if (m == 1) return &k_happly<T, 1, P>;
  return &k_happly<T, 2, P>;
}

template <typename T>
hipError_t launch_ht(const Geom& g, const StencilCoef<T>& cf, const T* v, const double* sr, const double* si,
                     const HapplyShifts& sh, const void* x, void* y, int nvec, int block, size_t shmem, int num_cu,
                     hipStream_t s) {
  // few workgroups: split the march along x.  A segment reads its own 12 halo
  // planes, so of the splits of at most two rounds of the workgroups that run at
  // once the one with the fewest plane steps is taken (more rounds are bound by
  // memory, where the halo costs): 64 FP64 vectors of 48^3, one 768-thread
  // workgroup per compute unit, 67 us whole and 74 in halves; 65 of 60x30x40 93 us
  // whole and 85 in thirds; 300 FP32 vectors of 128x8x8, four workgroups per
  // compute unit, 103 us whole and 60 in thirds
  const int fit = std::max(1, std::min(4 * kHapplyWaves<T> / (block / 64), (int)(160 * 1024 / shmem)));
  const long long wgs = (long long)g.ntiles * nvec, cap = (long long)fit * num_cu;
  int nseg = 1;
  long long best = -1;
  for (int k = 1; k <= g.nx && (k == 1 || k * wgs <= 2 * cap); ++k) {
    const long long seg = (g.nx + k - 1) / k, steps = (k * wgs + cap - 1) / cap * (seg + 2 * R);
    if (best < 0 || steps < best) {
      best = steps;
      nseg = k;
    }
  }
  const int seg = (g.nx + nseg - 1) / nseg;
  const int m = tile_mode(g, block);
  const int pitch = pitch_for(g);
  const HapplyKernel<T> k = pitch == 56   ? happly_kernel<T, 56>(m)
                            : pitch == 64 ? happly_kernel<T, 64>(m)
                                          : happly_kernel<T, 128>(m);
  hipLaunchKernelGGL(k, dim3(g.ntiles, nvec, (g.nx + seg - 1) / seg), dim3(block), shmem, s, g, cf, v, sr, si, x, y, seg,
                     sh);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_cocg(const CocgArgs& a, bool fp32_refine, int grid, int block, size_t shmem, int num_cu,
                       hipStream_t s) {
  if (launch_cocg_resident(a, fp32_refine, grid, s)) return hipGetLastError();
  if (a.prec) block = a.g.pc_block;
  CocgArgs b = a;
  if (!a.prec) {
    // residual elements in the LDS that this many workgroups per compute unit
    // leave free, in whole trips of the streaming sweeps
    const int per_cu = std::max(1, (grid + num_cu - 1) / num_cu);
    const long long free_lds = 160 * 1024 / per_cu - (long long)shmem;
    const long long trip = (long long)kSweep * block, elem = fp32_refine ? sizeof(float2) : sizeof(double2);
    const long long n = std::min(a.g.N, std::max(0LL, free_lds) / elem);
    b.r_lds = (int)(n / trip * trip);
    shmem += (size_t)b.r_lds * elem;
  }
  hipLaunchKernelGGL(cocg_pick(a.g, block, fp32_refine, a.nl.n_proj > 0), dim3(grid), dim3(block), shmem, s, b);
  return hipGetLastError();
}

hipError_t launch_happly(const Geom& g, const StencilCoef<double>& c64, const StencilCoef<float>& c32,
                         const double* v64, const float* v32, int nvec, const double* shift_re,
                         const double* shift_im, bool host_shifts, const void* x, void* y, bool fp32,
                         int block, int num_cu, hipStream_t s) {
  // without the preconditioner's bases and planes, which this kernel does not
  // use: with them one workgroup of 48^3 filled a compute unit's LDS (137 KB against 57)
  Geom gp = g;
  gp.prec = 0;
  const size_t shmem = cocg_shmem_bytes(gp, block, fp32, 0);
  HapplyShifts sh{};
  if (host_shifts) {
    if (nvec > kMaxFieldWeights) return hipErrorInvalidValue;
    sh.n = nvec;
    for (int v = 0; v < nvec; ++v) {
      sh.re[v] = shift_re[v];
      sh.im[v] = shift_im[v];
    }
    shift_re = shift_im = nullptr;
  }
  if (fp32) return launch_ht<float>(g, c32, v32, shift_re, shift_im, sh, x, y, nvec, block, shmem, num_cu, s);
  return launch_ht<double>(g, c64, v64, shift_re, shift_im, sh, x, y, nvec, block, shmem, num_cu, s);
}

hipError_t launch_nl_apply(const NlArgs& nl, long long N, int nvec, const void* x, void* y,
                           void* coef, bool fp32, hipStream_t s) {
  if (nl.n_proj == 0) return hipSuccess;
  const size_t shmem = (size_t)nl.n_proj * (fp32 ? sizeof(float2) : sizeof(double2));
  const dim3 ga((unsigned)((N + 255) / 256), (unsigned)nvec);
  if (fp32) {
    hipLaunchKernelGGL((k_nl_coef<float>), dim3(nvec), dim3(256), shmem, s, nl, x, N, coef);
    hipLaunchKernelGGL((k_nl_add<float>), ga, dim3(256), 0, s, nl, N, (const void*)coef, y);
  } else {
    hipLaunchKernelGGL((k_nl_coef<double>), dim3(nvec), dim3(256), shmem, s, nl, x, N, coef);
    hipLaunchKernelGGL((k_nl_add<double>), ga, dim3(256), 0, s, nl, N, (const void*)coef, y);
  }
  return hipGetLastError();
}

}  // namespace rpa
