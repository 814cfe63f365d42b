// Batched Sternheimer solves (paper: Eq. 4, COCG with Galerkin initial guess,
// Implementation section) as one persistent launch.
//
// Design (gfx950, wave64):
//  * One workgroup owns one complex-symmetric system (H - eps_n - i omega) x = b
//    at a time and runs COCG to convergence with no grid-wide synchronisation;
//    workgroups take systems from an atomic work counter (longest-first order
//    is chosen by the host), so per-system iteration counts that differ by
//    10x across omega do not idle the chip.
//  * The 37-point stencil of the 12th-order FD Hamiltonian marches along x:
//    each thread owns one (y, z) column of a tile of ty rows x nz columns and
//    keeps the 13 planes x-6..x+6 of its column in registers; the current
//    plane (plus 6 halo rows on each side in y) sits in LDS, double
//    buffered, so each step needs a single barrier.  Every vector element is
//    read from HBM once per sweep (plus the y halo and the periodic x wrap).
//  * COCG per iteration is three sweeps: p = r + beta p with the solution's
//    pending alpha p (5 vector passes), the stencil q = A p with mu = p^T q
//    (about 2.5), r -= alpha q with r^T r and ||r||^2 (3).  The stencil's
//    operand is one vector that it only reads, so the march carries nothing
//    but its column and the potential.  The residual's first elements stay in
//    the LDS that the march leaves free (cells up to 24^3 are bound by the
//    traffic of all workgroups' vectors through the last-level cache, about
//    7 TB/s).  All reductions are per workgroup in a fixed order, so results
//    do not depend on scheduling.  Measured against a stencil sweep that forms
//    p on the fly (two halo'd operands in FP64, A p by recurrence in FP32) and
//    one update sweep: density of 64 start vectors on 24^3 in FP64 279 -> 99 ms,
//    chi0 of 64 vectors on 24^3 in FP32 30.1 -> 23.4 ms, the plain launches of
//    16 start vectors on 48^3 with 128 orbitals 926 -> 760 ms.
//  * FP32_REFINE: COCG in FP32 with reliable updates: the FP32 correction is
//    folded into the FP64 solution and the residual replaced by the FP64
//    residual r = b - A x (an FP64 stencil sweep) whenever the recursive
//    residual has dropped by a fixed factor; the search direction is kept.
//    b = -psi_n (.) u is formed on the fly in FP64 and never stored.
#pragma once

#include <type_traits>
#include <utility>

#include "internal.h"

namespace rpa {

namespace {

template <typename T> struct V2;
template <> struct V2<float> { typedef float2 t; };
template <> struct V2<double> { typedef double2 t; };

// The thread id, opaque to the optimiser: what a pass over the
// grid derives from it is computed inside that pass.  Hoisted out of the
// solver's loop instead, the addresses of the preconditioned solver's passes
// took 571 spilled registers per thread.
__device__ __forceinline__ int opaque_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Element `off` after the uniform address p (one 32-bit offset register).
template <typename E>
__device__ __forceinline__ E& at32(E* p, unsigned off) {
  typedef typename std::conditional<std::is_const<E>::value, const char, char>::type C;
  return *reinterpret_cast<E*>(reinterpret_cast<C*>(p) + (unsigned)(off * (unsigned)sizeof(E)));
}

// Buffer access to element `off` bytes after the uniform address p: one
// descriptor in scalar registers and one 32-bit offset per lane.  Through
// plain pointers every array of a march took a 64-bit address in vector
// registers and a 64-bit add per access.
template <typename E>
__device__ __forceinline__ E buf_load(const E* p, unsigned off) {
  const __amdgpu_buffer_rsrc_t d =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<E*>(p), 0, 0xffffffffu, 0x00027000);
  if constexpr (sizeof(E) == 4) return __builtin_bit_cast(E, __builtin_amdgcn_raw_buffer_load_b32(d, off, 0, 0));
  else if constexpr (sizeof(E) == 8) return __builtin_bit_cast(E, __builtin_amdgcn_raw_buffer_load_b64(d, off, 0, 0));
  else return __builtin_bit_cast(E, __builtin_amdgcn_raw_buffer_load_b128(d, off, 0, 0));
}
typedef unsigned buf_u2 __attribute__((ext_vector_type(2)));
typedef unsigned buf_u4 __attribute__((ext_vector_type(4)));
template <typename E>
__device__ __forceinline__ void buf_store(E* p, unsigned off, const E& v) {
  const __amdgpu_buffer_rsrc_t d = __builtin_amdgcn_make_buffer_rsrc(p, 0, 0xffffffffu, 0x00027000);
  if constexpr (sizeof(E) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(buf_u2, v), d, off, 0, 0);
  else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(buf_u4, v), d, off, 0, 0);
}

}  // namespace
}  // namespace rpa

#include "precond_impl.h"

namespace rpa {

namespace {

constexpr int R = kRadius;
constexpr int QN = 2 * R + 1;
constexpr int kMinGap = 4;     // fewest FP32 iterations between reliable updates
constexpr int kMaxGap = 100;   // most FP32 iterations between true-residual checks

__device__ __forceinline__ float2 mk2(float a, float b) { return make_float2(a, b); }
__device__ __forceinline__ double2 mk2(double a, double b) { return make_double2(a, b); }

template <typename T2>
__device__ __forceinline__ T2 zero2() { T2 z; z.x = 0; z.y = 0; return z; }

// Every value that steers control flow around a barrier is broadcast from
// lane 0 into a scalar register, so the compiler sees wave-uniform branches
// (values read back from LDS are otherwise treated as divergent, which puts
// __syncthreads() into divergent control flow).
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double uni(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffLL));
  const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

__device__ __forceinline__ float uni(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// ---------------------------------------------------------------------------
// Workgroup reduction of K doubles, fixed order, result broadcast to all.
// red must hold (nwaves + 1) * K doubles.
template <int K>
__device__ __forceinline__ void block_reduce(double (&v)[K], double* red) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    double x = v[k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    v[k] = x;
  }
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) red[wave * K + k] = v[k];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      double s = 0.0;
      for (int w = 0; w < nw; ++w) s += red[w * K + k];
      red[nw * K + k] = s;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = uni(red[nw * K + k]);
  __syncthreads();
}

template <typename T>
__device__ __forceinline__ T wave_sum(T x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

template <typename T>
__device__ __forceinline__ const T* nl_pick(const float* a, const double* b) {
  if constexpr (sizeof(T) == 4) return a;
  else return b;
}

// Nonlocal projections of one vector x (Background section, separable V_nl):
// c_p = chi_p^T x for every projector.  Each wave takes whole support groups
// (the projectors of a group share their support, so x is gathered once per
// group); lane 0 stores w_p = gamma_p h^3 c_p into coef (LDS) and adds
// sum_p w_p c_p = x^T V_nl x (unconjugated) to mu.  The caller synchronises
// before coef is read.
template <typename T, typename XT>
__device__ void nl_project(const NlArgs& nl, const typename V2<XT>::t* x,
                           typename V2<T>::t* coef, double& mu_re, double& mu_im) {
  const int lane = threadIdx.x & 63;
  const int wave = uni((int)(threadIdx.x >> 6));
  const int nw = (int)(blockDim.x >> 6);
  const T* bv = nl_pick<T>(nl.bv32, nl.bv64);
  for (int gi = wave; gi < nl.n_groups; gi += nw) {
    const int4 G = nl.ginfo[gi];
    const int s0 = uni(G.x), S = uni(G.y) - s0, p0 = uni(G.z), np = uni(G.w);
    const T* val = bv + uni(nl.gvoff[gi]);
    const int* idx = nl.bidx + s0;
    T ar[kMaxGroup], ai[kMaxGroup];
#pragma unroll
    for (int k = 0; k < kMaxGroup; ++k) { ar[k] = 0; ai[k] = 0; }
    for (int j = lane; j < S; j += 64) {
      const typename V2<XT>::t v = x[idx[j]];
      const T vr = (T)v.x, vi = (T)v.y;
#pragma unroll
      for (int k = 0; k < kMaxGroup; ++k) {
        if (k < np) {
          const T c = val[k * S + j];
          ar[k] += c * vr;
          ai[k] += c * vi;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kMaxGroup; ++k) {
      if (k < np) {
        ar[k] = wave_sum(ar[k]);
        ai[k] = wave_sum(ai[k]);
        if (lane == 0) {
          const double gd = nl.gdv[p0 + k];
          const double cr = (double)ar[k], ci = (double)ai[k];
          const double wr = gd * cr, wi = gd * ci;
          typename V2<T>::t w;
          w.x = (T)wr;
          w.y = (T)wi;
          coef[p0 + k] = w;
          mu_re += wr * cr - wi * ci;
          mu_im += wr * ci + wi * cr;
        }
      }
    }
  }
}

// (V_nl x)_i = sum over the entries of point i of w_p chi_p(i), added to (ar, ai).
template <typename T>
__device__ __forceinline__ void nl_point(const int* pm_ptr, const int* pm_proj, const T* pm_v,
                                         const typename V2<T>::t* coef, long long i, T& ar,
                                         T& ai) {
  const int e1 = pm_ptr[i + 1];
  for (int e = pm_ptr[i]; e < e1; ++e) {
    const T c = pm_v[e];
    const typename V2<T>::t w = coef[pm_proj[e]];
    ar += c * w.x;
    ai += c * w.y;
  }
}

// ---------------------------------------------------------------------------
// x-marching stencil sweep over all tiles of one system.
//
// Pol provides (po = uniform plane offset, c = per-lane offset in the plane):
//   T2 load(size_t po, int c)  -- operand value at a point
//   Aux aux(size_t po, int c)  -- centre-only data (potential, right-hand side)
//   void center(size_t po, int c, T2 val, T2 nbr, const Aux&) -- nbr is the
//   sum of the off-centre stencil terms.
//
// Each thread keeps planes x-R .. x+R+PF of its column in a register FIFO
// whose slots rotate by compile-time phase (the x loop is unrolled by the
// FIFO length U), so no register moves are needed; planes are loaded PF steps
// before their first use.  The current plane sits in LDS with a compile-time
// row pitch PITCH, padded with R periodic copies on each side in z (and in y
// when one tile covers the whole plane), so all 24 in-plane neighbour reads
// are immediate offsets from one per-thread base address.
// f(0) ... f(N - 1) with compile-time arguments: register arrays indexed
// inside never depend on the loop unroller.
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(f, std::make_integer_sequence<int, N>{});
}
#define RPA_INLINE __attribute__((always_inline))

template <typename T, bool FULL, int HS, int PITCH, class Pol, int PPS>
struct Marcher {
  typedef typename V2<T>::t T2;
  typedef typename Pol::Aux AuxT;
  // grid offsets: a whole-plane tile has at most 768 points per plane, and an
  // axis' dense basis keeps n_x far below the 2.8 million that 32 bits hold
  typedef typename std::conditional<FULL, int, long long>::type Off;
  static constexpr int PF = Pol::kPF;
  static constexpr int U = QN + PF;   // FIFO: planes x-R .. x+R+PF
  static constexpr int PA = PF + 1;   // aux/halo pipelines: planes x .. x+PF
  static constexpr int NH = FULL ? 0 : HS;
  // The x loop is unrolled by U, so a slot index (phase within the block) of
  // a pipeline of period PA equals x mod PA only if PA divides U
  // (PF in {1, 2, 3, 5} for the 13-plane stencil).
  static_assert(U % PA == 0, "prefetch depth must make PF+1 divide 2R+1+PF");

  static_assert(PPS == 1 || PPS == 2, "one or two planes per barrier");
  static_assert(U % PPS == 0, "plane pairs must not straddle the unrolled block");

  const Geom& g;
  const StencilCoef<T>& cf;
  Pol& pol;
  T2* buf0;            // plane buffers: 2 * PPS of them, bufs apart
  size_t bufs;         // elements per buffer
  int plane;
  int nx;
  int y0n;             // column offset of the tile's first row
  unsigned col;        // own column offset in the tile
  int ci;              // LDS index of the own point
  int edge;            // periodic copies: 1 left z pad, 2 right z pad, 4 / 8 y pads (whole planes)
  bool hv[HS];
  int hl[HS];          // LDS index of halo points
  unsigned hcol[HS];   // halo column offsets in the plane
  T2 fifo[U];
  AuxT ax[PA];
  T2 hq[HS][PA];

  __device__ __forceinline__ static int wrapx(int p, int n) { return p >= n ? p - n : p; }

  // store plane x (FIFO phase PH) into buf
  template <int PH>
  __device__ __forceinline__ void put(T2* buf) {
    const T2 c = fifo[(PH + R) % U];
    buf[ci] = c;
    if (edge & 1) buf[ci - g.nz] = c;
    if (edge & 2) buf[ci + g.nz] = c;
    if (FULL) {
      if (edge & 4) buf[ci - g.ny * PITCH] = c;
      if (edge & 8) buf[ci + g.ny * PITCH] = c;
    }
    static_for<NH>([&](auto H) RPA_INLINE {
      if (hv[H]) buf[hl[H]] = hq[H][PH % PA];
    });
  }

  // PPS consecutive planes x, x+1 share one barrier: both are stored into
  // their own buffers of the current set, then both are computed.  TAIL: the
  // block may end inside the pair (only the last block of a march).
  template <int PH, bool TAIL>
  __device__ __forceinline__ void step(int x, int xe) {
    T2* set = buf0 + (size_t)(((x / PPS) & 1) * PPS) * bufs;
    const bool second = PPS == 2 && (!TAIL || x + 1 < xe);
    put<PH>(set);
    if (second) put<PH + 1>(set + bufs);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    point<PH>(x, xe, set);
    __builtin_amdgcn_sched_barrier(0);
    if (second) point<PH + 1>(x + 1, xe, set + bufs);
    __builtin_amdgcn_sched_barrier(0);
  }

  // No branch in here: threads without a column of their own repeat the
  // tile's first one (same values to the same addresses, Pol::own masks the
  // sums), and the refills past the last plane re-read it.  The loads and
  // stores share one counter that completes in order, and behind a branch the
  // compiler has to assume the smaller count: with the store of q in an
  // if (own) every step waited for the previous step's store.
  template <int PH>
  __device__ __forceinline__ void point(int x, int xe, const T2* buf) {
    const T2 c = fifo[(PH + R) % U];
    const T2* w = buf + (ci - (R * PITCH + R));
    T xr = 0, xi = 0, yr = 0, yi = 0, zr = 0, zi = 0;
    static_for<R>([&](auto K) RPA_INLINE {
      constexpr int k = K + 1;
      const T2 a = fifo[(PH + R - k) % U];
      const T2 b = fifo[(PH + R + k) % U];
      xr += cf.w[k] * (a.x + b.x);
      xi += cf.w[k] * (a.y + b.y);
    });
    static_for<R>([&](auto K) RPA_INLINE {
      constexpr int k = K + 1;
      const T2 a = w[(R - k) * PITCH + R];
      const T2 b = w[(R + k) * PITCH + R];
      yr += cf.w[k] * (a.x + b.x);
      yi += cf.w[k] * (a.y + b.y);
    });
    static_for<R>([&](auto K) RPA_INLINE {
      constexpr int k = K + 1;
      const T2 a = w[R * PITCH + R - k];
      const T2 b = w[R * PITCH + R + k];
      zr += cf.w[k] * (a.x + b.x);
      zi += cf.w[k] * (a.y + b.y);
    });
    const T sx = cf.sx * xr + cf.sy * yr + cf.sz * zr;
    const T sy = cf.sx * xi + cf.sy * yi + cf.sz * zi;
    pol.center((Off)x * plane + y0n, col, c, mk2(sx, sy), ax[PH % PA]);
    // refill the pipelines: the FIFO slot of plane x-R takes plane x+R+PF+1,
    // the aux/halo slot of plane x takes plane x+PF+1
    const int xn = x + PF + 1;
    const int xc = xn < xe ? xn : xe - 1;
    const Off po = (Off)xc * plane + y0n, pw = (Off)wrapx(xc + R, nx) * plane + y0n;
    fifo[PH % U] = pol.load(pw, col);
    ax[PH % PA] = pol.aux(po, col);
    static_for<NH>([&](auto H) RPA_INLINE { hq[H][PH % PA] = pol.load(po - y0n, hcol[H]); });
  }

  // U planes from x; full blocks need no bounds checks between steps
  template <int PH>
  __device__ __forceinline__ void block_full(int x, int xe) {
    if constexpr (PH < U) {
      step<PH, false>(x, xe);
      block_full<PH + PPS>(x + PPS, xe);
    }
  }

  template <int PH>
  __device__ __forceinline__ void block(int x, int xe) {
    if constexpr (PH < U) {
      if (x < xe) {
        step<PH, true>(x, xe);
        block<PH + PPS>(x + PPS, xe);
      }
    }
  }

  // Planes [xb, xe) of tiles [t_begin, t_end).
  __device__ __forceinline__ void run(int t_begin, int t_end, int xb, int xe) {
    const int tid = opaque_tid();
    const int bs = (int)blockDim.x;
    const int ny = g.ny, nz = g.nz, ty = FULL ? g.ny : g.ty;
    pol.own = tid < ty * nz;
    col = pol.own ? tid : 0;
    const int ly = (int)col / nz, z = (int)col - ly * nz;
    ci = (ly + R) * PITCH + z + R;
    // a point is copied into the left pad if it is among the last R of the
    // row and into the right pad if among the first R (both when nz < 2R)
    edge = (z >= nz - R ? 1 : 0) | (z < R ? 2 : 0) | (FULL && ly >= ny - R ? 4 : 0) | (FULL && ly < R ? 8 : 0);
    const int nhalo = 2 * R * nz;
    int hrow[HS], hz[HS];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const int hid = tid + h * bs;
      hv[h] = hid < nhalo;
      const int hr = hv[h] ? hid / nz : 0;
      hz[h] = hv[h] ? hid - hr * nz : 0;
      hrow[h] = hr;
      hl[h] = (hr < R ? hr : ty + hr) * PITCH + hz[h] + R;
    }
    for (int t = t_begin; t < t_end; ++t) {
      const int y0 = t * ty;
      y0n = y0 * nz;
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        int gr = hrow[h] < R ? y0 - R + hrow[h] : y0 + ty + (hrow[h] - R);
        gr = gr < 0 ? gr + ny : (gr >= ny ? gr - ny : gr);
        hcol[h] = gr * nz + hz[h];
      }
      // prologue: FIFO slot i holds plane xb + i - R (phase 0); aux/halo slot i plane xb + i
      static_for<U>([&](auto I) RPA_INLINE {
        int px = (xb + (I - R)) % nx;          // nx > R: at most one period below
        px = px < 0 ? px + nx : px;
        fifo[I] = pol.load((Off)px * plane + y0n, col);
      });
      static_for<PA>([&](auto I) RPA_INLINE {
        const int px = xb + I < xe ? xb + I : xe - 1;
        ax[I] = pol.aux((Off)px * plane + y0n, col);
        static_for<NH>([&](auto H) RPA_INLINE { hq[H][I] = pol.load((Off)px * plane, hcol[H]); });
      });
      int x = xb;
      for (; x + U <= xe; x += U) block_full<0>(x, xe);
      if (x < xe) block<0>(x, xe);
      __syncthreads();
    }
  }
};

// FP32 sweeps march two planes per barrier (four plane buffers), FP64 ones one.
template <typename T>
constexpr int planes_per_step() { return sizeof(T) == 4 ? 2 : 1; }

template <typename T, bool FULL, int HS, int PITCH, class Pol>
__device__ __forceinline__ void march(const Geom& g, const StencilCoef<T>& cf, Pol& pol,
                                      typename V2<T>::t* lds, int t_begin, int t_end, int xb, int xe) {
  const int rows = (FULL ? g.ny : g.ty) + 2 * R;
  Marcher<T, FULL, HS, PITCH, Pol, planes_per_step<T>()> m{g, cf, pol};
  m.buf0 = lds;
  m.bufs = (size_t)rows * PITCH;
  m.plane = g.ny * g.nz;
  m.nx = g.nx;
  m.run(t_begin, t_end, xb, xe);
}

// Bytes of LDS used by the plane buffers of the march (padded pitch): the
// FP32 form of one tile takes four buffers, the FP64 form two of twice the size.
__host__ __device__ inline size_t lds_plane_bytes(const Geom& g, int pitch, bool fp32_iter) {
  const size_t rows_pad = (size_t)g.ty + 2 * R;
  size_t b = 2 * rows_pad * pitch * sizeof(double2);
  if (g.prec) {
    // the preconditioner's bases and planes (FP64 for the FP64 solver, which
    // the FP32 path also launches for the systems it hands over); without a
    // launch shape yet, the bound that decides whether a problem is accepted
    const size_t elem = fp32_iter ? sizeof(float) : sizeof(double);
    const int planes = fp32_iter ? g.pc_planes32 : g.pc_planes64;
    const size_t pb = planes ? pc_lds_bytes(g, elem, planes) : prec_lds_bytes(g, elem);
    b = b > pb ? b : pb;
  }
  return (b + 255) & ~(size_t)255;
}

// Bytes of LDS for the reductions (4 doubles per wave plus the result).
__host__ __device__ inline size_t red_bytes(int block) {
  const size_t nw = (size_t)(block + 63) / 64;
  return ((nw + 1) * 4 * sizeof(double) + 255) & ~(size_t)255;
}

// ---------------------------------------------------------------------------
// Policies

// FP64 residual r = b - (H - sigma) x with b = -psi_n (.) u; stores r in TI.
template <typename TI, bool NL>
struct ResidPol {
  typedef typename V2<TI>::t TI2;
  const double2* x;
  const double* v;
  const double* psi;
  const double* u;
  TI2* r;
  double c0, eps, om;
  double rr, bb, rho_re, rho_im;
  bool own;                       // set by the march; sums of repeated columns are dropped
  const int* pm_ptr;              // point-major projector entries (NL)
  const int* pm_proj;
  const double* pm_v;
  const double2* coef;            // w_p of x (LDS)
  static constexpr int kPF = 1;
  struct Aux { double v, psi, u; };
  __device__ double2 load(long long po, unsigned c) const { return buf_load(x + po, c * (unsigned)sizeof(*x)); }
  __device__ Aux aux(long long po, unsigned c) const {
    Aux a;
    a.v = buf_load(v + po, c * (unsigned)sizeof(*v));
    a.psi = buf_load(psi + po, c * (unsigned)sizeof(*psi));
    a.u = buf_load(u + po, c * (unsigned)sizeof(*u));
    return a;
  }
  __device__ void center(long long po, unsigned c, double2 xv, double2 nb, const Aux& ax) {
    const double a = c0 + ax.v - eps;
    double axr = a * xv.x + om * xv.y + nb.x;
    double axi = a * xv.y - om * xv.x + nb.y;
    if constexpr (NL) nl_point<double>(pm_ptr, pm_proj, pm_v, coef, (long long)po + c, axr, axi);
    const double bval = -ax.psi * ax.u;
    const double rx = bval - axr;
    const double ry = -axi;
    TI2 rs; rs.x = (TI)rx; rs.y = (TI)ry;
    buf_store(r + po, c * (unsigned)sizeof(rs), rs);
    const double sx = (double)rs.x, sy = (double)rs.y;
    rr += own ? rx * rx + ry * ry : 0.0;
    bb += own ? bval * bval : 0.0;
    rho_re += own ? sx * sx - sy * sy : 0.0;
    rho_im += own ? 2.0 * sx * sy : 0.0;
  }
};

// COCG stencil sweep: q = (H_loc - sigma) p, mu = p^T q.  Nothing is computed
// from a value as soon as it is loaded, so the loads of later planes stay in
// flight across steps.
template <typename T>
struct ApplyPol {
  typedef typename V2<T>::t T2;
  const T2* p;
  T2* q;
  const T* v;
  T c0, eps, om;
  double mu_re, mu_im;
  bool own;
  static constexpr int kPF = 1;
  typedef T Aux;
  __device__ T aux(long long po, unsigned c) const { return buf_load(v + po, c * (unsigned)sizeof(*v)); }
  __device__ T2 load(long long po, unsigned c) const { return buf_load(p + po, c * (unsigned)sizeof(*p)); }
  __device__ void center(long long po, unsigned c, T2 pv, T2 nb, const T& vv) {
    const T a = c0 + vv - eps;
    T2 h;
    h.x = a * pv.x + om * pv.y + nb.x;
    h.y = a * pv.y - om * pv.x + nb.y;
    buf_store(q + po, c * (unsigned)sizeof(h), h);
    mu_re += own ? (double)(pv.x * h.x - pv.y * h.y) : 0.0;
    mu_im += own ? (double)(pv.x * h.y + pv.y * h.x) : 0.0;
  }
};

// Plain operator application (test hook and stencil measurement); the
// vectors are stored in the compute precision.
template <typename T>
struct HPol {
  typedef typename V2<T>::t T2;
  const T2* x;
  T2* y;
  const T* v;
  T c0, sr, si;
  bool own;
  static constexpr int kPF = sizeof(T) == 4 ? 3 : 2;
  typedef T Aux;
  __device__ T aux(long long po, unsigned c) const { return buf_load(v + po, c * (unsigned)sizeof(*v)); }
  __device__ T2 load(long long po, unsigned c) const { return buf_load(x + po, c * (unsigned)sizeof(*x)); }
  __device__ void center(long long po, unsigned c, T2 xv, T2 nb, const T& vv) {
    const T a = c0 + vv - sr;
    T2 o;
    o.x = a * xv.x + si * xv.y + nb.x;
    o.y = a * xv.y - si * xv.x + nb.y;
    buf_store(y + po, c * (unsigned)sizeof(o), o);
  }
};

// ---------------------------------------------------------------------------
// Streaming passes of one system (whole workgroup).

// Point-major nonlocal entries and the coefficients w_p of p (null: none).
template <typename T>
struct NlPoint {
  const int* ptr;
  const int* proj;
  const T* v;
  const typename V2<T>::t* coef;
  __device__ __forceinline__ NlPoint from(long long i) const { return {ptr ? ptr + i : ptr, proj, v, coef}; }
};

// The streaming sweeps take kSweep elements per thread and trip, the next
// trip's loads issued before this trip's stores: loads and stores complete
// in order on one counter, so loads issued after stores would wait for them.

constexpr int kSweep = 4;

// Within a sweep an element's index is 32 bits; systems that may be longer
// (not whole-plane tiles) go in blocks of kSweepBlock elements.  64-bit
// indices cost the sweeps scalar registers (FP64 systems of 24^3 99 -> 102 ms).
constexpr int kSweepBlock = 1 << 30;
template <bool FULL, class F>
__device__ __forceinline__ void sweep_blocks(long long N, F&& f) {
  if constexpr (FULL) {
    f(0, (int)N);
  } else {
#pragma unroll 1
    for (long long i = 0; i < N; i += kSweepBlock) f(i, (int)min(N - i, (long long)kSweepBlock));
  }
}

template <class Load, class Use>
__device__ __forceinline__ int stream_sweep(int begin, int end, Load&& load, Use&& use) {
  const int trip = kSweep * (int)blockDim.x;
  const int full = (end - begin) / trip;   // trips without a bounds check
  if (full > 0) load(begin, 0);
  int i0 = begin;
#pragma unroll 1
  for (int k = 0; k + 2 <= full; k += 2) {
    load(i0 + trip, 1);
    use(i0, 0);
    if (k + 2 < full) load(i0 + 2 * trip, 0);
    use(i0 + trip, 1);
    i0 += 2 * trip;
  }
  if (full & 1) {
    use(i0, 0);
    i0 += trip;
  }
  return i0;                               // first element not done
}

// The residual of one system: its first `nl` elements (whole trips of the
// sweeps) live in LDS, the others in global memory.  Only the streaming
// sweeps touch it, each thread its own elements.
template <typename T>
struct SplitVec {
  typename V2<T>::t* l;
  typename V2<T>::t* g;
  int nl;
  __device__ __forceinline__ SplitVec from(long long i) const { return {l, g + i, i == 0 ? nl : 0}; }
};

// r -= alpha (q + V_nl p);  returns ||r||^2, r^T r.
template <typename T, bool NL>
__device__ __forceinline__ void residual_sweep(int N, const SplitVec<T>& r, const typename V2<T>::t* q, T ar, T ai,
                                               const NlPoint<T>& nl, double& rr, double& rho_re, double& rho_im) {
  typedef typename V2<T>::t T2;
  const int st = blockDim.x;
  const unsigned tid = opaque_tid();
  T2 qv[2][kSweep], rv[2][kSweep];
  auto one = [&](int i, T2 b, T2 a) RPA_INLINE {
    if constexpr (NL) nl_point<T>(nl.ptr, nl.proj, nl.v, nl.coef, i + (int)tid, b.x, b.y);
    a.x -= ar * b.x - ai * b.y;
    a.y -= ar * b.y + ai * b.x;
    const double sx = (double)a.x, sy = (double)a.y;
    rr += sx * sx + sy * sy;
    rho_re += sx * sx - sy * sy;
    rho_im += 2.0 * sx * sy;
    return a;
  };
  int i = stream_sweep(
      0, r.nl,
      [&](int i0, int h) RPA_INLINE {
#pragma unroll
        for (int u = 0; u < kSweep; ++u) qv[h][u] = at32(q + (i0 + u * st), tid);
      },
      [&](int i0, int h) RPA_INLINE {
#pragma unroll
        for (int u = 0; u < kSweep; ++u) {
          T2* rl = r.l + (i0 + u * st + (int)tid);
          *rl = one(i0 + u * st, qv[h][u], *rl);
        }
      });
  i = stream_sweep(
      i, N,
      [&](int i0, int h) RPA_INLINE {
#pragma unroll
        for (int u = 0; u < kSweep; ++u) {
          qv[h][u] = at32(q + (i0 + u * st), tid);
          rv[h][u] = at32(r.g + (i0 + u * st), tid);
        }
      },
      [&](int i0, int h) RPA_INLINE {
#pragma unroll
        for (int u = 0; u < kSweep; ++u) at32(r.g + (i0 + u * st), tid) = one(i0 + u * st, qv[h][u], rv[h][u]);
      });
  for (; i + (int)tid < N; i += st) at32(r.g + i, tid) = one(i, at32(q + i, tid), at32(r.g + i, tid));
}

// x (pend) += alpha p_old (xfresh: x = alpha p_old);  p = first ? r : r + beta p.
template <typename T>
__device__ __forceinline__ void direction_sweep(int N, const SplitVec<T>& r, typename V2<T>::t* p,
                                                typename V2<T>::t* x, T ar, T ai, T br, T bi, bool first, bool pend,
                                                bool xfresh) {
  typedef typename V2<T>::t T2;
  const int st = blockDim.x;
  const unsigned tid = opaque_tid();
  if (first || !pend || xfresh) {
    // the first iteration and the one after a fold: rare, so not pipelined
    for (int i = 0; i + (int)tid < N; i += st) {
      T2 a = i < r.nl ? r.l[i + (int)tid] : at32(r.g + i, tid);
      if (!first) {
        const T2 b = at32(p + i, tid);
        if (pend) at32(x + i, tid) = {ar * b.x - ai * b.y, ar * b.y + ai * b.x};
        a.x += br * b.x - bi * b.y;
        a.y += br * b.y + bi * b.x;
      }
      at32(p + i, tid) = a;
    }
    return;
  }
  T2 pv[2][kSweep], rv[2][kSweep], xv[2][kSweep];
  auto one = [&](int i, T2 a, T2 b, T2 c) RPA_INLINE {
    c.x += ar * b.x - ai * b.y;
    c.y += ar * b.y + ai * b.x;
    at32(x + i, tid) = c;
    a.x += br * b.x - bi * b.y;
    a.y += br * b.y + bi * b.x;
    at32(p + i, tid) = a;
  };
  int i = stream_sweep(
      0, r.nl,
      [&](int i0, int h) RPA_INLINE {
#pragma unroll
        for (int u = 0; u < kSweep; ++u) {
          pv[h][u] = at32(p + (i0 + u * st), tid);
          xv[h][u] = at32(x + (i0 + u * st), tid);
        }
      },
      [&](int i0, int h) RPA_INLINE {
#pragma unroll
        for (int u = 0; u < kSweep; ++u) one(i0 + u * st, r.l[i0 + u * st + (int)tid], pv[h][u], xv[h][u]);
      });
  i = stream_sweep(
      i, N,
      [&](int i0, int h) RPA_INLINE {
#pragma unroll
        for (int u = 0; u < kSweep; ++u) {
          rv[h][u] = at32(r.g + (i0 + u * st), tid);
          pv[h][u] = at32(p + (i0 + u * st), tid);
          xv[h][u] = at32(x + (i0 + u * st), tid);
        }
      },
      [&](int i0, int h) RPA_INLINE {
#pragma unroll
        for (int u = 0; u < kSweep; ++u) one(i0 + u * st, rv[h][u], pv[h][u], xv[h][u]);
      });
  for (; i + (int)tid < N; i += st) one(i, at32(r.g + i, tid), at32(p + i, tid), at32(x + i, tid));
}

// x += d (has_d) + alpha p (p non-null), the sum formed in the iteration's precision
template <typename T>
__device__ __forceinline__ void fold_pair(long long N, double2* x, const typename V2<T>::t* d, bool has_d,
                                          const typename V2<T>::t* p, T ar, T ai) {
  typedef typename V2<T>::t T2;
  for (long long i = threadIdx.x; i < N; i += blockDim.x) {
    T2 e = has_d ? d[i] : zero2<T2>();
    if (p) {
      const T2 pv = p[i];
      e.x += ar * pv.x - ai * pv.y;
      e.y += ar * pv.y + ai * pv.x;
    }
    double2 w = x[i];
    w.x += (double)e.x;
    w.y += (double)e.y;
    x[i] = w;
  }
}

__device__ __forceinline__ void zero_sweep(long long N, double2* x) {
  for (long long i = threadIdx.x; i < N; i += blockDim.x) x[i] = make_double2(0.0, 0.0);
}

// complex division a / b of uniform values; the quotient is uniform again (in
// scalar registers: held in vector registers across the sweeps, the solvers'
// scalars took room that the marches then spilled)
__device__ __forceinline__ void cdiv(double ar, double ai, double br, double bi, double& cr,
                                     double& ci) {
  const double den = br * br + bi * bi;
  cr = uni((ar * br + ai * bi) / den);
  ci = uni((ai * br - ar * bi) / den);
}

__device__ __forceinline__ void record(const CocgArgs& a, int s, int its, int cycles, int status) {
  // per-frequency statistics of finished solves; a solve the FP32 launch hands
  // over (status 3) is counted once, by the FP64 launch, with the FP32
  // iterations (still in out_iters) added; reliable updates are summed per bin
  if (a.ostats != nullptr && status != 3) {
    unsigned long long tot = (unsigned long long)its, cyc = (unsigned long long)cycles;
    if (a.is_followup) {
      tot += (unsigned long long)a.out_iters[s];
      cyc += (unsigned long long)a.out_cycles[s];
    }
    const int nb = a.n_bins;
    const int bin = a.obin[s / a.n_occ];
    atomicAdd(&a.ostats[bin], 1ULL);
    atomicAdd(&a.ostats[nb + bin], tot);
    atomicAdd(&a.ostats[2 * nb + bin], tot * tot);
    atomicMin(&a.ostats[3 * nb + bin], tot);
    atomicMax(&a.ostats[4 * nb + bin], tot);
    atomicAdd(&a.ostats[5 * nb + bin], cyc);
  }
  a.out_iters[s] = its;
  a.out_cycles[s] = cycles;
  a.out_status[s] = status;
  atomicAdd(&a.stats[0], (unsigned long long)its);
  atomicMax(&a.stats[1], (unsigned long long)its);
  atomicAdd(&a.stats[2], (unsigned long long)cycles);
  if (status == 1) atomicAdd(&a.stats[3], 1ULL);
  if (status == 2) atomicAdd(&a.stats[4], 1ULL);
  if (status == 3) atomicAdd(&a.stats[5], 1ULL);
}

// ---------------------------------------------------------------------------
// One system by plain COCG.
// FP64: x itself accumulates alpha p and the recursive residual decides.
// FP32 (REFINE): COCG with reliable updates (Sleijpen and van der Vorst,
// 1996): the search direction is kept for the whole solve, while every time
// the FP32 recursive residual has dropped by the factor delta (inner_tol) the
// FP32 correction d is folded into the FP64 solution and the residual is
// replaced by the true FP64 residual b - A x64.  Convergence is declared on
// the FP64 residual only.
template <bool REFINE, bool FULL, int HS, int PITCH, bool NL>
__device__ __forceinline__ void solve_plain(const CocgArgs& a, int s, char* smem, double* red, char* nlc) {
  typedef typename std::conditional<REFINE, float, double>::type T;
  typedef typename V2<T>::t T2;
  const Geom& g = a.g;
  const long long N = g.N;
  const int b = s / a.n_occ;
  const int n = s - b * a.n_occ;
  T2* r = reinterpret_cast<T2*>(a.slot_ws + (size_t)blockIdx.x * a.slot_bytes);
  T2* q = r + N;
  T2* p = r + 2 * (size_t)N;
  double2* x = a.x64 + (size_t)s * N;
  T2* d;                           // alpha p accumulates here
  if constexpr (REFINE) d = r + 3 * (size_t)N;
  else d = x;
  const SplitVec<T> rs{reinterpret_cast<T2*>(nlc + (size_t)a.nl.n_proj * sizeof(double2)), r, a.r_lds};
  const double eps = a.eps[n];
  const double om = a.omega[b];
  const int maxit = REFINE ? a.maxit32 : a.maxit;

  // nonlocal coefficients: FP64 for the residual sweeps, the iteration's
  // precision otherwise (same LDS region, never live at the same time)
  double2* coef64 = reinterpret_cast<double2*>(nlc);
  T2* coef = reinterpret_cast<T2*>(nlc);
  const NlPoint<T> nlp{a.nl.pm_ptr, a.nl.pm_proj, nl_pick<T>(a.nl.pm_v32, a.nl.pm_v64), coef};

  ResidPol<T, NL> rp;
  rp.x = x; rp.v = a.v64; rp.psi = a.psi64 + (size_t)n * N; rp.u = a.u64 + (size_t)b * N;
  rp.r = r; rp.c0 = a.c64.c0; rp.eps = eps; rp.om = om;
  rp.pm_ptr = a.nl.pm_ptr; rp.pm_proj = a.nl.pm_proj; rp.pm_v = a.nl.pm_v64;
  rp.coef = coef64;

  int its = 0, updates = 0, status = 0, last_upd = 0, no_gain = 0;
  bool failed = false;             // FP32 iteration produced a non-finite value
  bool start = true, resid = true; // the residual is (re)computed from x
  bool first = true, pend = false; // no direction yet; alpha p not in d yet
  bool dfresh = REFINE;            // d holds nothing yet
  double rnorm = 0.0, thr = 0.0;   // current residual estimate, its target
  double rmax = 0.0, best_true = 0.0;  // true residual at the last update, smallest seen
  double rho_r = 0.0, rho_i = 0.0, al_r = 0.0, al_i = 0.0, br = 0.0, bi = 0.0;
  for (;;) {
    double rho_nr, rho_ni;
    if (resid) {
      // r = b - A x in FP64 (stored rounded to T)
      if constexpr (NL) {
        double d0 = 0.0, d1 = 0.0;
        nl_project<double, double>(a.nl, x, coef64, d0, d1);
        __syncthreads();
      }
      rp.rr = rp.bb = rp.rho_re = rp.rho_im = 0.0;
      march<double, FULL, HS, PITCH>(g, a.c64, rp, reinterpret_cast<double2*>(smem), 0, g.ntiles, 0, g.nx);
      double w4[4] = {rp.rr, rp.bb, rp.rho_re, rp.rho_im};
      block_reduce<4>(w4, red);
      for (int i = threadIdx.x; i < rs.nl; i += blockDim.x) rs.l[i] = r[i];
      rnorm = uni(sqrt(w4[0]));
      rho_nr = w4[2];
      rho_ni = w4[3];
      rmax = rnorm;
      resid = false;
      if (start) {
        const double bnorm = sqrt(w4[1]);
        if (bnorm == 0.0) {
          zero_sweep(N, x);
          rnorm = 0.0;
          break;
        }
        thr = uni(a.tol * bnorm);
        best_true = rnorm;
      } else if (rnorm < 0.5 * best_true) {
        best_true = rnorm;
        no_gain = 0;
      } else if (++no_gain >= 4) {
        status = 1;                // FP32 stagnation
        break;
      }
    } else {
      double u3[3] = {0.0, 0.0, 0.0};
      sweep_blocks<FULL>(N, [&](long long i, int len) RPA_INLINE {
        residual_sweep<T, NL>(len, rs.from(i), q + i, uni((T)al_r), uni((T)al_i), nlp.from(i), u3[0], u3[1], u3[2]);
      });
      block_reduce<3>(u3, red);
      ++its;
      rnorm = uni(sqrt(u3[0]));
      rho_nr = u3[1];
      rho_ni = u3[2];
      if constexpr (REFINE) {
        if (!isfinite(rnorm) || !isfinite(rho_nr) || !isfinite(rho_ni)) { failed = true; break; }
        // reliable update when the recursive residual has dropped by delta, on
        // apparent convergence, and at least every kMaxGap iterations (an FP32
        // recursion that stalls above delta * rmax is caught there)
        if ((rnorm < a.inner_tol * rmax && its - last_upd >= kMinGap) || rnorm <= thr ||
            its - last_upd >= kMaxGap) {
          fold_pair<T>(N, x, d, !dfresh, p, uni((T)al_r), uni((T)al_i));
          __syncthreads();
          dfresh = true;
          pend = false;
          ++updates;
          last_upd = its;
          resid = true;
          continue;
        }
      }
    }
    if (!(rnorm > thr)) break;     // converged, or NaN
    if (!start) cdiv(rho_nr, rho_ni, rho_r, rho_i, br, bi);
    start = false;
    rho_r = rho_nr;
    rho_i = rho_ni;
    if (its >= maxit) { status = 1; break; }
    sweep_blocks<FULL>(N, [&](long long i, int len) RPA_INLINE {
      direction_sweep<T>(len, rs.from(i), p + i, d + i, uni((T)al_r), uni((T)al_i), uni((T)br), uni((T)bi), first, pend,
                         dfresh);
    });
    __syncthreads();
    if (pend) dfresh = false;
    pend = false;
    first = false;
    ApplyPol<T> ap;
    ap.p = p; ap.q = q; ap.v = nl_pick<T>(a.v32, a.v64);
    ap.eps = uni((T)eps); ap.om = uni((T)om);
    ap.mu_re = ap.mu_im = 0.0;
    if constexpr (REFINE) {
      ap.c0 = a.c32.c0;
      march<T, FULL, HS, PITCH>(g, a.c32, ap, reinterpret_cast<T2*>(smem), 0, g.ntiles, 0, g.nx);
    } else {
      ap.c0 = a.c64.c0;
      march<T, FULL, HS, PITCH>(g, a.c64, ap, reinterpret_cast<T2*>(smem), 0, g.ntiles, 0, g.nx);
    }
    double m2[2] = {ap.mu_re, ap.mu_im};
    if constexpr (NL) nl_project<T, T>(a.nl, p, coef, m2[0], m2[1]);
    block_reduce<2>(m2, red);
    if (REFINE && (!isfinite(m2[0]) || !isfinite(m2[1]))) { failed = true; break; }
    if (fabs(m2[0]) + fabs(m2[1]) < 1e-300) { status = 2; break; }
    cdiv(rho_r, rho_i, m2[0], m2[1], al_r, al_i);
    pend = true;
  }
  // a correction not in x yet (convergence in FP64, maxit and breakdown exits)
  if (!failed && (pend || (REFINE && !dfresh))) {
    __syncthreads();
    if constexpr (REFINE) fold_pair<T>(N, x, d, !dfresh, pend ? p : nullptr, uni((T)al_r), uni((T)al_i));
    else fold_pair<double>(N, x, nullptr, false, p, al_r, al_i);
    __syncthreads();
  }
  // FP32 not converged (maxit, stagnation, breakdown, non-finite values): x64
  // holds the last folded solution, which the FP64 launch continues from
  if (REFINE && (failed || status != 0 || !(rnorm <= thr)))
    status = a.fail_list ? 3 : (status ? status : 1);
  if (!REFINE && status == 0 && !(rnorm <= thr)) status = 1;   // NaN residual is not convergence
  if (threadIdx.x == 0) {
    record(a, s, its, updates, status);
    if (status == 3) a.fail_list[atomicAdd(a.fail_count, 1)] = s;
  }
}

// One system, preconditioned COCG (passes in precond_impl.h).  FP64: x
// itself accumulates alpha p.  FP32 (REFINE): reliable updates as above.
// q = A p follows its recurrence; every QR iterations or so it is formed
// afresh from p (q = M p + (V - shift) p, one more application of the basis
// transforms), at a reliable update in FP32.  FP64 takes 8: rounding in the
// recurrence ends the longest solves early (24^3, tol 1e-10, right-hand sides
// perturbed by 1e-15: 94 iterations at an unrecurred q and at 8, 91 in half of
// the runs at 24 or without).  At 8, iterations and true residuals are those of
// q formed by the stencil in each iteration on nine grids from 7x8x9 to 48^3,
// omega 0.02 to 49, tol 1e-8 to 1e-13.  FP32 measures its true residual and
// takes 24.
//
// Where a few iterations reach the FP32 rounding of A x (omega far above the
// potential), the recursive residual has fallen below the true one when that is
// measured.  beta then compares the new residual with one that the kept
// direction no longer belongs to, and with q from the recurrence the solve
// stalls or diverges: at omega 49.4, tol 1e-10 on nine grids 171 iterations in
// the mean and 99 of 520 systems handed to FP64 (q by the stencil: 12 and 0; at
// 187 all were handed over either way).  So a true residual kRestart times the
// recursive one leaves the direction: 6 iterations there, none handed over up to
// omega 2000.  Slow solves pass the test; kRestart 1.01 costs 2% more iterations
// at omega 0.02 than 1.1, which at omega 30 lets single systems take 22 instead of 7.
constexpr double kRestart = 1.03;

template <bool REFINE, bool FULL, int HS, int PITCH, bool NL>
__device__ __forceinline__ void solve_pc(const CocgArgs& a, int s, char* smem, double* red, char* nlc) {
  typedef typename std::conditional<REFINE, float, double>::type T;
  typedef typename V2<T>::t T2;
  constexpr int QR = REFINE ? 24 : 8;
  const Geom& g = a.g;
  const long long N = g.N;
  const int b = s / a.n_occ;
  const int n = s - b * a.n_occ;
  T2* r = reinterpret_cast<T2*>(a.slot_ws + (size_t)blockIdx.x * a.slot_bytes);
  T2* q = r + N;
  T2* p = r + 2 * N;
  T2* t = r + 3 * N;
  double2* x = a.x64 + (size_t)s * N;
  T2* d;                           // alpha p accumulates here
  if constexpr (REFINE) d = r + 4 * N;
  else d = x;
  const double eps = a.eps[n];
  const double om = a.omega[b];
  const T sr = uni((T)fmax(a.prec->vbar - eps, a.prec->floor)), si = uni((T)(-om));
  double2* coef64 = reinterpret_cast<double2*>(nlc);
  T2* coef = reinterpret_cast<T2*>(nlc);
  const int* pm_ptr = a.nl.pm_ptr;
  const int* pm_proj = a.nl.pm_proj;
  const T* pm_v = nl_pick<T>(a.nl.pm_v32, a.nl.pm_v64);
  auto nlp = [&](long long i, T2& qv) {
    if constexpr (NL) nl_point<T>(pm_ptr, pm_proj, pm_v, coef, i, qv.x, qv.y);
  };
  // the recursive residual across a reliable update: whole-plane tiles keep it
  // above what reductions of two values use of their buffer (as a live scalar it
  // cost their passes 1 to 5%), the others in rmax (in LDS it cost them 2%)
  double* rec_lds = nullptr;
  if constexpr (REFINE && FULL) rec_lds = red + 2 * ((blockDim.x >> 6) + 1);
  const int maxit = REFINE ? a.maxit32 : a.maxit;

  ResidPol<T, NL> rp;
  rp.x = x; rp.v = a.v64; rp.psi = a.psi64 + (size_t)n * N; rp.u = a.u64 + (size_t)b * N;
  rp.r = r; rp.c0 = a.c64.c0; rp.eps = eps; rp.om = om;
  rp.pm_ptr = a.nl.pm_ptr; rp.pm_proj = a.nl.pm_proj; rp.pm_v = a.nl.pm_v64;
  rp.coef = coef64;

  int its = 0, updates = 0, status = 0, last_upd = 0, last_q = 0, no_gain = 0;
  bool failed = false, start = true, resid = true, upd = false, first = true, pend = false;
  bool dfresh = REFINE, refresh = false;
  double rnorm = 0.0, thr = 0.0, rmax = 0.0, best_true = 0.0;
  double rho_r = 0.0, rho_i = 0.0, al_r = 0.0, al_i = 0.0;
  for (;;) {
    if (resid) {
      // r = b - A x in FP64
      if constexpr (NL) {
        double d0 = 0.0, d1 = 0.0;
        nl_project<double, double>(a.nl, x, coef64, d0, d1);
        __syncthreads();
      }
      rp.rr = rp.bb = rp.rho_re = rp.rho_im = 0.0;
      march<double, FULL, HS, PITCH>(g, a.c64, rp, reinterpret_cast<double2*>(smem), 0, g.ntiles, 0, g.nx);
      double w2[2] = {rp.rr, rp.bb};
      block_reduce<2>(w2, red);
      rnorm = uni(sqrt(w2[0]));
      if constexpr (REFINE) {
        double rec = rmax;         // the recursive residual, set at the update
        if constexpr (FULL) rec = uni(*rec_lds);
        if (!start && rnorm > kRestart * rec) {
          first = true;            // leave the search direction
          last_q = its;
        }
      }
      rmax = rnorm;
      if (start) {
        const double bnorm = sqrt(w2[1]);
        if (bnorm == 0.0) {
          zero_sweep(N, x);
          rnorm = 0.0;
          break;
        }
        thr = uni(a.tol * bnorm);
        best_true = rnorm;
        start = false;
      } else if (rnorm < 0.5 * best_true) {
        best_true = rnorm;
        no_gain = 0;
      } else if (++no_gain >= 4) {
        status = 1;                                    // FP32 stagnation
        break;
      }
      if (!(rnorm > thr)) break;
      resid = false;
      upd = false;
      refresh = !first && its - last_q >= QR;
      PcCtx<T>(g, *a.prec, smem).stage();
      __syncthreads();
    }
    double rr[1] = {0.0};
    pc_forward<T>(PcCtx<T>(g, *a.prec, smem), refresh ? p : r, q, t, upd, uni((T)al_r), uni((T)al_i), nlp, rr[0]);
    if (upd) {
      block_reduce<1>(rr, red);
      ++its;
      rnorm = uni(sqrt(rr[0]));
      if constexpr (REFINE) {
        if (!isfinite(rnorm)) { failed = true; break; }
        // reliable update when the recursive residual has dropped by delta, on
        // apparent convergence, and at least every kMaxGap iterations
        if ((rnorm < a.inner_tol * rmax && its - last_upd >= kMinGap) || rnorm <= thr ||
            its - last_upd >= kMaxGap) {
          if constexpr (FULL) {
            if (threadIdx.x == 0) *rec_lds = rnorm;
          } else {
            rmax = rnorm;
          }
          fold_pair<T>(N, x, d, !dfresh, p, uni((T)al_r), uni((T)al_i));
          __syncthreads();
          dfresh = true;
          pend = false;
          ++updates;
          last_upd = its;
          resid = true;
          continue;
        }
      } else {
        if (!(rnorm > thr)) break;                     // converged, or NaN
        if (its - last_q >= QR) {
          // p has its last alpha pending; q is stale only for the next beta
          refresh = true;
          upd = false;
          last_q = its;
          continue;
        }
      }
    } else if (!refresh) {
      __syncthreads();
    }
    if (!refresh && its >= maxit) { status = 1; break; }
    double q2[2] = {0.0, 0.0};
    pc_modes<T>(PcCtx<T>(g, *a.prec, smem), *a.prec, t, sr, si, refresh, q2[0], q2[1]);
    block_reduce<2>(q2, red);
    PcUpdate<T> u;
    u.r = r; u.p = p; u.q = q; u.d = d; u.v = nl_pick<T>(a.v32, a.v64);
    u.shift = uni((T)(eps + fmax(a.prec->vbar - eps, a.prec->floor)));
    u.ar = uni((T)al_r); u.ai = uni((T)al_i);
    u.first = first; u.pend = pend && !refresh; u.dfresh = dfresh; u.refresh = refresh;
    u.br = u.bi = 0;
    if (!refresh) {
      if (REFINE && (!isfinite(q2[0]) || !isfinite(q2[1]))) { failed = true; break; }
      if (fabs(q2[0]) + fabs(q2[1]) < 1e-300) { status = 2; break; }
      if (!first) {
        double br, bi;
        cdiv(q2[0], q2[1], rho_r, rho_i, br, bi);
        u.br = uni((T)br);
        u.bi = uni((T)bi);
      }
      rho_r = q2[0];
      rho_i = q2[1];
    }
    double m2[2] = {0.0, 0.0};
    pc_inverse<T>(PcCtx<T>(g, *a.prec, smem), t, u, m2[0], m2[1]);
    if (refresh) {
      refresh = false;
      last_q = its;
      continue;
    }
    if (pend) dfresh = false;
    pend = false;
    first = false;
    if constexpr (NL) nl_project<T, T>(a.nl, p, coef, m2[0], m2[1]);
    block_reduce<2>(m2, red);
    if (REFINE && (!isfinite(m2[0]) || !isfinite(m2[1]))) { failed = true; break; }
    if (fabs(m2[0]) + fabs(m2[1]) < 1e-300) { status = 2; break; }
    cdiv(rho_r, rho_i, m2[0], m2[1], al_r, al_i);
    upd = true;
    pend = true;
  }
  // a correction not in x yet (convergence in FP64, maxit and breakdown exits)
  if (!failed && (pend || (REFINE && !dfresh))) {
    __syncthreads();
    if constexpr (REFINE) fold_pair<T>(N, x, d, !dfresh, pend ? p : nullptr, uni((T)al_r), uni((T)al_i));
    else fold_pair<double>(N, x, nullptr, false, p, al_r, al_i);
    __syncthreads();
  }
  // FP32 not converged (maxit, stagnation, breakdown, non-finite values): x64
  // holds the last folded solution, which the FP64 launch continues from
  if (REFINE && (failed || status != 0 || !(rnorm <= thr)))
    status = a.fail_list ? 3 : (status ? status : 1);
  if (!REFINE && status == 0 && !(rnorm <= thr)) status = 1;   // NaN residual is not convergence
  if (threadIdx.x == 0) {
    record(a, s, its, updates, status);
    if (status == 3) a.fail_list[atomicAdd(a.fail_count, 1)] = s;
  }
}

// M: 0 = tile covers the whole plane, 1 = y halo with one slot per thread,
// 2 = y halo with two slots per thread.  PITCH: LDS row pitch (>= nz + 2R).
// V: bit 0 = nonlocal projector term (separate kernels, so the projector-free
// ones carry none of its code or registers), bit 1 = preconditioned solves.
template <bool REFINE, int M, int PITCH, int V>
__global__ void __launch_bounds__(kMaxBlock) k_cocg(CocgArgs a) {
  constexpr bool NL = (V & 1) != 0;
  constexpr bool PC = (V & 2) != 0;
  constexpr bool FULL = M == 0;
  constexpr int HS = M == 2 ? 2 : 1;
  // All LDS is dynamic, so that what setup accepts is what a launch may use, and
  // starts aligned: behind a static int the buffer began at 8, where each
  // ds_read_b128 took 54 cycles of the LDS instead of 8 (the FP64 stencil sweep
  // of a 24^3 system 165 us instead of 30)
  extern __shared__ __attribute__((aligned(256))) double smem_d[];
  char* smem = reinterpret_cast<char*>(smem_d);
  const Geom& g = a.g;
  double* red = reinterpret_cast<double*>(smem + lds_plane_bytes(g, PITCH, REFINE));
  char* nlc = smem + lds_plane_bytes(g, PITCH, REFINE) + red_bytes(blockDim.x);
  // the next system's index travels in the reduction buffer: block_reduce ends
  // with a barrier after its last read, so between systems nothing is live there
  int* s_item = reinterpret_cast<int*>(red);
  int item = 0;
  // the FP64 launch after an FP32 one takes the systems the latter handed over
  const int n_items = a.n_items_dev ? uni(*a.n_items_dev) : a.n_items;
  if (threadIdx.x == 0) *s_item = atomicAdd(a.counter, 1);
  __syncthreads();
  item = uni(*s_item);
  __syncthreads();
  while (item < n_items) {
    const int s = uni(a.order[item]);
    const int b = s / a.n_occ;
    const int live = a.active == nullptr ? 1 : uni(a.active[b]);
    if (live) {
      if constexpr (PC) solve_pc<REFINE, FULL, HS, PITCH, NL>(a, s, smem, red, nlc);
      else solve_plain<REFINE, FULL, HS, PITCH, NL>(a, s, smem, red, nlc);
    } else if (threadIdx.x == 0) {
      a.out_iters[s] = 0;
      a.out_cycles[s] = 0;
      a.out_status[s] = 0;
    }
    if (threadIdx.x == 0) *s_item = atomicAdd(a.counter, 1);
    __syncthreads();
    item = uni(*s_item);
    __syncthreads();
  }
}

}  // namespace
}  // namespace rpa
