// Plain FP64 COCG of small systems with the search direction in LDS and the
// residual and A p in registers.
//
// The marching solver (cocg_impl.h) moves about 11 vector passes per
// iteration, and its plane-by-plane sequence of barriers leaves grids of a few
// thousand points bound by latency.  Here a thread owns the column t mod
// (ny nz) in every G-th plane, so that element k of thread t is point
// t + k G ny nz: p is written once per iteration, one barrier, and every point
// takes its 36 neighbours from LDS.  Of the vectors only the solution is read
// and written in memory.  Bound by instruction issue (about 250 vector
// instructions per point and wave, 92 of them FP64).  The compiler spills 149
// registers, most of them around the opening residual's march: an iteration of
// about 4500 instructions reloads 69 values.
#include "cocg_impl.h"

namespace rpa {

namespace {

// most elements per thread: r and q take 8 of its 168 registers per element
constexpr int kResidentMax = 12;
constexpr int kResidentChunk = 4;      // solution elements in flight per thread
constexpr int kResidentPitch = 56;     // of the residual's march (nz <= 44)

// elements beyond the bound read as zero and are not written
__device__ __forceinline__ __amdgpu_buffer_rsrc_t bounded(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00027000);
}
__device__ __forceinline__ double2 bnd_load(__amdgpu_buffer_rsrc_t d, int i) {
  return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(d, (unsigned)i * 16u, 0, 0));
}
__device__ __forceinline__ void bnd_store(__amdgpu_buffer_rsrc_t d, int i, double2 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(buf_u4, v), d, (unsigned)i * 16u, 0, 0);
}

// The recurrences, stopping rule and status values are solve_plain<false>'s.
__device__ __forceinline__ void solve_resident(const CocgArgs& a, int groups, int per, int s, char* smem, double* red) {
  constexpr int K = kResidentMax, C = kResidentChunk;
  constexpr unsigned SZ = sizeof(double2);
  static_assert(K % C == 0, "whole chunks");
  const Geom& g = a.g;
  const int N = (int)g.N, plane = g.ny * g.nz, stride = groups * plane;
  const int b = s / a.n_occ;
  const int n = s - b * a.n_occ;
  double2* rg = reinterpret_cast<double2*>(a.slot_ws + (size_t)blockIdx.x * a.slot_bytes);
  double2* x = a.x64 + (size_t)s * N;
  double2* ps = reinterpret_cast<double2*>(smem);
  const double eps = a.eps[n];
  const double om = a.omega[b];
  // first point; threads without a column start beyond the end
  const int tid = (int)threadIdx.x < stride ? (int)threadIdx.x : N;
  double2 r[K];

  ResidPol<double, false> rp;
  rp.x = x; rp.v = a.v64; rp.psi = a.psi64 + (size_t)n * N; rp.u = a.u64 + (size_t)b * N;
  rp.r = rg; rp.c0 = a.c64.c0; rp.eps = eps; rp.om = om;
  rp.pm_ptr = nullptr; rp.pm_proj = nullptr; rp.pm_v = nullptr; rp.coef = nullptr;
  rp.rr = rp.bb = rp.rho_re = rp.rho_im = 0.0;
  march<double, true, 1, kResidentPitch>(g, a.c64, rp, reinterpret_cast<double2*>(smem), 0, 1, 0, g.nx);
  double w4[4] = {rp.rr, rp.bb, rp.rho_re, rp.rho_im};
  block_reduce<4>(w4, red);
  double rnorm = uni(sqrt(w4[0]));
  double rho_nr = w4[2], rho_ni = w4[3];
  const double bnorm = sqrt(w4[1]);
  const double thr = uni(a.tol * bnorm);
  int its = 0, status = 0;
  bool pend = false;               // alpha p not in x yet
  double rho_r = 0.0, rho_i = 0.0, al_r = 0.0, al_i = 0.0, br = 0.0, bi = 0.0;
  if (bnorm == 0.0) {
    zero_sweep(N, x);
    rnorm = 0.0;
  } else {
    const __amdgpu_buffer_rsrc_t rb = bounded(rg, SZ * (unsigned)N);
    static_for<K>([&](auto I) RPA_INLINE { r[I] = bnd_load(rb, tid + I * stride); });
    const __amdgpu_buffer_rsrc_t xb = bounded(x, SZ * (unsigned)N);
    while (rnorm > thr) {          // NaN ends it
      const bool first = its == 0;
      if (!first) cdiv(rho_nr, rho_ni, rho_r, rho_i, br, bi);
      rho_r = rho_nr;
      rho_i = rho_ni;
      if (its >= a.maxit) { status = 1; break; }
      // x += alpha p_old;  p = r + beta p_old
      static_for<K / C>([&](auto J) RPA_INLINE {
        if (J * C < per) {
          double2 xv[C];
          if (!first) {
            static_for<C>([&](auto U) RPA_INLINE { xv[U] = bnd_load(xb, tid + (J * C + U) * stride); });
          }
          static_for<C>([&](auto U) RPA_INLINE {
            constexpr int k = J * C + U;
            const int i = tid + k * stride;
            if (i < N) {
              double2 e = r[k];
              if (!first) {
                const double2 o = ps[i];
                xv[U].x += al_r * o.x - al_i * o.y;
                xv[U].y += al_r * o.y + al_i * o.x;
                e.x += br * o.x - bi * o.y;
                e.y += br * o.y + bi * o.x;
              }
              ps[i] = e;
            }
          });
          if (!first) {
            static_for<C>([&](auto U) RPA_INLINE { bnd_store(xb, tid + (J * C + U) * stride, xv[U]); });
          }
        }
      });
      pend = false;
      __syncthreads();
      // q = (H - sigma) p at the thread's points, mu = p^T q
      double m2[2] = {0.0, 0.0};
      double2 q[K];
      {
        const StencilCoef<double>& cf = a.c64;
        const int t = opaque_tid();
        const int t0 = t < stride ? t : N;
        const int col = t % plane, y = col / g.nz, z = col - y * g.nz;
        unsigned yo[2 * R], zo[2 * R];   // byte offsets of the neighbours in the plane
        static_for<R>([&](auto J) RPA_INLINE {
          constexpr int j = J + 1;
          const int yp = y + j, ym = y - j, zp = z + j, zm = z - j;
          yo[J] = SZ * (unsigned)((yp >= g.ny ? yp - g.ny : yp) * g.nz + z);
          yo[R + J] = SZ * (unsigned)((ym < 0 ? ym + g.ny : ym) * g.nz + z);
          zo[J] = SZ * (unsigned)(y * g.nz + (zp >= g.nz ? zp - g.nz : zp));
          zo[R + J] = SZ * (unsigned)(y * g.nz + (zm < 0 ? zm + g.nz : zm));
        });
        const unsigned PB = SZ * (unsigned)plane, NB = SZ * (unsigned)N, cb = SZ * (unsigned)col;
        auto at = [&](unsigned o) RPA_INLINE { return *reinterpret_cast<const double2*>(smem + o); };
        static_for<K>([&](auto I) RPA_INLINE {
          q[I] = make_double2(0.0, 0.0);
          if (I < per) {
            const int i = t0 + I * stride;
            if (i < N) {
              const double vv = buf_load(a.v64, (unsigned)i * 8u);
              const unsigned o = SZ * (unsigned)i, pb = o - cb;
              double2 sx = make_double2(0.0, 0.0), sy = sx, sz = sx;
              static_for<R>([&](auto J) RPA_INLINE {
                const double w = cf.w[J + 1];
                // planes wrap at the ends of the array: the smaller of the two unsigned offsets is inside
                const unsigned up = o + (J + 1) * PB, dn = o - (J + 1) * PB;
                const double2 xa = at(min(up, up - NB)), xc = at(min(dn, dn + NB));
                const double2 ya = at(pb + yo[J]), yc = at(pb + yo[R + J]);
                const double2 za = at(pb + zo[J]), zc = at(pb + zo[R + J]);
                sx.x += w * (xa.x + xc.x);
                sx.y += w * (xa.y + xc.y);
                sy.x += w * (ya.x + yc.x);
                sy.y += w * (ya.y + yc.y);
                sz.x += w * (za.x + zc.x);
                sz.y += w * (za.y + zc.y);
              });
              const double2 pv = at(o);
              const double c = cf.c0 + vv - eps;
              double2 h;
              h.x = c * pv.x + om * pv.y + (cf.sx * sx.x + cf.sy * sy.x + cf.sz * sz.x);
              h.y = c * pv.y - om * pv.x + (cf.sx * sx.y + cf.sy * sy.y + cf.sz * sz.y);
              q[I] = h;
              m2[0] += pv.x * h.x - pv.y * h.y;
              m2[1] += pv.x * h.y + pv.y * h.x;
            }
          }
        });
      }
      block_reduce<2>(m2, red);
      if (fabs(m2[0]) + fabs(m2[1]) < 1e-300) { status = 2; break; }
      cdiv(rho_r, rho_i, m2[0], m2[1], al_r, al_i);
      pend = true;
      // r -= alpha q; elements beyond the end are zero in both
      double u3[3] = {0.0, 0.0, 0.0};
      static_for<K>([&](auto I) RPA_INLINE {
        if (I < per) {
          r[I].x -= al_r * q[I].x - al_i * q[I].y;
          r[I].y -= al_r * q[I].y + al_i * q[I].x;
          u3[0] += r[I].x * r[I].x + r[I].y * r[I].y;
          u3[1] += r[I].x * r[I].x - r[I].y * r[I].y;
          u3[2] += 2.0 * r[I].x * r[I].y;
        }
      });
      block_reduce<3>(u3, red);
      ++its;
      rnorm = uni(sqrt(u3[0]));
      rho_nr = u3[1];
      rho_ni = u3[2];
    }
    if (pend) {                    // the last direction's share
#pragma unroll 1
      for (int i = tid; i < N; i += stride) {
        const double2 o = ps[i];
        double2 w = x[i];
        w.x += al_r * o.x - al_i * o.y;
        w.y += al_r * o.y + al_i * o.x;
        x[i] = w;
      }
    }
  }
  __syncthreads();
  if (status == 0 && !(rnorm <= thr)) status = 1;   // NaN residual is not convergence
  if (threadIdx.x == 0) record(a, s, its, 0, status);
}

__global__ void __launch_bounds__(kMaxBlock) k_cocg_resident(CocgArgs a, int groups, int per, int lds) {
  extern __shared__ __attribute__((aligned(256))) double smem_d[];
  char* smem = reinterpret_cast<char*>(smem_d);
  double* red = reinterpret_cast<double*>(smem + lds);
  __shared__ int s_item;
  const int n_items = a.n_items_dev ? uni(*a.n_items_dev) : a.n_items;
  // the next item is drawn at the end of a pass, before a barrier: drawn at the
  // head of the loop it let the compiler join this test of the thread id with
  // the one that ends a solve, and put the loop's barriers into divergent flow
  if (threadIdx.x == 0) s_item = atomicAdd(a.counter, 1);
  __syncthreads();
  int item = uni(s_item);
  __syncthreads();
  while (item < n_items) {
    const int s = uni(a.order[item]);
    const int live = a.active == nullptr ? 1 : uni(a.active[s / a.n_occ]);
    if (live) {
      solve_resident(a, groups, per, s, smem, red);
    } else if (threadIdx.x == 0) {
      a.out_iters[s] = 0;
      a.out_cycles[s] = 0;
      a.out_status[s] = 0;
    }
    if (threadIdx.x == 0) s_item = atomicAdd(a.counter, 1);
    __syncthreads();
    item = uni(s_item);
    __syncthreads();
  }
}

}  // namespace

// FP64, whole-plane tiles, no projectors.  Measured with 8 orbitals (marching
// -> this, ms): 1024 systems of 24x16x24 19.9 -> 12.8, of 16^3 9.4 -> 7.3, of
// 12^3 3.9 -> 3.7, of 10x11x12 3.7 -> 3.5; 32 systems of 12^3 1.52 -> 1.12.  With
// planes of 128 points and less the marching solver's small workgroups share
// a compute unit: 1024 of 8x8x16 2.4 -> 2.6.  The same in FP32, where the
// neighbours' addresses cost more than the 97 instructions of a point, was
// slower from 12^3 (3.6 -> 4.5) to 24^3 (16.0 -> 20.7).
bool launch_cocg_resident(const CocgArgs& a, bool fp32_refine, int grid, hipStream_t s) {
  const Geom& g = a.g;
  const long long plane = (long long)g.ny * g.nz;
  if (fp32_refine || a.prec || a.nl.n_proj > 0 || g.ty != g.ny || g.nz + 2 * R > kResidentPitch || plane <= 128 ||
      plane > kMaxBlock)
    return false;
  // planes per thread, and the fewest groups of columns that keep it
  const int most = (int)(kMaxBlock / plane);
  const int per = (g.nx + most - 1) / most;
  const int groups = (g.nx + per - 1) / per;
  if (per > kResidentMax) return false;
  const int block = (int)((groups * plane + 63) / 64 * 64);
  const size_t march = 2 * (size_t)(g.ny + 2 * R) * kResidentPitch * sizeof(double2);
  const size_t dir = (size_t)g.N * sizeof(double2);
  const size_t lds = ((march > dir ? march : dir) + 255) & ~(size_t)255;
  const size_t shmem = lds + red_bytes(block);
  if (shmem + 256 > 160 * 1024) return false;
  hipLaunchKernelGGL(k_cocg_resident, dim3(grid), dim3(block), shmem, s, a, groups, per, (int)lds);
  return true;
}

}  // namespace rpa
