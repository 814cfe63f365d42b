// Preconditioned COCG for one system per persistent workgroup (preconditioned
// Sternheimer solves, named in the Conclusions and Future Work section).  The
// preconditioner is M = -1/2 Lap_h + sigma with the same 12th-order FD
// Laplacian as in H, inverted exactly in its per-axis eigenbasis:
//
//   z = M^-1 r = (Vx (x) Vy (x) Vz) diag(1 / (kx_a + ky_b + kz_c + sigma)) (Vx (x) Vy (x) Vz)^T r
//
// Im sigma = -omega, so A - M = V - eps_n - Re sigma is a real diagonal and
// A z = r + (V - eps_n - Re sigma) z needs no stencil: with it
// q = A p = A z + beta q_old is pointwise like p = z + beta p_old.  One
// iteration is three passes over the grid, each fused with the vector
// updates that its data allow:
//
//   forward   per x-planes:   r -= alpha q (||r||^2), t = Vy^T R Vz
//   modes     per 16 columns: t = Vx diag(scale) Vx^T t, rho = r^T z taken
//                             from the forward coefficients
//   inverse   per x-planes:   z = Vy T Vz^T; d += alpha_old p; p = z + beta p;
//                             q = r + (V - shift) z + beta q; mu = p^T q
//
// Per point and iteration 14 vector passes (112 B in FP32), against 20 for
// a separate M^-1 apply, stencil sweep (with its halo) and update sweep, and
// no stencil.  The contractions run on the 16x16x4 matrix-core
// instructions, both products of a pass chained in registers: with K taken
// in the order in which the accumulator holds its rows, an accumulator tile
// is the next product's B operand.  Several planes share a barrier (as many
// as give every wave an output tile), the next planes' loads are in
// registers meanwhile, and the modes pass has no barrier at all.
//
// Bound by the traffic of its 14 passes.  Measured against a stencil sweep on
// z plus three separate transform passes (16-row tiles, bases and planes in
// LDS): chi0 on 36x24x20 with 24 orbitals and 24 vectors, FP32 to 1e-10,
// 41.7 -> 14.8 ms; the preconditioned launches of 16 start vectors on 48^3
// with 128 orbitals 244 -> 108 ms.
#pragma once

#include "internal.h"

namespace rpa {

namespace {

typedef float mf4 __attribute__((ext_vector_type(4)));
typedef double md4 __attribute__((ext_vector_type(4)));

template <typename T> struct Mma;
template <> struct Mma<float> {
  typedef mf4 acc;
  static __device__ __forceinline__ acc step(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // accumulator v of lane l holds output row kL (l / 16) + kV v, column l % 16
  static constexpr int kL = 4, kV = 1;
};
template <> struct Mma<double> {
  typedef md4 acc;
  static __device__ __forceinline__ acc step(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static constexpr int kL = 1, kV = 4;
};

template <typename T>
__device__ __forceinline__ const T* prec_pick(const float* a, const double* b) {
  if constexpr (sizeof(T) == 4) return a;
  else return b;
}

__host__ __device__ inline int prec_pad(int n) { return (n + 15) & ~15; }

// The accepted problem sizes: two complex planes of the padded size and two
// bases in LDS, and kPrecRegs plane elements per thread of the stencil tile's
// workgroup (the solver itself needs less: with one plane per round at most
// 84 KB next to the reduction buffer and the projector coefficients).
constexpr int kPrecRegs = 4;
__host__ __device__ inline size_t prec_lds_bytes(const Geom& g, size_t elem) {
  const int px = prec_pad(g.nx), py = prec_pad(g.ny), pz = prec_pad(g.nz);
  const int rows = px > py ? px : py;
  const int pm = rows > pz ? rows : pz;
  const size_t ld = (size_t)pz + 1;
  const size_t bas = 2 * (size_t)pm * (pm + 1);
  return ((4 * (size_t)rows * ld + bas) * elem + 255) & ~(size_t)255;
}
__host__ __device__ inline int prec_regs(const Geom& g, int block) {
  const int px = prec_pad(g.nx), py = prec_pad(g.ny), pz = prec_pad(g.nz);
  const int e = (px > py ? px : py) * pz;
  return (e + block - 1) / block;
}

// Plane elements each thread prefetches per round of planes.
template <typename T>
constexpr int pc_elems() { return sizeof(T) == 4 ? 12 : 6; }

// LDS of the solver: the three bases (FP32; the FP64 bases stay in global
// memory) and `planes` padded complex planes.  One compile-time row stride
// for all (odd: the 16 rows of an operand fall into different banks), so that
// operand reads are immediate offsets from a few addresses.
constexpr int kPcLd = kMaxPrecDim + 1;
__host__ __device__ inline size_t pc_lds_bytes(const Geom& g, size_t elem, int planes) {
  const size_t px = prec_pad(g.nx), py = prec_pad(g.ny), pz = prec_pad(g.nz);
  const size_t bas = elem == 4 ? px + py + pz : 0;
  return ((bas + 2 * (size_t)planes * py) * kPcLd * elem + 255) & ~(size_t)255;
}

// Planes per round: an output tile (16 columns of one plane) for every wave,
// within the prefetch registers and `lds` bytes.
template <typename T>
int pc_planes(const Geom& g, int block, size_t lds) {
  const int ct = prec_pad(g.nz) / 16, waves = block / 64;
  int p = waves / ct;
  const long long most = (long long)pc_elems<T>() * block / ((long long)g.ny * g.nz);
  if (p > most) p = (int)most;
  if (p > g.nx) p = g.nx;
  while (p > 1 && pc_lds_bytes(g, sizeof(T), p) > lds) --p;
  return p < 1 ? 1 : p;
}

template <typename T>
struct PcCtx {
  typedef typename V2<T>::t T2;
  static constexpr int kL = Mma<T>::kL, kV = Mma<T>::kV;
  const Geom& g;
  int px, py, pz, slab;            // padded sizes, elements of one LDS plane component
  int ry, rx, ct;                  // 16-row tiles in y and x, 16-column tiles in z
  int planes, plane;               // planes per round, elements of a grid plane
  unsigned mz, my;                 // exact division by nz and ny for small dividends
  const T* bas[3];                 // LDS bases (FP32)
  const T* fw[3];                  // padded bases in global memory, grid-major and mode-major
  const T* iv[3];
  T* pl;                           // LDS planes: [plane][re, im][py][kPcLd]
  int tid, lane, li, lk, wave, nw, bs;

  __device__ __forceinline__ PcCtx(const Geom& g_, const PrecArgs& pa, char* smem) : g(g_) {
    px = prec_pad(g.nx); py = prec_pad(g.ny); pz = prec_pad(g.nz);
    slab = py * kPcLd;
    rx = px >> 4; ry = py >> 4; ct = pz >> 4;
    planes = sizeof(T) == 4 ? g.pc_planes32 : g.pc_planes64;
    plane = g.ny * g.nz;
    mz = 0xffffffffu / (unsigned)g.nz + 1;
    my = 0xffffffffu / (unsigned)g.ny + 1;
    T* s = reinterpret_cast<T*>(smem);
    bas[0] = s;
    bas[1] = s + (sizeof(T) == 4 ? px * kPcLd : 0);
    bas[2] = bas[1] + (sizeof(T) == 4 ? py * kPcLd : 0);
    pl = const_cast<T*>(bas[2]) + (sizeof(T) == 4 ? pz * kPcLd : 0);
    for (int a = 0; a < 3; ++a) {
      fw[a] = prec_pick<T>(pa.v32[a], pa.v64[a]);
      iv[a] = prec_pick<T>(pa.vt32[a], pa.vt64[a]);
    }
    tid = opaque_tid();
    lane = tid & 63;
    li = lane & 15;
    lk = lane >> 4;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    bs = blockDim.x;
    nw = bs >> 6;
  }

  // Element (k0 + kl * lk, o0 + li) of a basis, k0 and o0 uniform: forward k =
  // grid point, o = mode; inverse the other way round.
  template <bool FWD, int AXIS>
  __device__ __forceinline__ T basis(int k0, int kl, int o0) const {
    if constexpr (sizeof(T) == 4) {
      return FWD ? bas[AXIS][(kl * lk * kPcLd + li) + (k0 * kPcLd + o0)]
                 : bas[AXIS][(li * kPcLd + kl * lk) + (o0 * kPcLd + k0)];
    } else {
      const int l = AXIS == 0 ? px : (AXIS == 1 ? py : pz);
      const T* b = (FWD ? fw[AXIS] : iv[AXIS]) + (k0 * l + o0);
      return b[(unsigned)(kl * lk * l + li)];
    }
  }

  // bases into LDS and zeros into the planes (whose padding is never written
  // again); the caller synchronises
  __device__ __forceinline__ void stage() const {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const int P = a == 0 ? px : (a == 1 ? py : pz);
        T* dst = const_cast<T*>(bas[a]);
        for (int e = tid; e < P * P; e += bs) {
          const int i = e / P;
          dst[i * kPcLd + (e - i * P)] = fw[a][e];
        }
      }
    }
    for (int e = tid; e < 2 * planes * slab; e += bs) pl[e] = 0;
  }

  // LDS offset of element e of a round of planes (plane-major, rows of nz)
  __device__ __forceinline__ int place(int e) const {
    const int row = (int)__umulhi((unsigned)e, mz);
    const int p = (int)__umulhi((unsigned)row, my);
    return 2 * p * slab + (row - p * g.ny) * kPcLd + (e - row * g.nz);
  }
};

// One wave: 16 columns (tile c) of L^T X R for the LDS plane at X, rows by
// rows of 16 through epi(row tile, re, im).
template <typename T, bool FWD, class Epi>
__device__ __forceinline__ void pc_plane_tile(const PcCtx<T>& x, const T* X, int c, Epi& epi) {
  typedef typename Mma<T>::acc acc;
  acc tr[4], ti[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (r < x.ry) {
      acc cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
      const T* ar = X + (16 * r * kPcLd) + (x.li * kPcLd + x.lk);
      const T* ai = ar + x.slab;
#pragma unroll 1
      for (int k0 = 0; k0 < x.pz; k0 += 16) {
#pragma unroll
        for (int u = 0; u < 16; u += 4) {
          const T b = x.template basis<FWD, 2>(k0 + u, 1, 16 * c);
          cr = Mma<T>::step(ar[k0 + u], b, cr);
          ci = Mma<T>::step(ai[k0 + u], b, ci);
        }
      }
      tr[r] = cr;
      ti[r] = ci;
    }
  }
#pragma unroll 1
  for (int ro = 0; ro < x.ry; ++ro) {
    epi.load(ro);
    acc cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
      if (rb < x.ry) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const T a = x.template basis<FWD, 1>(16 * rb + x.kV * v, x.kL, 16 * ro);
          cr = Mma<T>::step(a, tr[rb][v], cr);
          ci = Mma<T>::step(a, ti[rb][v], ci);
        }
      }
    }
    epi.store(ro, cr, ci);
  }
}

// Where the accumulators of column tile c of grid plane i lie: element
// row(ro, v) * nz from the uniform base plus the lane's offset.
template <typename T>
struct PcOut {
  const PcCtx<T>& x;
  unsigned base;                   // of the plane and column tile
  unsigned lane;
  bool in;                         // column inside the grid
  __device__ __forceinline__ PcOut(const PcCtx<T>& x_, int i, int c)
      : x(x_), base((unsigned)i * x_.plane + 16 * c), lane(x_.kL * x_.lk * x_.g.nz + x_.li), in(16 * c + x_.li < x_.g.nz) {}
  __device__ __forceinline__ unsigned row(int ro, int v) const { return base + (16 * ro + x.kV * v) * x.g.nz; }
  __device__ __forceinline__ bool ok(int ro, int v) const {
    return in && 16 * ro + x.kV * v + x.kL * x.lk < x.g.ny;
  }
};

template <typename T>
struct EpiMode {                   // the half-transformed plane
  PcOut<T> o;
  typename V2<T>::t* t;
  __device__ __forceinline__ void load(int) {}
  __device__ __forceinline__ void store(int ro, const typename Mma<T>::acc& re, const typename Mma<T>::acc& im) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (o.ok(ro, v)) {
        typename V2<T>::t z;
        z.x = re[v];
        z.y = im[v];
        at32(t + o.row(ro, v), o.lane) = z;
      }
    }
  }
};

// Vectors and scalars of the inverse pass.
template <typename T>
struct PcUpdate {
  const typename V2<T>::t* r;
  typename V2<T>::t* p;
  typename V2<T>::t* q;
  typename V2<T>::t* d;            // solution or FP32 correction: d += alpha p (pend)
  const T* v;
  T shift;                         // eps_n + Re sigma
  T br, bi;                        // beta (first: unused)
  T ar, ai;                        // alpha of the last iteration (pend)
  bool first, pend, dfresh;        // dfresh: d holds nothing yet
  bool refresh;                    // q = M p + (V - shift) p only
};

template <typename T>
struct EpiUpdate {
  typedef typename V2<T>::t T2;
  PcOut<T> o;
  const PcUpdate<T>& u;
  double& mu_re;
  double& mu_im;
  T2 rv[4], pv[4], qv[4], dv[4];
  T vv[4];
  // loads at rows and columns outside the grid read the plane's first element
  __device__ __forceinline__ void load(int ro) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const bool k = o.ok(ro, v);
      const unsigned row = k ? o.row(ro, v) + o.lane : 0u;
      vv[v] = at32(u.v, row);
      if (!u.first) pv[v] = at32(u.p, row);
      if (!u.refresh) {
        rv[v] = at32(u.r, row);
        if (!u.first) qv[v] = at32(u.q, row);
        if (u.pend && !u.dfresh) dv[v] = at32(u.d, row);
      }
    }
  }
  __device__ __forceinline__ void store(int ro, const typename Mma<T>::acc& re, const typename Mma<T>::acc& im) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (!o.ok(ro, v)) continue;
      const unsigned i = o.row(ro, v) + o.lane;
      const T f = vv[v] - u.shift;
      T2 pn, qn;
      if (u.refresh) {
        qn.x = re[v] + f * pv[v].x;
        qn.y = im[v] + f * pv[v].y;
        at32(u.q, i) = qn;
        continue;
      }
      pn.x = re[v];
      pn.y = im[v];
      qn.x = rv[v].x + f * re[v];
      qn.y = rv[v].y + f * im[v];
      if (u.pend) {
        const T dx = u.ar * pv[v].x - u.ai * pv[v].y;
        const T dy = u.ar * pv[v].y + u.ai * pv[v].x;
        T2 dn;
        dn.x = u.dfresh ? dx : dv[v].x + dx;
        dn.y = u.dfresh ? dy : dv[v].y + dy;
        at32(u.d, i) = dn;
      }
      if (!u.first) {
        pn.x += u.br * pv[v].x - u.bi * pv[v].y;
        pn.y += u.br * pv[v].y + u.bi * pv[v].x;
        qn.x += u.br * qv[v].x - u.bi * qv[v].y;
        qn.y += u.br * qv[v].y + u.bi * qv[v].x;
      }
      at32(u.p, i) = pn;
      at32(u.q, i) = qn;
      mu_re += (double)(pn.x * qn.x - pn.y * qn.y);
      mu_im += (double)(pn.x * qn.y + pn.y * qn.x);
    }
  }
};

// Forward pass: with upd, r -= alpha (q + V_nl p) first, and rr += ||r||^2.
// nlp(i, q) adds the nonlocal term of element i.
template <typename T, class Nl>
__device__ __forceinline__ void pc_forward(const PcCtx<T>& x, typename V2<T>::t* r, const typename V2<T>::t* q,
                                           typename V2<T>::t* t, bool upd, T ar, T ai, const Nl& nlp, double& rr) {
  typedef typename V2<T>::t T2;
  constexpr int E = pc_elems<T>();
  T2 rv[E], qv[E];
  auto load = [&](int i0) {
    const int cnt = min(x.planes, x.g.nx - i0) * x.plane;
    const T2* rs = r + i0 * x.plane;
    const T2* qs = q + i0 * x.plane;
#pragma unroll
    for (int k = 0; k < E; ++k) {
      if (k * x.bs + x.tid < cnt) {
        rv[k] = at32(rs + k * x.bs, x.tid);
        if (upd) qv[k] = at32(qs + k * x.bs, x.tid);
      }
    }
  };
  load(0);
#pragma unroll 1
  for (int i0 = 0; i0 < x.g.nx; i0 += x.planes) {
    const int np = min(x.planes, x.g.nx - i0), cnt = np * x.plane;
    T2* rs = r + i0 * x.plane;
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int e = k * x.bs + x.tid;
      if (e < cnt) {
        T2 a = rv[k];
        if (upd) {
          T2 b = qv[k];
          nlp(i0 * x.plane + e, b);
          a.x -= ar * b.x - ai * b.y;
          a.y -= ar * b.y + ai * b.x;
          at32(rs + k * x.bs, x.tid) = a;
          rr += (double)a.x * (double)a.x + (double)a.y * (double)a.y;
        }
        const int at = x.place(e);
        x.pl[at] = a.x;
        x.pl[at + x.slab] = a.y;
      }
    }
    __syncthreads();
    if (i0 + x.planes < x.g.nx) load(i0 + x.planes);
#pragma unroll 1
    for (int job = x.wave; job < np * x.ct; job += x.nw) {
      const int p = job / x.ct, c = job - p * x.ct;
      EpiMode<T> epi{PcOut<T>(x, i0 + p, c), t};
      pc_plane_tile<T, true>(x, x.pl + 2 * p * x.slab, c, epi);
    }
    __syncthreads();
  }
}

// Inverse pass.
template <typename T>
__device__ __forceinline__ void pc_inverse(const PcCtx<T>& x, const typename V2<T>::t* t, const PcUpdate<T>& u,
                                           double& mu_re, double& mu_im) {
  typedef typename V2<T>::t T2;
  constexpr int E = pc_elems<T>();
  T2 tv[E];
  auto load = [&](int i0) {
    const int cnt = min(x.planes, x.g.nx - i0) * x.plane;
    const T2* ts = t + i0 * x.plane;
#pragma unroll
    for (int k = 0; k < E; ++k)
      if (k * x.bs + x.tid < cnt) tv[k] = at32(ts + k * x.bs, x.tid);
  };
  load(0);
#pragma unroll 1
  for (int i0 = 0; i0 < x.g.nx; i0 += x.planes) {
    const int np = min(x.planes, x.g.nx - i0), cnt = np * x.plane;
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int e = k * x.bs + x.tid;
      if (e < cnt) {
        const int at = x.place(e);
        x.pl[at] = tv[k].x;
        x.pl[at + x.slab] = tv[k].y;
      }
    }
    __syncthreads();
    if (i0 + x.planes < x.g.nx) load(i0 + x.planes);
#pragma unroll 1
    for (int job = x.wave; job < np * x.ct; job += x.nw) {
      const int p = job / x.ct, c = job - p * x.ct;
      EpiUpdate<T> epi{PcOut<T>(x, i0 + p, c), u, mu_re, mu_im, {}, {}, {}, {}, {}};
      pc_plane_tile<T, false>(x, x.pl + 2 * p * x.slab, c, epi);
    }
    __syncthreads();
  }
}

// Modes pass, in place on t: x forward, times 1 / (kin + sigma) (mul: times
// kin + sigma), x inverse; adds r^T M^-1 r = sum over modes of c s c (the
// basis is real orthogonal) to rho.  Each wave takes 16 columns at a time.
template <typename T>
__device__ __forceinline__ void pc_modes(const PcCtx<T>& x, const PrecArgs& pa, typename V2<T>::t* t, T sr, T si,
                                         bool mul, double& rho_re, double& rho_im) {
  typedef typename V2<T>::t T2;
  typedef typename Mma<T>::acc acc;
  constexpr bool PREFETCH = sizeof(T) == 4;    // the FP64 form has no registers for it
  const int nx = x.g.nx;
  const T* kx = prec_pick<T>(pa.k32[0], pa.k64[0]);
  const T* ky = prec_pick<T>(pa.k32[1], pa.k64[1]);
  const T* kz = prec_pick<T>(pa.k32[2], pa.k64[2]);
  T2 xv[16];
  const unsigned in_off = x.lk * x.plane + x.li, out_off = x.kL * x.lk * x.plane + x.li;
  auto load = [&](int task) {
    const bool in = 16 * task + x.li < x.plane;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (b < x.rx) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = 16 * b + 4 * u;
          T2 z;
          z.x = 0;
          z.y = 0;
          if (in && i + x.lk < nx) z = at32(t + (i * x.plane + 16 * task), in_off);
          xv[4 * b + u] = z;
        }
      }
    }
  };
  const int ntask = (x.plane + 15) >> 4;
  if (PREFETCH && x.wave < ntask) load(x.wave);
#pragma unroll 1
  for (int task = x.wave; task < ntask; task += x.nw) {
    if (!PREFETCH) load(task);
    const int c = 16 * task + x.li;
    const bool in = c < x.plane;
    const int b = in ? (int)__umulhi((unsigned)c, x.mz) : 0;
    const T kyz = (in ? ky[b] + kz[c - b * x.g.nz] : T(0)) + sr;
    acc tr[4], ti[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      if (m < x.rx) {
        acc cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
          if (kb < x.rx) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const T a = x.template basis<true, 0>(16 * kb + 4 * u, 1, 16 * m);
              cr = Mma<T>::step(a, xv[4 * kb + u].x, cr);
              ci = Mma<T>::step(a, xv[4 * kb + u].y, ci);
            }
          }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const T s = kx[16 * m + x.kV * v + x.kL * x.lk] + kyz;    // kinetic eigenvalue + Re sigma
          const T re = cr[v], im = ci[v];
          T zr, zi;
          if (mul) {
            zr = re * s - im * si;
            zi = im * s + re * si;
          } else {
            const T den = s * s + si * si;
            zr = (re * s + im * si) / den;
            zi = (im * s - re * si) / den;
          }
          rho_re += (double)re * (double)zr - (double)im * (double)zi;
          rho_im += (double)re * (double)zi + (double)im * (double)zr;
          cr[v] = zr;
          ci[v] = zi;
        }
        tr[m] = cr;
        ti[m] = ci;
      }
    }
    if (PREFETCH && task + x.nw < ntask) load(task + x.nw);
#pragma unroll 1
    for (int ro = 0; ro < x.rx; ++ro) {
      acc cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        if (m < x.rx) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const T a = x.template basis<false, 0>(16 * m + x.kV * v, x.kL, 16 * ro);
            cr = Mma<T>::step(a, tr[m][v], cr);
            ci = Mma<T>::step(a, ti[m][v], ci);
          }
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 16 * ro + x.kV * v;
        if (in && i + x.kL * x.lk < nx) {
          T2 z;
          z.x = cr[v];
          z.y = ci[v];
          at32(t + (i * x.plane + 16 * task), out_off) = z;
        }
      }
    }
  }
}

}  // namespace
}  // namespace rpa
