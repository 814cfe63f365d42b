// A stand-in for the HIP runtime, for host tests of the library's bookkeeping
// without a GPU: allocations are host memory that is recorded, copies copy,
// and kernels are not run but checked against what they may assume.  The
// definitions here take the place of the runtime's for the whole process.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "internal.h"
#include "rpa.h"

namespace {

std::map<char*, size_t> g_mem;      // live device allocations
size_t g_bytes = 0;                 // their total
constexpr int kCus = 256;
int (*g_occupancy)(const void* fn) = nullptr;   // workgroups per compute unit (null: 2)

struct Launch {
  const void* fn;
  dim3 grid, block;
  size_t shmem;
  void** args;
};
void (*g_on_launch)(const Launch&) = nullptr;

}  // namespace

extern "C" {

hipError_t hipMalloc(void** p, size_t n) {
  *p = std::calloc(1, n);
  if (!*p) return hipErrorOutOfMemory;
  g_mem[static_cast<char*>(*p)] = n;
  g_bytes += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  auto it = g_mem.find(static_cast<char*>(p));
  if (it == g_mem.end()) std::abort();
  g_bytes -= it->second;
  g_mem.erase(it);
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::calloc(1, n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = kCus; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = nullptr; return hipErrorInvalidSymbol; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* fn, int, size_t) {
  *n = g_occupancy ? g_occupancy(fn) : 2;
  return hipSuccess;
}
struct { dim3 grid, block; size_t shmem; hipStream_t s; } g_call;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t s) {
  g_call = {grid, block, shmem, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* s) {
  *grid = g_call.grid;
  *block = g_call.block;
  *shmem = g_call.shmem;
  *s = g_call.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void** args, size_t shmem, hipStream_t) {
  if (g_on_launch) g_on_launch(Launch{fn, grid, block, shmem, args});
  return hipSuccess;
}

}  // extern "C"

namespace {

int fail(const std::string& what) {
  std::printf("FAIL %s\n", what.c_str());
  return 1;
}

// A problem on a grid of n points with n_occ orbitals (its arrays live as long as the process).
rpa_setup_params problem(int nx, int ny, int nz, int n_occ, rpa_precision precision, bool precond) {
  rpa_setup_params p;
  std::memset(&p, 0, sizeof(p));
  const int n[3] = {nx, ny, nz};
  for (int d = 0; d < 3; ++d) {
    p.n[d] = n[d];
    p.L[d] = 0.45 * n[d];
  }
  const size_t N = (size_t)nx * ny * nz;
  p.fd_radius = rpa::kRadius;
  p.n_occ = n_occ;
  p.v_loc = static_cast<double*>(std::calloc(N, sizeof(double)));
  p.psi = static_cast<double*>(std::calloc(N * n_occ, sizeof(double)));
  p.eps = static_cast<double*>(std::calloc(n_occ, sizeof(double)));
  p.precision = precision;
  p.stern_tol = 1e-8;
  p.stern_maxit = 100;
  p.precond = precond;
  return p;
}

// n_proj projectors of three points, every two of them on the same ones.
void add_projectors(rpa_setup_params& p, int n_proj) {
  const long long N = (long long)p.n[0] * p.n[1] * p.n[2];
  auto* ptr = new std::vector<int64_t>(n_proj + 1);
  auto* idx = new std::vector<int64_t>(3 * n_proj);
  auto* val = new std::vector<double>(3 * n_proj, 0.5);
  auto* gamma = new std::vector<double>(n_proj, 1.0);
  for (int q = 0; q <= n_proj; ++q) (*ptr)[q] = 3 * q;
  for (int e = 0; e < 3 * n_proj; ++e) (*idx)[e] = (5 * (e / 6) + e % 3) % N;
  p.n_proj = n_proj;
  p.proj_ptr = ptr->data();
  p.proj_idx = idx->data();
  p.proj_val = val->data();
  p.proj_gamma = gamma->data();
}

// --- slots: the workspaces of every Sternheimer launch lie inside their allocation

bool g_slots_ok = true;
int g_cocg = 0;
template <int V>
bool is_cocg(const void* fn) {
  for (int m = 0; m < 3; ++m)
    for (int r = 0; r < 2; ++r)
      for (rpa::CocgKernel k : {rpa::cocg_kernel<V, 56>(m, r), rpa::cocg_kernel<V, 64>(m, r), rpa::cocg_kernel<V, 128>(m, r)})
        if (fn == reinterpret_cast<const void*>(k)) return true;
  return false;
}
void check_slots(const Launch& l) {
  if (!is_cocg<0>(l.fn) && !is_cocg<2>(l.fn)) return;
  const rpa::CocgArgs& a = *static_cast<const rpa::CocgArgs*>(l.args[0]);
  auto it = g_mem.find(a.slot_ws);
  const size_t need = (size_t)l.grid.x * a.slot_bytes;
  ++g_cocg;
  std::printf("%u workgroups of %lld bytes in %zu\n", l.grid.x, a.slot_bytes, it == g_mem.end() ? 0 : it->second);
  if (it == g_mem.end() || need > it->second) g_slots_ok = false;
}

int slots(int nx, int ny, int nz, int n_occ, int nvec, int precision, int precond) {
  rpa_setup_params p = problem(nx, ny, nz, n_occ, (rpa_precision)precision, precond != 0);
  rpa_handle h = nullptr;
  if (rpa_setup(&p, nullptr, &h) != RPA_OK) return fail(rpa_last_error(nullptr));
  g_on_launch = check_slots;
  const size_t N = (size_t)nx * ny * nz;
  std::vector<double> u(nvec * N), x(2 * nvec * n_occ * N);
  if (rpa_sternheimer_solve(h, 0.5, nvec, u.data(), x.data(), nullptr, nullptr) != RPA_OK)
    return fail(rpa_last_error(nullptr));
  rpa_destroy(h);
  if (g_cocg != (precision == RPA_FP64 ? 1 : 2)) return fail("a launch was not seen");
  return g_slots_ok ? 0 : fail("workspaces end beyond their allocation");
}

// --- workspace: what a call allocates is what the serving admission counts for it

int workspace(int nx, int ny, int nz, int n_occ, int n_pts, int m, int precision, int window) {
  rpa_setup_params p = problem(nx, ny, nz, n_occ, (rpa_precision)precision, true);
  if (window) {
    p.precond_omega_min = 0.5;
    p.precond_omega_max = 20.0;
  }
  // the plain kernels run with two workgroups per compute unit, the preconditioned ones with one
  g_occupancy = [](const void* fn) { return is_cocg<0>(fn) ? 2 : 1; };
  rpa_handle h = nullptr;
  if (rpa_setup(&p, nullptr, &h) != RPA_OK) return fail(rpa_last_error(nullptr));
  const size_t resident = g_bytes;
  const double omega = 1.0;
  std::vector<int64_t> pts(n_pts);
  std::vector<double> d(n_pts);
  if (lanczos_energy_density(h, 1, &omega, n_pts, pts.data(), m, d.data(), nullptr, nullptr) != RPA_OK)
    return fail(rpa_last_error(nullptr));
  const size_t used = g_bytes - resident;
  const uint64_t counted = rpa::lanczos_workspace_bytes(p, n_pts, m, kCus, true);
  rpa_destroy(h);
  std::printf("allocated %zu counted %llu\n", used, (unsigned long long)counted);
  // the statistics' few counters are left to the admission's margin
  const size_t counters = 16 * 1024;
  return used <= counted + counters && counted <= used + counters ? 0 : fail("the count is not what is allocated");
}

// --- resident: the server counts what a worker's setup keeps, and its own copy

int resident(int nx, int ny, int nz, int n_occ, int precond, int n_proj) {
  rpa_setup_params p = problem(nx, ny, nz, n_occ, RPA_FP32_REFINE, precond != 0);
  add_projectors(p, n_proj);
  rpa_handle h = nullptr;
  if (rpa_setup(&p, nullptr, &h) != RPA_OK) return fail(rpa_last_error(nullptr));
  const size_t kept = g_bytes;
  rpa_destroy(h);
  rpa_server_params sp;
  std::memset(&sp, 0, sizeof(sp));
  sp.n_workers = 2;
  sp.fake_executor_us = 1;
  rpa_server s = nullptr;
  int32_t id = 0;
  uint64_t high = 0;
  if (rpa_server_create(&sp, &s) != RPA_OK || rpa_server_add_cell(s, &p, &id) != RPA_OK ||
      rpa_server_status(s, nullptr, nullptr, nullptr, &high) != RPA_OK)
    return fail("server");
  rpa_server_destroy(s);
  const uint64_t own = 8ULL * nx * ny * nz * (1 + n_occ);
  std::printf("kept %zu counted %llu\n", kept, (unsigned long long)((high - own) / 2));
  // a shared support is stored once and counted for each projector
  const uint64_t shared = n_proj > 0 ? 40ULL * n_proj : 0;
  return high >= own + 2 * kept && high <= own + 2 * (kept + shared) ? 0 : fail("the count is not what is kept");
}

// --- expand: launches within the grid limit that together cover every start
// vector and point once

struct ExpandLaunch {
  long long b0, bn, c0, threads, groups;
};
std::vector<ExpandLaunch> g_expand;
long long g_expand_vec = 0;          // elements of a start vector's G

int expand(long long N, int n_occ, int ng, int B) {
  g_expand_vec = (long long)ng * n_occ;
  g_on_launch = [](const Launch& l) {
    // psi, G, B, n_occ, ng, N, first chunk, x
    const double2* G = *static_cast<const double2**>(l.args[1]);
    g_expand.push_back({(long long)(reinterpret_cast<uintptr_t>(G) / sizeof(double2)) / g_expand_vec,
                        *static_cast<int*>(l.args[2]), *static_cast<long long*>(l.args[6]),
                        (long long)l.grid.x * l.block.x, l.grid.x});
  };
  if (rpa::launch_expand(nullptr, nullptr, B, n_occ, ng, N, nullptr, nullptr) != hipSuccess) return fail("launch");
  const long long tn = n_occ <= 16 ? 1 : 2, ntn = (n_occ + 16 * tn - 1) / (16 * tn), chunks = (N + 63) / 64;
  long long b = 0, c = 0;            // next start vector, next chunk of its range
  for (const ExpandLaunch& l : g_expand) {
    if (l.threads >= 1LL << 32) return fail("grid of " + std::to_string(l.threads) + " threads");
    if (l.b0 != b || l.c0 != c) return fail("gap");
    // workgroups are dealt to the eight XCDs by chunk, four tiles each
    const long long per_chunk = (l.bn * ntn + 3) / 4;
    if (l.groups % (8 * per_chunk)) return fail("grid");
    c += l.groups / per_chunk;
    if (c >= chunks) {
      if (c >= chunks + 8) return fail("overrun");
      c = 0;
      b += l.bn;
    }
  }
  std::printf("%zu launches\n", g_expand.size());
  return b == B && c == 0 ? 0 : fail("not all covered");
}

// --- lds: the most projectors that setup accepts, and the largest dynamic LDS of
// the Sternheimer launches then

size_t g_lds = 0;

int lds(int nx, int ny, int nz, int precision, int precond, int window) {
  rpa_setup_params p = problem(nx, ny, nz, 2, (rpa_precision)precision, precond != 0);
  if (window) p.precond_omega_min = 1.0;
  g_on_launch = [](const Launch& l) {
    if (is_cocg<1>(l.fn) || is_cocg<3>(l.fn)) g_lds = l.shmem > g_lds ? l.shmem : g_lds;
  };
  rpa_handle h = nullptr;
  int n = rpa::kMaxProj;
  for (; n > 0; --n) {
    add_projectors(p, n);
    if (rpa_setup(&p, nullptr, &h) == RPA_OK) break;
  }
  if (n == 0) return fail(rpa_last_error(nullptr));
  const size_t N = (size_t)nx * ny * nz;
  std::vector<double> u(9 * N), x(36 * N);
  if (rpa_sternheimer_solve(h, 0.5, 9, u.data(), x.data(), nullptr, nullptr) != RPA_OK)
    return fail(rpa_last_error(nullptr));
  rpa_destroy(h);
  std::printf("projectors %d lds %zu\n", n, g_lds);
  return g_lds > 0 ? 0 : fail("no launch seen");
}

// --- stencil: the plain operator's launch of a handle

int stencil(int nx, int ny, int nz, int precision, int precond, int nvec) {
  rpa_setup_params p = problem(nx, ny, nz, 2, RPA_FP32_REFINE, precond != 0);
  rpa_handle h = nullptr;
  if (rpa_setup(&p, nullptr, &h) != RPA_OK) return fail(rpa_last_error(nullptr));
  g_on_launch = [](const Launch& l) {
    std::printf("grid %u %u %u block %u lds %zu\n", l.grid.x, l.grid.y, l.grid.z, l.block.x, l.shmem);
  };
  const std::vector<double> zero(nvec, 0.0);
  double x = 0.0, y = 0.0;           // the kernel does not run
  if (rpa_hamiltonian_apply(h, nvec, zero.data(), zero.data(), &x, &y, precision, nullptr) != RPA_OK)
    return fail(rpa_last_error(nullptr));
  rpa_destroy(h);
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  std::vector<int> v;
  for (int i = 2; i < argc; ++i) v.push_back(std::atoi(argv[i]));
  int r = 2;
  if (what == "slots" && v.size() == 7) r = slots(v[0], v[1], v[2], v[3], v[4], v[5], v[6]);
  if (what == "workspace" && v.size() == 8) r = workspace(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]);
  if (what == "resident" && v.size() == 6) r = resident(v[0], v[1], v[2], v[3], v[4], v[5]);
  if (what == "expand" && v.size() == 4) r = expand(std::atoll(argv[2]), v[1], v[2], v[3]);
  if (what == "lds" && v.size() == 6) r = lds(v[0], v[1], v[2], v[3], v[4], v[5]);
  if (what == "stencil" && v.size() == 6) r = stencil(v[0], v[1], v[2], v[3], v[4], v[5]);
  if (r == 0) std::printf("ok\n");
  return r;
}
