// Checks of libace's host logic without a GPU: the library's objects (host code
// under AddressSanitizer and UndefinedBehaviorSanitizer) are linked with the
// stand-in for the HIP runtime below, which hands out addresses of a "device"
// of a chosen size and shows every kernel launch to the check instead of
// running it.  So the reads and writes that a launch's arguments imply can be
// compared with the buffers, and allocations can be made to fail.
//
// Exit status: 0 when every check held, 1 otherwise.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <memory>
#include <string>
#include <vector>

#include "../../paper_1601_07159_amd/csrc/pass_bodies.h"

using ace::real_tri_units;

// ---------------------------------------------------------------- HIP runtime
namespace {

struct Device {
  size_t free_bytes = (size_t)1 << 40;
  std::map<char*, size_t> live;  // allocations
  char* next = (char*)0x100000000000;
  int mallocs = 0, refused = 0;
  bool capturing = false;
} dev;

struct Launch {
  std::string name;
  dim3 grid, block;
  void** args;
  template <typename T>
  T arg(int k) const {
    return *(T*)args[k];
  }
  bool is(const char* kernel) const { return name.find(kernel) != std::string::npos; }
};
std::function<void(const Launch&)> on_launch;

std::map<const void*, std::string>& kernel_names() {
  static std::map<const void*, std::string> m;
  return m;
}
struct {
  dim3 grid, block;
  size_t shmem;
  hipStream_t stream;
} call;

}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
  kernel_names()[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t stream) {
  call = {grid, block, shmem, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* stream) {
  *grid = call.grid;
  *block = call.block;
  *shmem = call.shmem;
  *stream = call.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
  if (on_launch) on_launch({kernel_names()[f], grid, block, args});
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  ++dev.mallocs;
  if (n > dev.free_bytes) {
    ++dev.refused;
    *p = nullptr;
    return hipErrorOutOfMemory;
  }
  dev.free_bytes -= n;
  *p = dev.next;
  dev.live[dev.next] = n;
  dev.next += (n + 0x1ffff) / 0x10000 * 0x10000;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  const auto it = dev.live.find((char*)p);
  if (it == dev.live.end()) return hipErrorInvalidValue;
  dev.free_bytes += it->second;
  dev.live.erase(it);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) {
  *f = dev.free_bytes;
  *t = (size_t)1 << 40;
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = dev.capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = (void*)0x200000000000;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t)1;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  dev.capturing = true;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  dev.capturing = false;
  *g = (hipGraph_t)1;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)1;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = (hipEvent_t)1;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.f;
  return hipSuccess;
}
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void*, size_t n, hipMemcpyKind k, hipStream_t) {
  if (k == hipMemcpyDeviceToHost) std::memset(d, 0, n);
  return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind,
                            hipStream_t) {
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 1;
  return hipSuccess;
}
}  // extern "C"

// --------------------------------------------------------------------- checks
namespace {

int g_checks = 0, g_failures = 0;
std::string g_case;

void expect(bool ok, const char* what, int line) {
  ++g_checks;
  if (!ok) {
    ++g_failures;
    std::printf("FAIL line %d: %s [%s]\n", line, what, g_case.c_str());
  }
}
#define EXPECT(cond) expect((cond), #cond, __LINE__)

ace_grid cubic(int n) {
  ace_grid g{};
  for (int a = 0; a < 3; ++a) {
    g.n[a] = n;
    g.L[a] = 0.43 * n;
  }
  g.kind = ACE_COULOMB;
  return g;
}

// Caller's arrays, far apart.
char* array_at(int k) { return (char*)0x400000000000 + (size_t)k * 0x10000000000; }

size_t cx_bytes(ace_prec p) { return p == ACE_FP64 || p == ACE_REAL64 ? 16 : 8; }

// Every value that the slab pass on split lines reads lies in the transposed
// copies, which lie in the workspace.
void slab_reads(ace_ctx c, size_t eb, int n, int* slabs) {
  const long ng = (long)n * n * n;
  auto copied = std::make_shared<std::vector<std::pair<char*, char*>>>();
  on_launch = [=](const Launch& l) {
    const char* end = (const char*)c->ws + c->ws_bytes;
    if (l.is("k_orbital_transpose")) {
      char* y = l.arg<char*>(2);
      const size_t bytes = (size_t)l.grid.x / n * ng * eb;
      EXPECT(y >= (char*)c->ws && y + bytes <= end);
      copied->push_back({y, y + bytes});
    }
    if (!l.is("k_slab_split")) return;
    ++*slabs;
    const char* phi = l.arg<const char*>(0);
    const char* psi = l.arg<const char*>(1);
    const char* buf = l.arg<const char*>(2);
    const int mode = l.arg<int>(3), i0 = l.arg<int>(4), A = l.arg<int>(5), j0 = l.arg<int>(6);
    const long p0 = l.arg<long>(7);
    const int np = l.arg<int>(8);
    EXPECT(buf + (size_t)np * ng * eb <= end);
    long imax = 0, jmax = 0, j = 0;
    for (long p = 0; p < np; ++p) {
      long i = i0 + p % A, jj = j0 + p / A;
      const long tri = (long)A * (A + 1) / 2;
      if (mode == 1 || (mode == 3 && p < tri)) {
        const long q = p + p0;
        while ((j + 1) * (j + 2) / 2 <= q) ++j;
        i = i0 + q - j * (j + 1) / 2;
        jj = (mode == 1 ? j0 : i0) + j;
      } else if (mode == 3) {
        i = (p - tri) % A;
        jj = j0 + (p - tri) / A;
      }
      imax = std::max(imax, i);
      jmax = std::max(jmax, jj);
    }
    bool phi_in = false, psi_in = false;
    for (const auto& r : *copied) {
      phi_in |= phi >= r.first && phi + (size_t)(imax + 1) * ng * eb <= r.second;
      psi_in |= psi >= r.first && psi + (size_t)(jmax + 1) * ng * eb <= r.second;
    }
    EXPECT(phi_in);
    EXPECT(psi_in);
  };
}

// W = V_X[phi] psi with phi and psi one array (any n_band against n_occ).
void shared_orbitals_on_split_lines() {
  for (int n : {40, 72})
    for (ace_prec prec : {ACE_FP64, ACE_FP32})
      for (auto [nocc, nband] : {std::pair{20, 10}, {20, 19}, {20, 20}, {20, 24}, {33, 12}})
        for (long symmetry : {0L, 1L})
          for (long budget : {0L, 3L, 37L}) {
            const ace_grid g = cubic(n);
            const long ng = (long)n * n * n;
            g_case = "n " + std::to_string(n) + " prec " + std::to_string(prec) + " nocc " +
                     std::to_string(nocc) + " nband " + std::to_string(nband) + " symmetry " +
                     std::to_string(symmetry) + " budget " + std::to_string(budget);
            ace_ctx c = nullptr;
            EXPECT(ace_create(&c, nullptr, nullptr) == ACE_OK);
            ace_set_tuning(c, ACE_TUNE_SYMMETRY, symmetry);
            ace_set_pair_budget(c, budget * ng * (long)cx_bytes(prec));
            int slabs = 0;
            slab_reads(c, cx_bytes(prec), n, &slabs);
            EXPECT(ace_build_W(c, &g, prec, array_at(0), nocc, ng, array_at(0), nband, ng,
                               array_at(1), ng, 1.0) == ACE_OK);
            EXPECT(slabs > 0 || (prec == ACE_FP32 && n < 72));
            on_launch = nullptr;
            ace_destroy(c);
          }
}

// Every spectrum that the accumulate pass reads was written by the slab pass
// before it, and it writes the bands of W only.
void spectra_reads(int nband, int* accums) {
  auto pairs = std::make_shared<long>(0);
  on_launch = [=](const Launch& l) {
    if (l.is("k_slab_split")) *pairs = l.arg<int>(8);
    if (l.is("k_pair_fwd_slab")) *pairs = l.arg<int>(10);
    if (l.is("k_pair_fwd_real")) *pairs = l.arg<int>(9);
    if (!l.is("k_pencil_accum")) return;
    ++*accums;
    long read = 0;  // one past the last pair
    if (l.is("k_pencil_accum_real_sym")) {
      const long A = l.arg<int>(5), extra = l.arg<int>(6) - (A + 1) / 2;
      read = real_tri_units((int)A) + (A + 1) / 2 * extra;
      EXPECT(extra >= 0 && A + extra <= nband);
    } else if (l.is("k_pencil_accum_real")) {
      read = (long)l.arg<int>(7) * l.arg<int>(9);
      EXPECT(l.arg<int>(8) + l.arg<int>(9) <= nband);
    } else {
      const long A = l.arg<int>(6), nbc = l.arg<int>(8);
      const int mode = l.arg<int>(10);
      const long tri = A * (A + 1) / 2;
      read = mode == 1 ? tri : mode == 3 ? tri + A * std::max(0L, nbc - A) : A * nbc;
      EXPECT(l.arg<int>(7) + nbc <= nband);
    }
    EXPECT(read <= *pairs);
  };
}

// One array for phi and psi, fewer bands than orbitals, with pair symmetry.
void fewer_bands_than_orbitals() {
  for (int n : {16, 48})
    for (ace_prec prec : {ACE_FP64, ACE_FP32, ACE_REAL64, ACE_REAL32})
      for (auto [nocc, nband] : {std::pair{2, 1}, {17, 16}, {17, 2}, {20, 10}, {9, 9}, {9, 12}})
        for (long budget : {0L, 2L, 5L, 60L}) {
          const ace_grid g = cubic(n);
          const long ng = (long)n * n * n;
          g_case = "n " + std::to_string(n) + " prec " + std::to_string(prec) + " nocc " +
                   std::to_string(nocc) + " nband " + std::to_string(nband) + " budget " +
                   std::to_string(budget);
          ace_ctx c = nullptr;
          EXPECT(ace_create(&c, nullptr, nullptr) == ACE_OK);
          ace_set_pair_budget(c, budget * ng * (long)cx_bytes(prec));
          int accums = 0;
          spectra_reads(nband, &accums);
          EXPECT(ace_build_W(c, &g, prec, array_at(0), nocc, ng, array_at(0), nband, ng,
                             array_at(1), ng, 1.0) == ACE_OK);
          if (prec == ACE_FP64 || prec == ACE_FP32)
            EXPECT(ace_apply_h(c, &g, prec, nullptr, nullptr, 0, 0, array_at(0), nocc, ng, 1.0,
                               array_at(0), nband, ng, array_at(1), ng) == ACE_OK);
          EXPECT(accums > 0);
          on_launch = nullptr;
          ace_destroy(c);
        }
}

// The optional copies of the split-line passes: what a call does where memory,
// a capture or a captured graph leaves no room for them.
void optional_copies() {
  const int n = 48, nocc = 20, nband = 24;
  const ace_grid g = cubic(n);
  const long ng = (long)n * n * n;
  const size_t everything = dev.free_bytes;
  int copies = 0;
  const auto build = [&](ace_ctx c, int bands) {
    copies = 0;
    on_launch = [&](const Launch& l) { copies += l.is("k_orbital_transpose"); };
    const ace_status st = ace_build_W(c, &g, ACE_FP64, array_at(0), nocc, ng, array_at(0), bands,
                                      ng, array_at(1), ng, 1.0);
    on_launch = nullptr;
    return st;
  };
  const auto fresh = [&](bool sized) {
    ace_ctx c = nullptr;
    EXPECT(ace_create(&c, nullptr, nullptr) == ACE_OK);
    if (sized) {  // a workspace for the build without copies
      ace_set_tuning(c, ACE_TUNE_FFT_SHAPE, 4);
      EXPECT(build(c, nband) == ACE_OK && copies == 0);
      ace_set_tuning(c, ACE_TUNE_FFT_SHAPE, 0);
    }
    return c;
  };
  {
    g_case = "memory for the workspace, none for copies";
    ace_ctx c = fresh(true);
    void* ws = c->ws;
    dev.free_bytes = 1 << 20;
    dev.mallocs = 0;
    EXPECT(build(c, nband) == ACE_OK && copies == 0);
    EXPECT(c->ws == ws && dev.live.count((char*)ws) == 1);
    EXPECT(dev.mallocs == 1);
    EXPECT(std::strlen(ace_last_error(c)) == 0);
    EXPECT(build(c, nband) == ACE_OK && dev.mallocs == 1);  // not asked for again
    double* e = (double*)array_at(2);
    EXPECT(ace_exchange_energy(c, &g, ACE_FP64, array_at(0), nocc, ng, nullptr, 0, 0, e) == ACE_OK);
    EXPECT(c->ws == ws && std::strlen(ace_last_error(c)) == 0);
    dev.free_bytes = everything;
    EXPECT(ace_reserve(c, &g, ACE_FP64, nocc, nband, 1) == ACE_OK);
    EXPECT(build(c, nband) == ACE_OK && copies == 1);
    ace_destroy(c);
  }
  {
    g_case = "the first call, memory for the workspace alone";
    ace_ctx c = fresh(true);
    const size_t bytes = c->ws_bytes;
    ace_destroy(c);
    EXPECT(dev.live.empty());
    dev.free_bytes = bytes;
    c = fresh(false);
    EXPECT(build(c, nband) == ACE_OK && copies == 0);
    EXPECT(c->ws_bytes == bytes && std::strlen(ace_last_error(c)) == 0);
    ace_destroy(c);
    dev.free_bytes = everything;
  }
  {
    g_case = "under capture, and after it";
    ace_ctx c = fresh(true);
    void* ws = c->ws;
    dev.capturing = true;
    EXPECT(build(c, nband) == ACE_OK && copies == 0);
    EXPECT(std::strlen(ace_last_error(c)) == 0);
    dev.capturing = false;
    EXPECT(build(c, nband) == ACE_OK && c->ws == ws);  // the graph holds its address
    ace_destroy(c);
  }
  {
    g_case = "room: the copies are used, the old buffer goes";
    ace_ctx c = fresh(true);
    EXPECT(build(c, nband) == ACE_OK && copies == 1);
    EXPECT(dev.live.size() == 1 && dev.live.count((char*)c->ws) == 1);
    ace_destroy(c);
  }
  {
    g_case = "a reservation, memory for all but the copies";
    ace_ctx c = fresh(false);
    EXPECT(ace_reserve(c, &g, ACE_FP64, nocc, nband, nband) == ACE_OK);
    const size_t all = c->ws_bytes;
    ace_destroy(c);
    c = fresh(false);
    dev.free_bytes = all - 1;
    EXPECT(ace_reserve(c, &g, ACE_FP64, nocc, nband, nband) == ACE_OK);
    EXPECT(c->ws_bytes < all && std::strlen(ace_last_error(c)) == 0);
    dev.mallocs = 0;
    EXPECT(build(c, nband) == ACE_OK && dev.mallocs == 0);
    ace_destroy(c);
    dev.free_bytes = everything;
  }
  {
    g_case = "a batch, memory for all but the copies";
    std::vector<ace_instance> inst(3);
    for (int k = 0; k < 3; ++k) {
      inst[k] = ace_instance{g, ACE_FP64, array_at(4 * k), nocc, ng, array_at(4 * k), nband, ng,
                             array_at(4 * k + 1), ng, array_at(4 * k + 2), ng,
                             (int*)array_at(4 * k + 3), 1.0};
    }
    ace_ctx c = fresh(false);
    EXPECT(ace_build_W_batched(c, 3, inst.data()) == ACE_OK);
    const size_t all = c->ws_bytes;
    ace_destroy(c);
    c = fresh(false);
    dev.free_bytes = all - 1;
    EXPECT(ace_build_W_batched(c, 3, inst.data()) == ACE_OK);
    EXPECT(c->ws_bytes < all && std::strlen(ace_last_error(c)) == 0);
    dev.mallocs = 0;
    EXPECT(ace_build_W_batched(c, 3, inst.data()) == ACE_OK && dev.mallocs == 0);
    ace_destroy(c);
    dev.free_bytes = everything;
  }
  EXPECT(dev.live.empty() && dev.free_bytes == everything);
}

// Direct energies of few pairs per orbital take no transposed copies.
void copies_by_pairs() {
  struct Case {
    int n;
    ace_prec prec;
    int nocc;
    bool copies;
  };
  for (const Case& k : {Case{48, ACE_FP64, 7, true}, Case{48, ACE_FP64, 6, false},
                        Case{64, ACE_FP64, 10, false}, Case{64, ACE_FP64, 11, true},
                        Case{72, ACE_FP64, 8, false}, Case{72, ACE_FP64, 11, true},
                        Case{72, ACE_FP32, 6, false}, Case{72, ACE_FP32, 7, true}}) {
    g_case = "copies " + std::to_string(k.n) + "^3, precision " + std::to_string(k.prec) + ", " +
             std::to_string(k.nocc) + " orbitals";
    ace_ctx c = nullptr;
    EXPECT(ace_create(&c, nullptr, nullptr) == ACE_OK);
    const ace_grid g = cubic(k.n);
    int copies = 0;
    on_launch = [&](const Launch& l) { copies += l.is("k_orbital_transpose"); };
    EXPECT(ace_exchange_energy(c, &g, k.prec, array_at(0), k.nocc, (long)k.n * k.n * k.n, nullptr, 0,
                               0, (double*)array_at(1)) == ACE_OK);
    on_launch = nullptr;
    EXPECT((copies > 0) == k.copies);
    ace_destroy(c);
  }
}

// The kernels of one V_ACE apply (reduction, expansion) in FP64.
struct Route {
  ace_prec prec;
  int n, nb, nx;
  const char *reduction, *expansion;
};
void apply_routes(std::initializer_list<Route> routes) {
  for (const Route& r : routes) {
    g_case = "apply " + std::to_string(r.nb) + " x " + std::to_string(r.nx) + " at " +
             std::to_string(r.n) + "^3, precision " + std::to_string(r.prec);
    ace_ctx c = nullptr;
    EXPECT(ace_create(&c, nullptr, nullptr) == ACE_OK);
    const ace_grid g = cubic(r.n);
    const long ng = (long)r.n * r.n * r.n;
    std::vector<std::string> names;
    on_launch = [&](const Launch& l) { names.push_back(l.name); };
    EXPECT(ace_apply(c, &g, r.prec, array_at(0), r.nb, ng, array_at(1), r.nx, ng, array_at(2), ng) ==
           ACE_OK);
    on_launch = nullptr;
    EXPECT(names.size() == 3 && names[0].find(r.reduction) != std::string::npos &&
           names[2].find(r.expansion) != std::string::npos);
    ace_destroy(c);
  }
}

// Expansions by slices of C where they gain: not for few grid points in FP64
// with four real products.
void expansion_routes() {
  apply_routes({{ACE_FP64, 16, 80, 48, "k_cn", "k_nn_slices"},
                {ACE_FP64, 16, 81, 48, "k_cn", "k_nn_mfma"},
                {ACE_FP64, 16, 256, 256, "k_cn", "k_nn_mfma"},
                {ACE_FP64, 24, 81, 48, "k_cn", "k_nn_slices"},
                {ACE_REAL64, 16, 256, 256, "k_cn", "k_nn_slices"},
                {ACE_FP32, 16, 256, 256, "k_cn", "k_nn_slices"}});
}

// A reduction product fits the scratch that is stated for it, in every mode.
template <typename T>
void reduction_scratch() {
  using namespace ace;
  for (CnMode mode : {kNative, kBf16Split, kFp64, kFp64Tiles, kFp32Chunks})
    for (long K : {512L, 13824L, 262144L})
      for (int na : {1, 31, 48, 64, 81, 136, 161, 257, 600})
        for (int nb : {1, 33, 64, 136, 257})
          for (bool herm : {false, true}) {
            if (sizeof(T) == 8 && mode == kBf16Split) continue;
            const int n2 = herm ? na : nb;
            g_case = "mode " + std::to_string(mode) + " K " + std::to_string(K) + " " +
                     std::to_string(na) + " x " + std::to_string(n2);
            ace_ctx c = nullptr;
            EXPECT(ace_create(&c, nullptr, nullptr) == ACE_OK);
            const cx<T>* A = (const cx<T>*)array_at(0);
            const cx<T>* B = (const cx<T>*)array_at(1);
            for (const cx<T>* second : {A, B}) {
              const size_t part = gemm_cn_partial_bytes(na, n2, K, sizeof(cx<T>), mode, herm);
              EXPECT(part <= gemm_cn_scratch_bytes(na, n2, K));
              EXPECT(ws_begin(c, part) == ACE_OK);
              EXPECT(gemm_cn<T>(c, A, K, na, second, K, n2, K, 1.0, (cx<double>*)array_at(2), na,
                                mode, false, herm) == ACE_OK);
              EXPECT(c->ws_used <= align_up(part, 256));
            }
            ace_destroy(c);
          }
}

}  // namespace

int main() {
  setvbuf(stdout, nullptr, _IOLBF, 0);
  shared_orbitals_on_split_lines();
  fewer_bands_than_orbitals();
  optional_copies();
  copies_by_pairs();
  expansion_routes();
  reduction_scratch<float>();
  reduction_scratch<double>();
  std::printf("plan checks: %d checks, %d failures\n", g_checks, g_failures);
  return g_failures ? 1 : 0;
}
