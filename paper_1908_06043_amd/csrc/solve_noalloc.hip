// sislice_ldlt_solve_noalloc: the shift-invert solve of sislice_ldlt_solve for
// callers that cannot allocate (code under graph capture, tight serving loops).
//
// It runs the same launches as sislice_ldlt_solve (the preparation of the
// diagonal-block inverses and look-ahead blocks, then the forward and backward
// sweeps), but every buffer beyond the caller's factors and right-hand sides
// lives in one file-scope device array of fixed size.  Nothing is allocated:
// no workspace growth, no pinned staging, no synchronisation.
//
// Each GPU holds its own copy of the array; its address on a device is taken
// once, when the first handle on that device is created, and used from then
// on.  The array keeps the contents of the last call; the ticket counters
// that must start at zero are cleared by a kernel at the start of each call.
// Calls that overlap on one GPU (two streams, two handles) share the array and
// race.
#include <mutex>
#include <vector>

#include "handle.hpp"
#include "solve.hpp"

// Largest order the array is sized for (right-hand sides up to 64): 14.1 MiB at
// n = 4096.
constexpr int64_t kNoallocMaxN = 4096;
constexpr size_t kScratchBytes = 15u << 20;

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace sislice {

namespace {

std::mutex g_scratch_mu;
std::vector<void*> g_scratch_addr;  // per device: device address of `scratch`

struct Layout {
  size_t perm, blk, linv, z, v, ctr, total;
};

// byte offset of the next 256-aligned region of `bytes`
size_t place(size_t& off, size_t bytes) {
  off = (off + 255) & ~size_t(255);
  const size_t o = off;
  off += bytes;
  return o;
}

Layout layout(int64_t n) {
  Layout L;
  size_t off = 0;
  L.perm = place(off, sizeof(int) * (size_t)n);
  L.blk = place(off, sizeof(int) * (size_t)n);
  L.linv = place(off, sizeof(double) * solve_linv_size(n));
  L.z = place(off, sizeof(double) * (size_t)n * kSolveApiRhs);
  L.v = place(off, sizeof(double) * (size_t)n * kSolveApiRhs);
  L.ctr = place(off, sizeof(unsigned) * 64);
  L.total = off;
  return L;
}

__global__ void k_noalloc_clear(unsigned* ctr) { ctr[threadIdx.x] = 0u; }

}  // namespace

void* noalloc_scratch_setup(int device) {
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if ((int)g_scratch_addr.size() <= device) g_scratch_addr.resize(device + 1, nullptr);
  if (!g_scratch_addr[device]) {
    void* p = nullptr;
    SL_HIP(hipSetDevice(device));
    SL_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    SL_CHECK_ARG(p != nullptr, "no device address for the solve scratch array");
    g_scratch_addr[device] = p;
  }
  return g_scratch_addr[device];
}

}  // namespace sislice

using namespace sislice;

extern "C" sislice_status sislice_ldlt_solve_noalloc(sislice_handle* h, int64_t n, const double* LD,
                                                     int64_t ldld, const int32_t* ipiv,
                                                     int64_t nrhs, double* X, int64_t ldx) {
  try {
    check_handle(h);
    SL_CHECK_ARG(n >= 0 && n <= kNoallocMaxN,
                 "n exceeds the allocation-free solve's scratch array (n <= 4096)");
    SL_CHECK_ARG(nrhs >= 0 && nrhs <= 64, "nrhs must be in [0, 64]");
    if (n == 0 || nrhs == 0) return SISLICE_OK;
    SL_CHECK_ARG(LD && ipiv && X && ldld >= n && ldx >= n, "bad argument");
    SL_CHECK_ARG(h->scratch != nullptr && h->wait_word != nullptr,
                 "handle has no scratch array or wait word");
    const Layout L = layout(n);
    SL_CHECK_ARG(L.total <= kScratchBytes, "scratch layout exceeds the array");
    char* base = static_cast<char*>(h->scratch);
    SolveScratch w;
    w.perm = reinterpret_cast<int*>(base + L.perm);
    w.blk = reinterpret_cast<int*>(base + L.blk);
    w.Linv = reinterpret_cast<double*>(base + L.linv);
    w.Z = reinterpret_cast<double*>(base + L.z);
    w.V = reinterpret_cast<double*>(base + L.v);
    w.ctr = reinterpret_cast<unsigned*>(base + L.ctr);
    struct NoProf {  // no timing events here: creating them may allocate
      sislice_handle* h;
      bool was;
      ~NoProf() { h->prof = was; }
    } np{h, h->prof};
    h->prof = false;
    hipLaunchKernelGGL(k_noalloc_clear, dim3(1), dim3(64), 0, h->stream, w.ctr);
    SL_LAUNCH_CHECK();
    solve_single_launch((int)n, LD, ldld, ipiv, (int)nrhs, X, ldx, w, h->stream);
    return SISLICE_OK;
  } catch (const Error& e) {
    std::fprintf(stderr, "sislice: %s\n", e.what());
    return e.status;
  }
}
