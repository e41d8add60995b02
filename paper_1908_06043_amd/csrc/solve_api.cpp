// sislice_ldlt_solve: X <- C^{-1} X through the documented factor format.
#include "handle.hpp"
#include "solve.hpp"

using namespace sislice;

extern "C" sislice_status sislice_ldlt_solve(sislice_handle* h, int64_t n, const double* LD,
                                             int64_t ldld, const int32_t* ipiv, int64_t nrhs,
                                             double* X, int64_t ldx) {
  try {
    check_handle(h);
    SL_CHECK_ARG(n >= 0 && n <= (int64_t)1 << 24, "n out of range");
    SL_CHECK_ARG(nrhs >= 0 && nrhs <= 64, "nrhs must be in [0, 64]");
    if (n == 0 || nrhs == 0) return SISLICE_OK;
    SL_CHECK_ARG(LD && ipiv && X && ldld >= n && ldx >= n, "bad argument");
    Sizer z;
    z.take<int>(n);
    z.take<int>(n);
    z.take<double>(solve_linv_size(n));
    z.take<double>((size_t)n * nrhs);
    z.take<double>((size_t)n * nrhs);
    Carver c(ws_get(h, kBufSolve, z.off));
    SolveScratch w;
    w.perm = c.take<int>(n);
    w.blk = c.take<int>(n);
    w.Linv = c.take<double>(solve_linv_size(n));
    w.Z = c.take<double>((size_t)n * nrhs);
    w.V = c.take<double>((size_t)n * nrhs);
    w.ctr = sync_words(h, 64);
    solve_single_launch((int)n, LD, ldld, ipiv, (int)nrhs, X, ldx, w, h->stream);
    return SISLICE_OK;
  } catch (const Error& e) {
    std::fprintf(stderr, "sislice: %s\n", e.what());
    return e.status;
  }
}
