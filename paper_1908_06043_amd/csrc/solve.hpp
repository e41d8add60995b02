// Multi-shift LDL^T solve kernels (launch interface).
#pragma once

#include "common.hpp"

namespace sislice {

constexpr int kSolveBlock = 64;    // rows per dependency block
constexpr int kSolveMaxRhs = 32;   // right-hand sides of one shift per launch
constexpr int kSolveApiRhs = 64;   // right-hand sides of one call through a single factor
constexpr int kSolveGroup = 16;    // its columns per group: one MFMA tile

struct SolveArgs {
  int n = 0, nshift = 0, nrhs = 0;
  const double* const* LD = nullptr;
  long ldld = 0;
  const int* const* perm = nullptr;
  const int* const* blk = nullptr;
  const double* const* Linv = nullptr;  // solve_linv_size(n) doubles per shift (solve_prep_launch)
  const double* const* Y = nullptr;     // input  n x nrhs (ldy)
  long ldy = 0;
  double* const* X = nullptr;           // output n x nrhs (ldx); may alias Y
  long ldx = 0;
  double* const* Z = nullptr;           // scratch n x nrhs (ldz); the forward result
  double* const* V = nullptr;           // scratch n x nrhs (ldz); the backward result
  long ldz = 0;
  unsigned* ctr = nullptr;              // nshift ticket counters, zero-initialised once
  // direct: one factor for the whole launch, "shift" s is its s-th group of nrhs
  // right-hand sides (the last group holds what is left of nrhs_all); the device tables
  // above are not read, input and output are X0 (ldx), scratch Z0 and V0 (ldz)
  int direct = 0, nrhs_all = 0;
  const double* LD0 = nullptr;
  const int* perm0 = nullptr;
  const int* blk0 = nullptr;
  const double* Linv0 = nullptr;
  double* X0 = nullptr;
  double* Z0 = nullptr;
  double* V0 = nullptr;
  int applyD = 1;                       // backward sweep applies D^{-1} first (0: identity)
  unsigned* wait_err = nullptr;         // raised when a hand-off wait exceeds wait_limit polls
  unsigned wait_limit = 0;              // (both set by solve_launch from the handle)
};

// mode 0: X = P^T L^{-T} D^{-1} L^{-1} P Y (both sweeps, Z/V scratch)
// mode 1: Z = L^{-1} P Y only (forward sweep; the result is left in Z)
// mode 2: X = P^T L^{-T} [D^{-1}] Z only (backward sweep reading Z)

// Preparation of the factors for the sweeps; `look` false forms perm, blk and the
// diagonal-block inverses only.
struct SolvePrepArgs {
  int n = 0, look = 1;
  long ldld = 0;
  const double* const* LD = nullptr;
  const int* const* ipiv = nullptr;
  int* const* perm = nullptr;
  int* const* blk = nullptr;
  double* const* Linv = nullptr;
  // direct: one factor, given here instead of in device tables
  int direct = 0;
  const double* LD0 = nullptr;
  const int* ipiv0 = nullptr;
  int* perm0 = nullptr;
  int* blk0 = nullptr;
  double* Linv0 = nullptr;
  // sentinels written into fill_cols columns (ld n) of both, when given
  double* fillZ = nullptr;
  double* fillV = nullptr;
  int fill_cols = 0;
};

void solve_prep_launch(int n, int S, const int* const* d_ipiv, int* const* d_perm,
                       int* const* d_blk, const double* const* d_LD, long ldld,
                       double* const* d_Linv, hipStream_t st, bool look = true);
// Scratch of solve_single_launch: perm, blk [n], Linv [solve_linv_size(n)], Z and V
// n x nrhs, and one zero ticket counter per group.
struct SolveScratch {
  int* perm = nullptr;
  int* blk = nullptr;
  double* Linv = nullptr;
  double* Z = nullptr;
  double* V = nullptr;
  unsigned* ctr = nullptr;
};
void solve_single_launch(int n, const double* LD, long ldld, const int* ipiv, int nrhs, double* X,
                         long ldx, const SolveScratch& w, hipStream_t st);
void solve_launch(SolveArgs a, hipStream_t st, int mode = 0);
// Scatter the 64x64 diagonal-block inverses (layout of solve_prep_launch's Linv)
// onto the block diagonal of an n x n matrix.
void diag_inv_scatter_launch(int n, const double* Linv, double* Li, long ldli, hipStream_t st);

inline long solve_nblk(long n) { return ceil_div(n, kSolveBlock); }
// Depth of the sweeps' look-ahead: the nearest kSolveLook blocks enter a block's
// result through precomputed products, the rest through P_b.
constexpr int kSolveLook = 2;
// per shift: the 64x64 diagonal-block inverses of L, then the forward and the
// backward look-ahead blocks of each depth ((1 + 2 kSolveLook) * nblk column-major
// 64x64 blocks)
inline size_t solve_linv_size(long n) {
  return (1 + 2 * (size_t)kSolveLook) * (size_t)solve_nblk(n) * kSolveBlock * kSolveBlock;
}


}  // namespace sislice
