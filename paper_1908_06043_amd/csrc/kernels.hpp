// Launch plans of the device kernels (internal to the library).
#pragma once

#include <algorithm>

#include "common.hpp"

namespace sislice {

constexpr int kSpecGroups = 256;  // workgroups of a shift's pivot-free panel, at most

// Whole panels that are updated together, at most (W of all of them is kept).  Order 12288, 49
// shifts: 880 ms with 2, 843 with 3, 795 with 6, 788 with 8; order 4096, 17 shifts: 23.6, 23.1,
// 22.9, 23.1.
constexpr int kDeferPanels = 6;

// Words of one shift's team area (k_bk_team): the roster, then the mailboxes.
constexpr int kTeamMax = 32;  // workgroups in a team
constexpr int kTeamRow = 136;  // words of one workgroup's row
constexpr int kTeamWords = 64 + 4 * (4 * kTeamMax + 128) + 2 * kTeamMax * kTeamRow;

// Polls (about half a microsecond each) that the first workgroup gives its team to gather, and
// the wait limit below which no team gathers: its members run at the same time and answer
// within microseconds, so from here on (some 60 ms) only a fault lets a wait expire.
constexpr unsigned kTeamGather = 40;
constexpr unsigned kTeamMinLimit = 1u << 16;

// One lock-step factorization of `nshift` shifted matrices of order n.
struct FactorPlan {
  int n = 0, nshift = 0, nb = 32;
  bool pivot = true;  // false: LDL^T without interchanges (B is SPD)
  const double* A = nullptr;
  const double* B = nullptr;
  long lda = 0, ldb = 0;
  const double* d_sigmas = nullptr;  // device [nshift]
  double* const* d_LD = nullptr;     // device table of nshift device pointers
  long ldld = 0;
  double* const* d_W = nullptr;  // panel buffers n x (max(defer, 1) nb + 2)
  long ldw = 0;
  int* const* d_perm = nullptr;
  int* const* d_sw = nullptr;
  int* const* d_blk = nullptr;
  int* const* d_colpanel = nullptr;
  int* const* d_pstart = nullptr;
  int* const* d_snap = nullptr;
  int* const* d_ipiv = nullptr;
  FactorState* d_state = nullptr;
  int64_t* d_inertia = nullptr;  // device [3 * nshift]
  int* pstart_base = nullptr;    // device [nshift * npmax] panel starts
  int npmax = 0;
  // pivot-free panel path (per shift): D of the panel and the columns that fail its test
  double* const* d_aux = nullptr;  // [nb] D | [kSpecGroups] rejected columns (a uint64 a workgroup)
  unsigned long long* d_team = nullptr;  // device [nshift * kTeamWords]: mailboxes of the panel teams
  unsigned* wait_err = nullptr;    // raised when a team's wait exceeds wait_limit polls
  unsigned wait_limit = 0;
  int nbpiv = 32;                  // columns a pivoting panel handles after a rejection (default_nbpiv)
  int wide_min = 1024;             // trailing order from which the update takes 128x128 tiles
  int defer = 0;                   // whole panels whose updates may wait for one another (W has room)
  int stream_c = 0;                // the 128-tile update streams C (shift groups on two streams)
  int cus = 256;                   // compute units of the device (its persistent grid)
  int groups = 1;                  // shift groups run on separate streams (with readback)
};

// The whole factorization: shift-form, then the panel/update steps with the
// per-shift progress read back every few steps, the deferred interchanges and
// the inertia.
void factor_launch(const FactorPlan& fp, hipStream_t st);
// The two parts on their own.  With readback == false every step up to the bound
// factor_npanel_max is launched and nothing synchronises (a sequence that a HIP
// graph can capture: its kernels read the shifted matrices through the plan's
// device tables only).
void factor_shift_form_launch(const FactorPlan& fp, hipStream_t st);
void factor_steps_launch(const FactorPlan& fp, hipStream_t st, bool readback);
// Whole panels that may wait for one another (W then holds as many, 4 GiB of them at most,
// so that a factorization which fills the memory still fits); 0: none.
int factor_defers(int n, int nb, int nshift, bool pivot);
// One-time kernel attributes of the factorization (outside any capture).
void factor_prepare();

// What the first inertia count holds of a factorization that is not one.
constexpr int64_t kUnfinishedInertia = -1;
constexpr int64_t kSpoiledInertia = -2;

// Narrowest panel that is not the last one: a pivoting panel stops at nb - 1
// columns (room for a closing 2x2 pivot) and, behind the pivot-free path, after
// nbpiv columns from the first rejected one.
inline int factor_min_panel(int nb, int nbpiv) {
  const int w = std::min(nbpiv, nb - 1);
  return w < 1 ? 1 : w;
}

// Upper bound on the number of panel steps (and so on the panels) of one
// factorization; sizes the panel-start and interchange-snapshot arrays.
inline int factor_npanel_max(int n, int nb, int nbpiv) {
  return (int)ceil_div(n, factor_min_panel(nb, nbpiv)) + 2;
}

}  // namespace sislice
