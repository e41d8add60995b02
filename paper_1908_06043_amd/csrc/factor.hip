// Blocked Bunch-Kaufman LDL^T of C = A - sigma B for several shifts at once,
// and the Sylvester inertia read from D.
//
// The paper (Section 2.1) identifies this factorization as the major cost of a
// spectral probe and (Section 2.2) reads the exact eigenvalue count below sigma
// from D.  The pivoting rule is Bunch-Kaufman's (alpha = (1+sqrt 17)/8).
//
// Design (gfx950): every shift of the GPU's share advances in lock step.
//   * k_bk_panel: one 1024-thread workgroup per shift factors a panel of up to nb
//     columns in the "lazy" form S = A_trail - L_panel W_panel^T: each column of
//     S (and the pivot-candidate column when Bunch-Kaufman needs it) is formed by
//     a GEMV against the panel so far, pivots are chosen by block-wide argmax
//     reductions, symmetric interchanges are applied to the not-yet-updated
//     trailing matrix (lower storage) and to the panel rows.
//   * k_bk_team: the same panel by a team of workgroups with L in registers, where
//     the teams of all shifts fit the device; k_fast_panel before it takes the
//     columns that need no pivoting.
//   * k_trailing_update, k_trailing_update_lds: the lower triangle of the trailing
//     matrix is updated with C22 -= L21 W21^T on FP64 MFMA (v_mfma_f64_16x16x4),
//     64x64 and 128x128 tiles, all shifts in one launch; large ones several panels at once.
//   * Interchanges found in later panels are applied to earlier L columns once at
//     the end (k_perm_suffix builds the suffix permutations, k_left_gather moves
//     the rows), so that P C P^T = L D L^T with a single permutation P.
// Panel widths depend on the pivots (nb-1 or nb columns), so the per-shift
// progress lives in device memory (FactorState) and the host launches an upper
// bound of panel/update pairs; launches past the end return at once.
#include <algorithm>
#include <cfloat>
#include <climits>

#include "common.hpp"
#include "handle.hpp"
#include "kernels.hpp"

namespace sislice {

// ------------------------------------------------------------------ helpers

__device__ __forceinline__ void wave_argmax(double& v, int& i) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double ov = __shfl_xor(v, off);
    const int oi = __shfl_xor(i, off);
    if (ov > v || (ov == v && oi < i)) {
      v = ov;
      i = oi;
    }
  }
}

// Block-wide (max |value|, smallest index) reduction; every thread gets the result.
template <int NW>
__device__ __forceinline__ void block_argmax(double& v, int& i, double* rv, int* ri) {
  wave_argmax(v, i);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) {
    rv[w] = v;
    ri[w] = i;
  }
  __syncthreads();
  v = rv[0];
  i = ri[0];
#pragma unroll
  for (int q = 1; q < NW; ++q) {
    const double ov = rv[q];
    const int oi = ri[q];
    if (ov > v || (ov == v && oi < i)) {
      v = ov;
      i = oi;
    }
  }
  __syncthreads();
}

// ------------------------------------------------------------------ kernels

// LD[i, j] = A[i, j] - sigma_s B[i, j] on the lower triangle (Algorithm 2, step 2)
// for every shift s: column j per workgroup, A and B read once for all shifts.
__global__ __launch_bounds__(256) void k_shift_form(int n, int S, const double* __restrict__ A,
                                                    long lda, const double* __restrict__ B,
                                                    long ldb, const double* __restrict__ sigmas,
                                                    double* const* LDs, long ldld) {
  const int j = blockIdx.x;
  for (int i = j + threadIdx.x; i < n; i += blockDim.x) {
    const double a = A[i + (long)j * lda], b = B[i + (long)j * ldb];
    for (int s = 0; s < S; ++s) LDs[s][i + (long)j * ldld] = a - sigmas[s] * b;
  }
}

__global__ __launch_bounds__(256) void k_factor_init(int n, FactorState* states, int* const* perms,
                                                     int* const* swps, unsigned long long* teams) {
  const int s = blockIdx.y;
  // no mailbox word carries a tag of this factorization yet
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kTeamWords; i += gridDim.x * blockDim.x)
    teams[(long)s * kTeamWords + i] = 0;
  int* perm = global_ptr(perms[s]);
  int* sw = global_ptr(swps[s]);
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    perm[i] = i;
    sw[i] = i;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    FactorState z;
    z.k0 = 0;
    z.kb = 0;
    z.done = (n == 0);
    z.npanel = 0;
    z.neg = z.zero = z.pos = 0;
    z.jstart = 0;
    z.whole = z.pend = 0;
    z.u_k0 = z.u_kb = z.u_w0 = 0;
    z.u_c0 = z.u_c1 = n;
    states[s] = z;
  }
}


// ---------------------------------------------------------------- pivot-free path
//
// Bunch-Kaufman takes a 1x1 pivot without interchange at column k exactly when
// |d_k| >= alpha * max_{i>k} |s_ik| for the Schur-complement column s at step k.
// As long as that holds for every column, the factorization is the pivot-free
// LDL^T, which parallelises like Cholesky: k_fast_panel factors the panel's diagonal
// block, solves for the rows below and tests every column, and k_fast_commit accepts
// the longest prefix of columns that pass and writes their L = W D^{-1}.  The pivoting panel kernel then continues from the first
// rejected column, so the result is the Bunch-Kaufman factorization itself.

// a[i] += m[lane i of the row] * f for the 16 registers a: m supplies one multiplier a lane, the
// same in each row of 16 lanes.  (s_nop: a DPP source written by the instruction before.)
__device__ __forceinline__ void axpy16(double* a, double m, double f) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %16, %17 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %16, %17 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %16, %17 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %16, %17 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %4, %16, %17 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %5, %16, %17 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %6, %16, %17 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %7, %16, %17 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %8, %16, %17 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %9, %16, %17 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %10, %16, %17 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %11, %16, %17 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %12, %16, %17 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %13, %16, %17 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %14, %16, %17 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %15, %16, %17 row_newbcast:15 row_mask:0xf bank_mask:0xf"
      : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]),
        "+v"(a[8]), "+v"(a[9]), "+v"(a[10]), "+v"(a[11]), "+v"(a[12]), "+v"(a[13]), "+v"(a[14]), "+v"(a[15])
      : "v"(m), "v"(f));
}

__device__ __forceinline__ double lane_f64(double x, int lane) {
  const long long u = __double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)u, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(u >> 32), lane);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The pivot-free panel: LDL^T of the diagonal block (nbe <= NB columns), the rows below it,
// W21 = C21 L11^{-T} by forward substitution along each row, and the columns that fail the
// test, one bit a column.
//
// What bounds it: the chain of the diagonal block, a pivot, its reciprocal and the
// multipliers, column by column.  One wavefront factors the block with a row a lane and the
// columns in registers: no barrier in the chain (a column's multipliers go through LDS to
// the lanes that broadcast them).  Every workgroup factors the block for itself, its fifth
// wavefront ahead of the four that hold a row a lane and follow U columns behind, so the
// rows cost neither a launch nor time of their own.  Columns sit in registers from the
// current one on and move down every U columns, so that a column's register is known at
// compile time in a loop small enough for the instruction cache; whole groups of 16 past
// the block are skipped.
//
// The test |d_k| >= alpha max_i |w_ik| holds exactly when it holds for every i, rounding
// being monotone, so a comparison per element and a bit per column replace the maxima; without
// the test (B of a definite pencil) an entry has to be finite.
//
// Measured, per launch: order 4096, 17 shifts 72 us as a launch for the block (four lanes a
// row, two barriers a column) and one for the rows, 29.5 so; order 2048, one matrix 55 and
// 23.4; order 1001, five shifts, 32 columns 23 and 11.7.  A column of the block is about 380
// cycles, one of the rows 360; without following one behind the other: 38 us at 4096.
template <int NB, bool PIVOT>
__global__ __launch_bounds__(320) void k_fast_panel(int n, const double* const* LDs, long ldld,
                                                    double* const* Wps, long ldw,
                                                    double* const* auxs,
                                                    const FactorState* states,
                                                    unsigned long long* teams, int nb) {
  constexpr int U = 8, G = NB / 16;
  // Column k of W and of L11 at [k * NB], for rows (of the block) past k.  What lies before,
  // and past the block, is read as well, into registers that hold no live column.
  __shared__ double sW[NB * NB];
  __shared__ double sL[NB * NB + 64];
  __shared__ unsigned long long sBad;
  __shared__ int sDone;  // columns whose W and L11 are in LDS
  const int s = blockIdx.y, tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const FactorState st = states[s];
  const int k0 = st.k0 + st.kb;
  if (st.done || k0 >= n) return;
  const int nbe = __builtin_amdgcn_readfirstlane(min(nb, n - k0));
  const double* LD = global_ptr(LDs[s]);
  double* Wp = global_ptr(Wps[s]) + st.pend * ldw;
  double* Dv = global_ptr(auxs[s]);
  unsigned long long* bad_of = reinterpret_cast<unsigned long long*>(Dv + nb);
  double x[NB];
  // (a row past the end stands for the last row once more; so does a column)
  auto load = [&](int first) {
    const double* p = LD + min(first + lane, n - 1) + (long)k0 * ldld;
#pragma unroll
    for (int m = 0; m < NB; ++m) {
      x[m] = *p;
      p += m + 1 < nbe ? ldld : 0;
    }
  };
  // (loads and stores share a counter: a load still in flight would make each column wait for
  // the stores of the column before)
  auto arrived = [] { __builtin_amdgcn_s_waitcnt(0x0f70); };  // vmcnt(0)
  auto shift = [&]() {
#pragma unroll
    for (int m = 0; m < NB; ++m) x[m] = m + U < NB ? x[m + U] : 0.0;
  };
  auto passes = [](double wk, double d) {
    return PIVOT ? kBkAlpha * fabs(wk) <= fabs(d) : fabs(wk) <= DBL_MAX;
  };
  if (tid == 0) {
    sBad = 0;
    sDone = 0;
    if (blockIdx.x == 0) {  // the pivoting panel's workgroups gather anew
      teams[(long)s * kTeamWords] = 0;
      teams[(long)s * kTeamWords + 1] = 0;
    }
  }
  __syncthreads();
  unsigned long long bad = 0;
  if (w == 4) {
    __builtin_amdgcn_s_setprio(3);  // (it shares a SIMD with one of the others)
    load(k0);
    arrived();
    double* wc = sW + lane;
    double* lc = sL + lane;
    auto multipliers = [&](double a, int k) {  // column k of the block
      const double l = a * (1.0 / lane_f64(a, min(k, 63)));
      if (NB == 64 || lane < NB) {
        wc[k * NB] = a;
        lc[k * NB] = l;
      }
    };
    multipliers(x[0], 0);
#pragma unroll 1
    for (int t0 = 0; t0 < nbe; t0 += U) {
      int left = nbe - t0;
#pragma unroll
      for (int kk = 0; kk < U; ++kk) {
        const int k = t0 + kk;
        const double f = -x[kk];
        const double* mp = sL + k * NB + t0 + (lane & 15);
        double m[G];
#pragma unroll
        for (int g = 0; g < G; ++g) m[g] = mp[16 * g];
        axpy16(x, m[0], f);
        // the next column is complete: its multipliers start before the columns to the right
        if (k + 1 < NB) multipliers(x[kk + 1], k + 1);
        asm volatile("" : "+s"(left));  // (compared here: not kept for every column, or copied)
#pragma unroll
        for (int g = 1; g < G; ++g)
          if (16 * g < left) axpy16(x + 16 * g, m[g], f);
      }
      // (LDS takes a wavefront's accesses in order)
      asm volatile("" ::: "memory");
      if (lane == 0) __hip_atomic_store(&sDone, t0 + U, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      shift();
    }
    __builtin_amdgcn_s_setprio(0);
    if (blockIdx.x == 0) {
      if (lane < nbe) {
        const double d = sW[lane * (NB + 1)];
        Dv[lane] = d;
        if (!(isfinite(d) && d != 0.0)) bad = 1ull << lane;
      }
      if (bad) atomicOr(&sBad, bad);
      bad = 0;
#pragma unroll 8
      for (int k = 0; k < nbe; ++k) {
        const double wk = sW[k * NB + min(lane, NB - 1)], d = sW[k * (NB + 1)];
        if (lane >= k && lane < nbe) Wp[(k0 + lane) + (long)k * ldw] = wk;
        bad |= lane > k && lane < nbe && !passes(wk, d) ? 1ull << k : 0ull;
      }
      if (bad) atomicOr(&sBad, bad);
    }
  } else {
    for (int r0 = k0 + nbe + 256 * (int)blockIdx.x + 64 * w; r0 < n; r0 += 256 * (int)gridDim.x) {
      load(r0);
      arrived();
      double* out = Wp + min(r0 + lane, n - 1);
#pragma unroll 1
      for (int t0 = 0; t0 < nbe; t0 += U) {
        while (__hip_atomic_load(&sDone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) <= t0)
          __builtin_amdgcn_s_sleep(1);
        asm volatile("" ::: "memory");
        const double* mp = sL + t0 * NB + t0 + (lane & 15);
        const double* dp = sW + t0 * (NB + 1);
        double m[2][G], d[2];
        auto fetch = [&](int kk) {
#pragma unroll
          for (int g = 0; g < G; ++g) m[kk & 1][g] = mp[kk * NB + 16 * g];
          d[kk & 1] = dp[kk * (NB + 1)];
        };
        int left = nbe - t0;
        unsigned long long fail[U];
        fetch(0);
#pragma unroll
        for (int kk = 0; kk < U; ++kk) {
          asm volatile("" : "+s"(left));
          if (kk + 1 < U) fetch(kk + 1);
          const double wk = x[kk];
          if (kk < left) *out = wk;
          fail[kk] = __ballot(!passes(wk, d[kk & 1]));
          out += ldw;
#pragma unroll
          for (int g = 0; g < G; ++g)
            if (g == 0 || 16 * g < left) axpy16(x + 16 * g, m[kk & 1][g], -wk);
        }
        unsigned bits = 0;
#pragma unroll
        for (int kk = 0; kk < U; ++kk) bits |= fail[kk] ? 1u << kk : 0u;
        bad |= (unsigned long long)bits << t0;
        shift();
      }
    }
    if (lane == 0 && bad) atomicOr(&sBad, bad);
  }
  __syncthreads();
  if (tid == 0) bad_of[blockIdx.x] = sBad;
}

// The accepted columns: the longest prefix that passed in every one of the `groups` (<= the
// workgroup's threads) workgroups of k_fast_panel.  sh: a word of LDS.
__device__ __forceinline__ int accepted_columns(const double* Dv, int nb, int nbe, int groups, int* sh) {
  const unsigned long long* bad_of = reinterpret_cast<const unsigned long long*>(Dv + nb);
  if (threadIdx.x == 0) *sh = nbe;
  __syncthreads();
  if ((int)threadIdx.x < groups) {
    const unsigned long long b = bad_of[threadIdx.x];
    if (b) atomicMin(sh, __ffsll((long long)b) - 1);
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(*sh);
}

// Column c of the accepted prefix: L = W D^{-1}, by the whole workgroup.
__device__ __forceinline__ void accept_column(int n, double* LD, long ldld, const double* Wp, long ldw,
                                              const double* Dv, int* blk, int* colpanel, int k0, int c,
                                              int panel) {
  const int col = k0 + c;
  const double rd = 1.0 / Dv[c];  // the column's multipliers l = w (1 / d)
  for (int i = col + 1 + threadIdx.x; i < n; i += blockDim.x)
    LD[i + (long)col * ldld] = Wp[i + (long)c * ldw] * rd;
  if (threadIdx.x == 0) {
    LD[col + (long)col * ldld] = Dv[c];
    blk[col] = 1;
    colpanel[col] = panel;
  }
}

// The panel state after js accepted columns, by the first wavefront.
__device__ __forceinline__ void accept_state(FactorState* st, const double* Dv, int js) {
  const int lane = threadIdx.x;
  const bool acc = lane < js;
  const bool negd = acc && Dv[lane] < 0.0;
  const unsigned long long negm = __ballot(negd), posm = __ballot(acc && !negd);
  if (lane == 0) {
    st->jstart = js;
    st->neg += __popcll(negm);
    st->pos += __popcll(posm);
  }
}

// The state after a panel of j columns from k0, js of them accepted by the pivot-free path
// (nbe: the columns that path took on), and the update that follows, at most `defer` whole
// panels together; one thread.
__device__ __forceinline__ void panel_done(FactorState* st, int n, int nb, int nbe, int k0, int j, int js,
                                           int panel, int defer) {
  const int pend = st->pend, k1 = k0 + j;
  const int before = js == nbe ? pend : 0;  // (otherwise the panels before have been caught up)
  const bool whole = js == nb;
  st->k0 = k0;
  st->kb = j;
  st->npanel = panel + 1;
  st->done = k1 >= n;
  st->jstart = 0;
  st->whole += whole;
  const bool wait = whole && before + nb < defer * nb && k1 < n;
  st->u_k0 = k0 - before;
  st->u_kb = before + j;
  st->u_w0 = pend - before;
  st->u_c0 = k1;
  st->u_c1 = wait ? min(n, k1 + nb) : n;
  st->pend = wait ? before + j : 0;
}

// The pivoting panel on one workgroup, for any number of rows.  Each column of S is
// formed from the panel's L in memory, so a column costs one CU's reads of (n - k) j
// doubles (4 us at order 4096); k_bk_team below keeps L in registers.
template <bool PIVOT, int NT>
__device__ __forceinline__ void bk_panel_rows(int n, double* const* LDs, long ldld,
                                              double* const* Wps, long ldw, int* const* perms,
                                              int* const* swps, int* const* blks,
                                              int* const* colpanels, int* const* pstarts,
                                              FactorState* states, int nb, int nbpiv, int s,
                                              int defer) {
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x;
  FactorState* st = states + s;
  double* __restrict__ LD = global_ptr(LDs[s]);
  double* __restrict__ Wp = global_ptr(Wps[s]) + st->pend * ldw;
  int* perm = global_ptr(perms[s]);
  int* sw = global_ptr(swps[s]);
  int* blk = global_ptr(blks[s]);
  int* colpanel = global_ptr(colpanels[s]);
  int* pstart = global_ptr(pstarts[s]);

  __shared__ double wk[kMaxNb + 2];
  __shared__ double red_v[NW];
  __shared__ int red_i[NW];
  __shared__ double sh_absakk, sh_arr;
  __shared__ int sh_k0, sh_done, sh_panel, sh_jstart;

  if (tid == 0) {
    const int k0 = st->k0 + st->kb;
    sh_k0 = k0;
    sh_done = (k0 >= n) || st->done;
    sh_panel = st->npanel;
    sh_jstart = st->jstart;
  }
  __syncthreads();
  if (sh_done) {
    if (tid == 0) {
      st->k0 = sh_k0 < n ? sh_k0 : n;
      st->kb = 0;
      st->done = 1;
      st->u_c0 = n;
    }
    return;
  }
  const int k0 = sh_k0, P = sh_panel;
  const int rem = n - k0;
  const int jstart = sh_jstart;
  const int jmax0 = (rem <= nb) ? rem : nb - 1;
  const int jmax = min(jmax0, jstart + nbpiv);
  long neg = 0, zer = 0, pos = 0;

  int j = jstart;
  while (j < jmax) {
    const int k = k0 + j;
    // row k of the panel's W
    for (int p = tid; p < j; p += NT) wk[p] = Wp[k + (long)p * ldw];
    __syncthreads();
    // column k of the Schur complement -> W(:, j); argmax below the diagonal
    double bv = -1.0;
    int bi = INT_MAX;
    for (int i0 = k + tid; i0 < n; i0 += 2 * NT) {
      const int i1 = i0 + NT;
      const bool two = i1 < n;
      double a0 = LD[i0 + (long)k * ldld], a1 = two ? LD[i1 + (long)k * ldld] : 0.0;
      double b0 = 0.0, b1 = 0.0;
      const double* L0 = LD + i0 + (long)k0 * ldld;
      const double* L1 = LD + (two ? i1 : i0) + (long)k0 * ldld;
      // eight columns per step with all sixteen loads issued first (one wait per
      // step); even columns accumulate into a, odd ones into b, in column order
      int p = 0;
      for (; p + 8 <= j; p += 8) {
        double x0[8], x1[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          x0[u] = L0[(long)(p + u) * ldld];
          x1[u] = L1[(long)(p + u) * ldld];
        }
#pragma unroll
        for (int u = 0; u < 8; u += 2) {
          const double w0 = wk[p + u], w1 = wk[p + u + 1];
          a0 -= x0[u] * w0;
          b0 -= x0[u + 1] * w1;
          a1 -= x1[u] * w0;
          b1 -= x1[u + 1] * w1;
        }
      }
      for (; p + 1 < j; p += 2) {
        const double w0 = wk[p], w1 = wk[p + 1];
        const double x00 = L0[(long)p * ldld], x01 = L0[(long)(p + 1) * ldld];
        const double x10 = L1[(long)p * ldld], x11 = L1[(long)(p + 1) * ldld];
        a0 -= x00 * w0;
        b0 -= x01 * w1;
        a1 -= x10 * w0;
        b1 -= x11 * w1;
      }
      if (p < j) {
        a0 -= L0[(long)p * ldld] * wk[p];
        a1 -= L1[(long)p * ldld] * wk[p];
      }
      a0 += b0;
      a1 += b1;
      Wp[i0 + (long)j * ldw] = a0;
      if (two) Wp[i1 + (long)j * ldw] = a1;
      if (i0 == k) {
        sh_absakk = fabs(a0);
      } else {
        const double a = fabs(a0);
        if (a > bv) {
          bv = a;
          bi = i0;
        }
      }
      if (two) {
        const double a = fabs(a1);
        if (a > bv) {
          bv = a;
          bi = i1;
        }
      }
    }
    block_argmax<NW>(bv, bi, red_v, red_i);
    const double absakk = sh_absakk;
    const double colmax = bv > 0.0 ? bv : 0.0;
    const int imax = bi;

    int kstep = 1, kp = k;
    if (PIVOT && absakk < kBkAlpha * colmax) {
      // candidate column imax of the Schur complement -> W(:, j+1)
      for (int p = tid; p < j; p += NT) wk[p] = Wp[imax + (long)p * ldw];
      __syncthreads();
      double rv = -1.0;
      int ri = INT_MAX;
      for (int i = k + tid; i < n; i += NT) {
        double acc = (i < imax) ? LD[imax + (long)i * ldld] : LD[i + (long)imax * ldld];
        const double* Lr = LD + i + (long)k0 * ldld;
        int p = 0;
        for (; p + 8 <= j; p += 8) {
          double x[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) x[u] = Lr[(long)(p + u) * ldld];
#pragma unroll
          for (int u = 0; u < 8; ++u) acc -= x[u] * wk[p + u];
        }
        for (; p < j; ++p) acc -= Lr[(long)p * ldld] * wk[p];
        Wp[i + (long)(j + 1) * ldw] = acc;
        if (i == imax) {
          sh_arr = fabs(acc);
        } else {
          const double a = fabs(acc);
          if (a > rv) {
            rv = a;
            ri = i;
          }
        }
      }
      block_argmax<NW>(rv, ri, red_v, red_i);
      const double rowmax = rv;
      const double arr = sh_arr;
      if (absakk * rowmax >= kBkAlpha * colmax * colmax) {
        kstep = 1;
        kp = k;
      } else if (arr >= kBkAlpha * rowmax) {
        kstep = 1;
        kp = imax;
      } else {
        kstep = 2;
        kp = imax;
      }
    }
    const int kk = k + kstep - 1;
    if (kp != kk) {
      // symmetric interchange kk <-> kp of the not-yet-updated trailing matrix:
      // kk becomes a pivot column, so only position kp needs column kk's entries
      for (int i = kk + 1 + tid; i < n; i += NT) {
        if (i == kp) continue;
        const double v = LD[i + (long)kk * ldld];
        if (i > kp)
          LD[i + (long)kp * ldld] = v;
        else
          LD[kp + (long)i * ldld] = v;
      }
      // rows kk, kp of the panel's L columns and of W
      for (int c = tid; c < j; c += NT) {
        double* a = LD + kk + (long)(k0 + c) * ldld;
        double* b = LD + kp + (long)(k0 + c) * ldld;
        const double t = *a;
        *a = *b;
        *b = t;
        double* wa = Wp + kk + (long)c * ldw;
        double* wb = Wp + kp + (long)c * ldw;
        const double tw = *wa;
        *wa = *wb;
        *wb = tw;
      }
      if (tid == 0) {
        LD[kp + (long)kp * ldld] = LD[kk + (long)kk * ldld];
        for (int q = j; q <= j + 1; ++q) {
          double* wa = Wp + kk + (long)q * ldw;
          double* wb = Wp + kp + (long)q * ldw;
          const double tw = *wa;
          *wa = *wb;
          *wb = tw;
        }
        const int tp = perm[kk];
        perm[kk] = perm[kp];
        perm[kp] = tp;
      }
    }
    if (tid == 0) {
      sw[k] = (kstep == 1) ? kp : k;
      if (kstep == 2) sw[k + 1] = kp;
    }
    __syncthreads();
    if (kstep == 1 && kp != k) {
      // the pivot column is the candidate column
      for (int i = k + tid; i < n; i += NT) Wp[i + (long)j * ldw] = Wp[i + (long)(j + 1) * ldw];
      __syncthreads();
    }
    if (kstep == 1) {
      const double d = Wp[k + (long)j * ldw];
      const double dinv = (d != 0.0) ? 1.0 / d : 0.0;
      for (int i = k + 1 + tid; i < n; i += NT)
        LD[i + (long)k * ldld] = Wp[i + (long)j * ldw] * dinv;
      if (tid == 0) {
        LD[k + (long)k * ldld] = d;
        blk[k] = 1;
        colpanel[k] = P;
        if (d < 0.0)
          ++neg;
        else if (d > 0.0)
          ++pos;
        else
          ++zer;
      }
    } else {
      const double d11 = Wp[k + (long)j * ldw];
      const double d21 = Wp[k + 1 + (long)j * ldw];
      const double d22 = Wp[k + 1 + (long)(j + 1) * ldw];
      // [l1 l2] = [w1 w2] D^{-1}, scaled by the off-diagonal d21 (never 0 here)
      const double a = d11 / d21, g = d22 / d21;
      const double t = 1.0 / (d21 * (a * g - 1.0));
      for (int i = k + 2 + tid; i < n; i += NT) {
        const double w1 = Wp[i + (long)j * ldw];
        const double w2 = Wp[i + (long)(j + 1) * ldw];
        LD[i + (long)k * ldld] = t * (g * w1 - w2);
        LD[i + (long)(k + 1) * ldld] = t * (a * w2 - w1);
      }
      if (tid == 0) {
        LD[k + (long)k * ldld] = d11;
        LD[k + 1 + (long)k * ldld] = d21;
        LD[k + 1 + (long)(k + 1) * ldld] = d22;
        blk[k] = 2;
        blk[k + 1] = 0;
        colpanel[k] = P;
        colpanel[k + 1] = P;
        const double det = d11 * d22 - d21 * d21;
        const double tr = d11 + d22;
        if (det < 0.0) {
          ++neg;
          ++pos;
        } else if (det > 0.0) {
          if (tr < 0.0)
            neg += 2;
          else
            pos += 2;
        } else {
          ++zer;
          if (tr < 0.0)
            ++neg;
          else if (tr > 0.0)
            ++pos;
          else
            ++zer;
        }
      }
    }
    __syncthreads();
    j += kstep;
  }
  if (tid == 0) {
    panel_done(st, n, nb, min(nb, rem), k0, j, jstart, P, defer);
    st->neg += neg;
    st->zero += zer;
    st->pos += pos;
    pstart[P] = k0;
  }
}

// Accepts the prefix, one workgroup a column, where no team follows (a team accepts for
// itself).  Without pivoting the panel ends here: the workgroup that arrives last, when all of
// the shift's (those past a ragged panel's columns as well) have read the state, writes it, or,
// where a column failed (a zero or non-finite pivot), goes on
// column by column after writing the accepted ones once more for itself.  That saves a launch
// a panel: planning at order 2048 5.56 -> 5.48 ms, a solve of order 1000 18.0 -> 17.6.
template <bool PIVOT>
__global__ __launch_bounds__(256) void k_fast_commit(int n, double* const* LDs, long ldld,
                                                     double* const* Wps, long ldw,
                                                     const double* const* auxs, int* const* perms,
                                                     int* const* swps, int* const* blks,
                                                     int* const* colpanels, int* const* pstarts,
                                                     FactorState* states, unsigned long long* teams,
                                                     int nb, int nbpiv, int groups) {
  __shared__ int sh;
  const int s = blockIdx.y, c = blockIdx.x;
  const FactorState st = states[s];
  const int k0 = st.k0 + st.kb;
  if (st.done || k0 >= n) return;
  const int nbe = min(nb, n - k0);
  if (PIVOT && c >= nbe) return;
  const double* Dv = global_ptr(auxs[s]);
  const double* Wp = global_ptr(Wps[s]) + st.pend * ldw;
  double* LD = global_ptr(LDs[s]);
  int* blk = global_ptr(blks[s]);
  int* colpanel = global_ptr(colpanels[s]);
  const int js = accepted_columns(Dv, nb, nbe, groups, &sh);
  if (c < js) accept_column(n, LD, ldld, Wp, ldw, Dv, blk, colpanel, k0, c, st.npanel);
  if (PIVOT) {
    if (c == 0 && threadIdx.x < 64) accept_state(states + s, Dv, js);
    return;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    sh = (int)__hip_atomic_fetch_add(reinterpret_cast<unsigned*>(teams + (long)s * kTeamWords), 1u,
                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (sh != (int)gridDim.x - 1) return;
  if (threadIdx.x < 64) accept_state(states + s, Dv, js);
  if (js == nbe) {
    if (threadIdx.x == 0) {
      panel_done(states + s, n, nb, nbe, k0, js, js, st.npanel, 0);
      global_ptr(pstarts[s])[st.npanel] = k0;
    }
    return;
  }
  for (int q = 0; q < js; ++q) accept_column(n, LD, ldld, Wp, ldw, Dv, blk, colpanel, k0, q, st.npanel);
  __syncthreads();
  bk_panel_rows<false, 256>(n, LDs, ldld, Wps, ldw, perms, swps, blks, colpanels, pstarts, states, nb,
                            nbpiv, s, 0);
}

__global__ __launch_bounds__(1024) void k_bk_panel(int n, double* const* LDs, long ldld,
                                                   double* const* Wps, long ldw, int* const* perms,
                                                   int* const* swps, int* const* blks,
                                                   int* const* colpanels, int* const* pstarts,
                                                   FactorState* states, int nb, int nbpiv, int defer) {
  bk_panel_rows<true, 1024>(n, LDs, ldld, Wps, ldw, perms, swps, blks, colpanels, pstarts, states,
                            nb, nbpiv, blockIdx.x, defer);
}

// The pivoting panel with the panel's L in registers: every thread holds one row, a
// workgroup NT rows, and the rows of a shift are spread over a team of workgroups.
//
// What bounds it: the chain of pivot decisions.  A column of S is one multiply-add per
// panel column and thread (no memory but the raw column, loaded two columns ahead, through
// pointers known to be global: each barrier would wait for it otherwise); then the team
// agrees on the pivot.  A row interchange moves no data between threads: the two rows'
// threads exchange labels (the row a thread stands for), and L is written once, at the
// end, under the final labels: the pivot-free columns' L as well, formed from their W when
// the panel starts (a launch less, and L is written once).  A thread that becomes a pivot
// retires.  The W rows of the
// panel's own NB rows, which supply the multipliers of coming columns, are replicated in
// every workgroup's LDS.
//
// The team's exchanges.  Per column each workgroup publishes its largest entry and its row,
// the first one also the new W column of the panel's rows, and each one the W of its best
// row; a column that fails the first test needs one more exchange, the candidate column's
// maximum.  Words travel as relaxed agent-scope atomics, each with a tag in its upper half:
// a reader polls the words it needs until their tags are right, so an exchange is one trip to
// the coherence point and there is no flag, no fence and no reset (areas alternate by column;
// a workgroup writes an area again only after every other one has answered the column in
// between, and so has read it).  Data of S and W that another workgroup may read or write
// later go through the same kind of access, and a workgroup that wrote some waits for its
// stores before it publishes again.  Every element is formed by the operations, in the
// order, of bk_panel_rows, and maxima do not depend on the order, so the factors are the
// same bits whatever the split.
//
// Measured, all pivoting panels of a factorization: 17 shifts in lock step at order 4096
// (teams of up to 8) 18.9 ms from memory, 9.1 so; five shifts at order 1001 (one workgroup
// a shift) 2.5 and 1.0 ms, 1.6 us a column that needs a second test.  An exchange is 1.5 us
// of a column.
//
// The team must run at the same time.  Workgroups sign in to a roster; the one that
// completes the team closes it, and if the team is not complete within about 20 us
// (kTeamGather polls) the first one closes it for itself and runs the panel alone
// (bk_panel_rows) while late ones leave.  So no workgroup ever waits for one that is not
// running, whatever else occupies the device.  Every wait is bounded besides (wait_limit
// unsuccessful polls each); with a limit that a running team could reach, no team gathers
// (gather 0: the first one closes at once) and there is no wait to expire.
struct TeamArgs {
  int n;
  double* const* LDs;
  long ldld;
  double* const* Wps;
  long ldw;
  int* const* perms;
  int* const* swps;
  int* const* blks;
  int* const* colpanels;
  int* const* pstarts;
  FactorState* states;
  const double* const* auxs;
  unsigned long long* teams;
  unsigned* wait_err;
  unsigned wait_limit;
  unsigned gather;        // polls for the team to gather; 0: it never does
  int nb, nbpiv, groups;  // groups: workgroups of k_fast_panel
  int defer;              // whole panels that may be updated together (0: each by itself)
};

__device__ __forceinline__ double team_ld(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void team_st(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void team_post(unsigned long long* w, unsigned tag, double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  __hip_atomic_store(w, ((unsigned long long)tag << 32) | (b >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(w + 1, ((unsigned long long)tag << 32) | (b & 0xffffffffull), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long team_word(const unsigned long long* w) {
  return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double team_value(unsigned long long hi, unsigned long long lo) {
  return __longlong_as_double((long long)((hi << 32) | (lo & 0xffffffffull)));
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(v >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// The maximum over a row of 16 lanes, in each of them; over the wavefront, uniform.
__device__ __forceinline__ double max16(double x) {
  x = fmax(x, dpp_f64<0xB1>(x));
  x = fmax(x, dpp_f64<0x4E>(x));
  x = fmax(x, dpp_f64<0x141>(x));
  return fmax(x, dpp_f64<0x140>(x));
}
__device__ __forceinline__ double max_wave(double x) {
  x = max16(x);
  x = fmax(x, dpp_f64<0x142>(x));  // lane 15 of each row to the next row: rows 1 and 3 hold pairs
  return fmax(lane_f64(x, 31), lane_f64(x, 63));
}
// The smallest index among the lanes of `who` (not empty), uniform.
__device__ __forceinline__ int min_index(unsigned long long who, int idx) {
  int best = INT_MAX;
  while (who) {
    const int l = __ffsll((long long)who) - 1;
    who &= who - 1;
    best = min(best, __builtin_amdgcn_readlane(idx, l));
  }
  return best;
}
// A workgroup barrier that orders LDS only (stores to memory stay in flight).
__device__ __forceinline__ void barrier_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// a += w[0] l[0] + w[2] l[2] + ..., b += w[1] l[1] + ... in order, 16 products in all, where
// w[p] is lane p's value in each row of 16 lanes.  The multiply-adds take w by DPP row
// broadcast: no LDS read and no scalar move per product (from LDS, 16 wavefronts' broadcast
// reads of a panel row took longer than the arithmetic).  The s_nop covers a VALU write of w.
__device__ __forceinline__ void fmac16_pair(double& a, double& b, double w, const double* l) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %2, %3 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %2, %4 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %2, %5 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %2, %6 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %2, %7 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %2, %8 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %2, %9 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %2, %10 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %2, %11 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %2, %12 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %2, %13 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %2, %14 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %2, %15 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %2, %16 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %2, %17 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %2, %18 row_newbcast:15 row_mask:0xf bank_mask:0xf"
      : "+v"(a), "+v"(b)
      : "v"(w), "v"(l[0]), "v"(l[1]), "v"(l[2]), "v"(l[3]), "v"(l[4]), "v"(l[5]), "v"(l[6]), "v"(l[7]),
        "v"(l[8]), "v"(l[9]), "v"(l[10]), "v"(l[11]), "v"(l[12]), "v"(l[13]), "v"(l[14]), "v"(l[15]));
}
// The same as one chain.
__device__ __forceinline__ void fmac16(double& a, double w, const double* l) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %3 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %4 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %5 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %6 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %7 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %8 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %9 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %10 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %11 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %12 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %13 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %14 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %15 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %16 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %1, %17 row_newbcast:15 row_mask:0xf bank_mask:0xf"
      : "+v"(a)
      : "v"(w), "v"(l[0]), "v"(l[1]), "v"(l[2]), "v"(l[3]), "v"(l[4]), "v"(l[5]), "v"(l[6]), "v"(l[7]),
        "v"(l[8]), "v"(l[9]), "v"(l[10]), "v"(l[11]), "v"(l[12]), "v"(l[13]), "v"(l[14]), "v"(l[15]));
}

// l[j] = x for a uniform j: the register is found by a tree of scalar branches.
template <int N, int BASE = 0, int LEN = N>
__device__ __forceinline__ void put_panel(double (&l)[N], int j, double x) {
  if constexpr (LEN == 1) {
    l[BASE] = x;
    asm volatile("; L%0" ::"n"(BASE));  // (merged branches would index l, which then leaves the registers)
  } else {
    if (j < BASE + LEN / 2)
      put_panel<N, BASE, LEN / 2>(l, j, x);
    else
      put_panel<N, BASE + LEN / 2, LEN - LEN / 2>(l, j, x);
  }
}

// NB: columns the panel may hold; NT rows (threads) a workgroup.
template <int NB, int NT, bool TEAM>
__global__ __launch_bounds__(NT) void k_bk_team(TeamArgs a) {
  constexpr int NW = NT / 64, LW = NB + 1;
  __shared__ double Wt[NB * LW];  // W of the panel's rows: Wt[r * LW + p] = W(k0 + r, p)
  __shared__ double wim[NB + 1];  // the candidate row's W, then its entry of column k
  __shared__ double redv[2][NW];
  __shared__ int redi[2][NW];
  __shared__ double redc[NW];
  __shared__ double sh_v[2], sh_arr;
  __shared__ int sh_i, sh_own, sh_size, sh_rank, sh_js, sh_k0, sh_panel, sh_pend;
  const int s = blockIdx.y, tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = a.n, nb = a.nb;
  FactorState* st = a.states + s;
  unsigned long long* team = a.teams + (long)s * kTeamWords;
  // One thread reads the state and signs in, in this order: once the team is complete, the
  // first workgroup may finish the panel and write the state at any time.
  if (tid == 0) {
    const int k = st->k0 + st->kb, panel = st->npanel, pend = st->pend;
    const bool over = st->done || k >= n;  // (the state stays as the last panel left it)
    asm volatile("" ::"v"(k), "v"(panel), "v"(pend) : "memory");
    sh_k0 = k;
    sh_panel = panel;
    sh_pend = pend;
    int r = over ? -1 : 0, sz = 1;
    if (TEAM && !over) {
      const int need = (n - k + NT - 1) / NT;
      const unsigned closed = 0x80000000u;
      unsigned* roster = reinterpret_cast<unsigned*>(team);
      unsigned* size = reinterpret_cast<unsigned*>(team + 1);
      const unsigned old = __hip_atomic_fetch_add(roster, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      r = (int)(old & 0xffffu);
      sz = 0;
      if ((old & closed) || r >= need) {
        r = -1;
      } else if (r == need - 1 && a.gather) {
        if (!(__hip_atomic_fetch_or(roster, closed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & closed))
          __hip_atomic_store(size, (unsigned)need, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (r >= 0) {
        // the roster always closes: the first workgroup sees to it
        for (unsigned polls = 0;; ++polls) {
          sz = (int)__hip_atomic_load(size, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (sz) break;
          if (r == 0 && polls >= a.gather &&
              !(__hip_atomic_fetch_or(roster, closed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & closed)) {
            __hip_atomic_store(size, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sz = 1;
            break;
          }
          __builtin_amdgcn_s_sleep(8);
        }
      }
    }
    sh_rank = r;
    sh_size = sz;
  }
  __syncthreads();
  const int rank = __builtin_amdgcn_readfirstlane(sh_rank);
  const int k0 = __builtin_amdgcn_readfirstlane(sh_k0);
  const int P = __builtin_amdgcn_readfirstlane(sh_panel);
  const int pend = __builtin_amdgcn_readfirstlane(sh_pend);
  if (rank < 0) return;
  const int rem = n - k0;
  const int need = (rem + NT - 1) / NT;
  if (TEAM) {
    const int size = __builtin_amdgcn_readfirstlane(sh_size);
    if (rank >= size) return;
    if (size < need) {
      const double* Dv = global_ptr(a.auxs[s]);
      const int js = accepted_columns(Dv, nb, min(nb, rem), a.groups, &sh_js);
      for (int c = 0; c < js; ++c)
        accept_column(n, global_ptr(a.LDs[s]), a.ldld, global_ptr(a.Wps[s]) + pend * a.ldw, a.ldw, Dv,
                      global_ptr(a.blks[s]), global_ptr(a.colpanels[s]), k0, c, P);
      if (tid < 64) accept_state(st, Dv, js);
      __syncthreads();
      bk_panel_rows<true, NT>(n, a.LDs, a.ldld, a.Wps, a.ldw, a.perms, a.swps, a.blks, a.colpanels,
                              a.pstarts, a.states, nb, a.nbpiv, s, a.defer);
      return;
    }
  }
  const int G = TEAM ? need : 1;
  const bool multi = TEAM && G > 1;
  // areas by parity: column maxima (B) and candidate maxima (C), G headers of four words,
  // then 64 values of two words; and each workgroup's best row (R): 64 values, its entry of
  // the column, S(imax, imax)
  unsigned long long* mail = team + 64;
  constexpr int kArea = 4 * kTeamMax + 128;
  auto areaB = [&](int t) { return mail + (t & 1) * kArea; };
  auto areaC = [&](int t) { return mail + (2 + (t & 1)) * kArea; };
  auto areaR = [&](int t, int r) { return mail + 4 * kArea + ((t & 1) * kTeamMax + r) * kTeamRow; };
  double* LD = global_ptr(a.LDs[s]);
  double* Wp = global_ptr(a.Wps[s]) + pend * a.ldw;
  const long ld = a.ldld, ldw = a.ldw;
  auto ld_s = [&](const double* p) { return multi ? team_ld(p) : *p; };
  auto st_s = [&](double* p, double v) {
    if (multi)
      team_st(p, v);
    else
      *p = v;
  };
  int* perm = global_ptr(a.perms[s]);
  int* sw = global_ptr(a.swps[s]);
  int* blk = global_ptr(a.blks[s]);
  int* colpanel = global_ptr(a.colpanels[s]);
  const double* Dv = global_ptr(a.auxs[s]);
  const int jstart = accepted_columns(Dv, nb, min(nb, rem), a.groups, &sh_js);
  if (tid < NB) wim[tid] = tid < jstart ? 1.0 / Dv[tid] : 0.0;
  __syncthreads();

  // this thread's row: the row it stands for, the row it began as, its original row (which
  // travels with the label) and the columns of L to write, set when it becomes a pivot.
  // The panel's own rows are the first wavefront of the first workgroup, and
  // only those take labels from others while they live.
  const int first = k0 + rank * NT + tid;
  int lab = first < n ? first : INT_MAX;
  const int lc = min(first, n - 1);
  const int pv = perm[lc];
  int wlim = -1;
  double L[NB];  // -L (-0 where there is none: adding the product changes nothing)
#pragma unroll
  for (int p = 0; p < NB; ++p) L[p] = p < jstart ? -(Wp[lc + (long)p * ldw] * wim[p]) : -0.0;
  for (int e = tid; e < NB * LW; e += NT) {
    const int r = e / LW, p = e % LW;
    Wt[e] = (p < jstart && r >= jstart && k0 + r < n) ? Wp[(k0 + r) + (long)p * ldw] : 0.0;
  }
  // column c of S as it stands in memory (a row above c reads what is there: it will be a
  // pivot by then)
  auto column = [&](int c, double& x) {
    const double* p = LD + (long)min(c, n - 1) * ld;
    x = ld_s(p + min(lab, n - 1));
  };
  int j = jstart;
  double c0, c1;
  column(k0 + j, c0);
  column(k0 + j + 1, c1);
  const int jmax0 = rem <= nb ? rem : nb - 1;
  const int jmax = min(jmax0, jstart + a.nbpiv);
  long neg = 0, zer = 0, pos = 0;
  if (w == NW - 1) {  // the accepted columns' pivots (none is zero)
    const bool acc = lane < jstart;
    const bool negd = acc && Dv[min(lane, nb - 1)] < 0.0;
    neg = __popcll(__ballot(negd));
    pos = __popcll(__ballot(acc && !negd));
  }
  unsigned polls = 0;  // wavefront 0's unsuccessful polls of this wait; past the limit it goes on as it is
  auto expired = [&]() {
    if (polls++ < a.wait_limit) return false;
    __hip_atomic_store(a.wait_err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
  };
  bool stored = false;  // S entries written since the last publication
  __syncthreads();

  for (int t = 1; j < jmax; ++t) {
    const int k = k0 + j;
    const unsigned tag = ((unsigned)(P + 1) << 8) | (unsigned)t;
    // the raw columns after the next one, for the end of this step
    double c2, c3;
    column(k + 2, c2);
    column(k + 3, c3);
    const bool top = rank == 0 && w == 0 && lab >= k && lab < k0 + NB;
    // ---- column k of the Schur complement: even panel columns into av, odd ones into bv
    double av = c0, bv = 0.0;
#pragma unroll
    for (int g = 0; g < NB; g += 16)
      if (g < j) {
        // (entries from j on are being written by the panel rows' threads)
        const double x = Wt[j * LW + g + (lane & 15)];
        const double wm = g + (lane & 15) < j ? x : 0.0;
        fmac16_pair(av, bv, wm, L + g);
      }
    double v = -1.0;  // (a NaN is never the largest)
    int vi = INT_MAX;
    av += bv;
    const double x = fabs(av);
    const bool in = lab > k && lab < n;
    if (in && (x > v || (x == v && lab < vi))) {
      v = x;
      vi = lab;
    }
    const double vm = max_wave(v);
    const int im = vm > -1.0 ? min_index(__ballot(v == vm), vi) : INT_MAX;
    // this wavefront's best row of W (written by this wavefront): the candidate's, if it wins
    const double wv = (im < n && lane < j) ? ld_s(Wp + im + (long)lane * ldw) : 0.0;
    if (lane == 0) {
      redv[t & 1][w] = vm;
      redi[t & 1][w] = im;
    }
    if (top) Wt[(lab - k0) * LW + j] = av;
    if (stored) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    barrier_lds();
    double colmax;
    int imax, own = 0;
    {
      const double x = lane < NW ? redv[t & 1][lane] : -1.0;
      const int xi = lane < NW ? redi[t & 1][lane] : INT_MAX;
      colmax = lane_f64(max16(x), 0);
      imax = colmax > -1.0 ? min_index(__ballot(lane < NW && x == colmax), xi) : INT_MAX;
    }
    if (multi && w == 0) {
      unsigned long long* ar = areaB(t);
      if (lane == 0) {
        team_post(ar + 4 * rank, tag, colmax);
        __hip_atomic_store(ar + 4 * rank + 2, ((unsigned long long)tag << 32) | (unsigned)imax,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (rank == 0 && lane < NB) team_post(ar + 4 * kTeamMax + 2 * lane, tag, Wt[lane * LW + j]);
    }
    if (imax < n && im == imax) {  // uniform: this wavefront holds the workgroup's best row
      const unsigned long long who = __ballot(lab == imax);
      const double ev = who ? lane_f64(av, __ffsll((long long)who) - 1) : 0.0;
      if (lane < NB) wim[lane] = wv;
      if (lane == 0) wim[NB] = ev;
      if (multi) {
        unsigned long long* ar = areaR(t, rank);
        if (lane < NB) team_post(ar + 2 * lane, tag, wv);
        if (lane == 0) team_post(ar + 128, tag, ev);
      }
    }
    if (multi) {
      if (w == 0) {
        const unsigned long long* ar = areaB(t);
        unsigned long long h0 = 0, h1 = 0, h2 = 0, t0 = 0, t1 = 0;
        const bool wh = lane < G, wt = rank > 0 && lane < NB;
        polls = 0;
        for (;;) {
          if (wh && ((h0 >> 32) != tag || (h1 >> 32) != tag || (h2 >> 32) != tag)) {
            h0 = team_word(ar + 4 * lane);
            h1 = team_word(ar + 4 * lane + 1);
            h2 = team_word(ar + 4 * lane + 2);
          }
          if (wt && ((t0 >> 32) != tag || (t1 >> 32) != tag)) {
            t0 = team_word(ar + 4 * kTeamMax + 2 * lane);
            t1 = team_word(ar + 4 * kTeamMax + 2 * lane + 1);
          }
          const bool ok = (!wh || ((h0 >> 32) == tag && (h1 >> 32) == tag && (h2 >> 32) == tag)) &&
                          (!wt || ((t0 >> 32) == tag && (t1 >> 32) == tag));
          if (__ballot(!ok) == 0 || expired()) break;
        }
        const double x = wh ? team_value(h0, h1) : -1.0;
        const int xi = wh ? (int)(unsigned)h2 : INT_MAX;
        colmax = max_wave(x);
        const unsigned long long who = __ballot(wh && x == colmax);
        imax = colmax > -1.0 && who ? min_index(who, xi) : INT_MAX;
        const unsigned long long mine = __ballot(wh && x == colmax && xi == imax);
        if (wt) Wt[lane * LW + j] = team_value(t0, t1);
        // (a wait that expired may leave a stale index: no access may follow it)
        if (imax <= k || imax >= n) colmax = -1.0;
        if (lane == 0) {
          sh_v[0] = colmax;
          sh_i = imax;
          sh_own = mine ? __ffsll((long long)mine) - 1 : -1;
        }
      }
      barrier_lds();
      colmax = sh_v[0];
      imax = __builtin_amdgcn_readfirstlane(sh_i);
      own = __builtin_amdgcn_readfirstlane(sh_own);
    }
    const double akk = Wt[j * LW + j], absakk = fabs(akk);
    colmax = colmax > 0.0 ? colmax : 0.0;
    int kstep = 1, kp = k;
    double b = 0.0, arr = 0.0;
    const bool cand = absakk < kBkAlpha * colmax;  // uniform over the team
    if (cand) {
      // ---- candidate column imax of the Schur complement
      const int i = min(lab, n - 1);
      b = ld_s(i < imax ? LD + imax + (long)i * ld : LD + i + (long)imax * ld);
      if (multi && rank != own && w == 0) {
        const unsigned long long* ar = areaR(t, max(own, 0));
        unsigned long long t0 = 0, t1 = 0, e0 = 0, e1 = 0;
        const bool wt = lane < NB, we = lane == 0;
        polls = 0;
        for (;;) {
          if (wt && ((t0 >> 32) != tag || (t1 >> 32) != tag)) {
            t0 = team_word(ar + 2 * lane);
            t1 = team_word(ar + 2 * lane + 1);
          }
          if (we && ((e0 >> 32) != tag || (e1 >> 32) != tag)) {
            e0 = team_word(ar + 128);
            e1 = team_word(ar + 129);
          }
          const bool ok = (!wt || ((t0 >> 32) == tag && (t1 >> 32) == tag)) &&
                          (!we || ((e0 >> 32) == tag && (e1 >> 32) == tag));
          if (__ballot(!ok) == 0 || expired()) break;
        }
        if (wt) wim[lane] = team_value(t0, t1);
        if (we) wim[NB] = team_value(e0, e1);
      }
      barrier_lds();
#pragma unroll
      for (int g = 0; g < NB; g += 16)
        if (g < j) {
          const double wm = wim[g + (lane & 15)];  // (zero from j on)
          fmac16(b, wm, L + g);
        }
      double x = -1.0;
      const double y = fabs(b);
      if (lab >= k && lab < n && lab != imax && y > x) x = y;
      if (lab == imax) sh_arr = b;
      x = max_wave(x);
      if (lane == 0) redc[w] = x;
      if (top) Wt[(lab - k0) * LW + j + 1] = b;
      barrier_lds();
      double rowmax = lane_f64(max16(lane < NW ? redc[lane] : -1.0), 0);
      arr = sh_arr;
      if (multi) {
        if (w == 0) {
          unsigned long long* ar = areaC(t);
          if (lane == 0) {
            team_post(ar + 4 * rank, tag, rowmax);
            if (rank == own) team_post(areaR(t, rank) + 130, tag, arr);
          }
          if (rank == 0 && lane < NB) team_post(ar + 4 * kTeamMax + 2 * lane, tag, Wt[lane * LW + j + 1]);
          unsigned long long h0 = 0, h1 = 0, t0 = 0, t1 = 0, e0 = 0, e1 = 0;
          const bool wh = lane < G, wt = rank > 0 && lane < NB, we = lane == 0 && rank != own;
          polls = 0;
          for (;;) {
            if (wh && ((h0 >> 32) != tag || (h1 >> 32) != tag)) {
              h0 = team_word(ar + 4 * lane);
              h1 = team_word(ar + 4 * lane + 1);
            }
            if (wt && ((t0 >> 32) != tag || (t1 >> 32) != tag)) {
              t0 = team_word(ar + 4 * kTeamMax + 2 * lane);
              t1 = team_word(ar + 4 * kTeamMax + 2 * lane + 1);
            }
            if (we && ((e0 >> 32) != tag || (e1 >> 32) != tag)) {
              e0 = team_word(areaR(t, max(own, 0)) + 130);
              e1 = team_word(areaR(t, max(own, 0)) + 131);
            }
            const bool ok = (!wh || ((h0 >> 32) == tag && (h1 >> 32) == tag)) &&
                            (!wt || ((t0 >> 32) == tag && (t1 >> 32) == tag)) &&
                            (!we || ((e0 >> 32) == tag && (e1 >> 32) == tag));
            if (__ballot(!ok) == 0 || expired()) break;
          }
          const double y = max_wave(wh ? team_value(h0, h1) : -1.0);
          if (wt) Wt[lane * LW + j + 1] = team_value(t0, t1);
          if (lane == 0) {
            sh_v[1] = y;
            if (we) sh_arr = team_value(e0, e1);
          }
        }
        barrier_lds();
        rowmax = sh_v[1];
        arr = sh_arr;
      }
      if (absakk * rowmax >= kBkAlpha * colmax * colmax) {
        kstep = 1;
        kp = k;
      } else if (fabs(arr) >= kBkAlpha * rowmax) {
        kstep = 1;
        kp = imax;
      } else {
        kstep = 2;
        kp = imax;
      }
    }
    const int kk = k + kstep - 1;
    const bool swap = kp != kk;
    // ---- pivot, its multipliers, and the column(s) of W under the final labels
    double d11, d21 = 0.0, d22 = 0.0;
    double l1, l2;
    if (kstep == 1) {
      d11 = swap ? arr : akk;
      const double dinv = d11 != 0.0 ? 1.0 / d11 : 0.0;
      if (swap) av = b;
      l1 = av * dinv;
      l2 = 0.0;
    } else {
      d11 = akk;
      d21 = wim[NB];
      d22 = arr;
      const double aa = d11 / d21, gg = d22 / d21;
      const double tt = 1.0 / (d21 * (aa * gg - 1.0));
      l1 = tt * (gg * av - b);
      l2 = tt * (aa * b - av);
    }
    if (swap) {
      // symmetric interchange kk <-> kp of S: kk becomes a pivot column, so only row and
      // column kp need column kk's entries.  The raw columns at hand follow: column kp is
      // column kk as it was, and row kp holds column kk's entry of the column's own row
      // (whose thread is in the same wavefront).
      const double rawk = kstep == 1 ? c0 : c1;  // column kk as it was
      if (lab > kk && lab < n && lab != kp)
        st_s(lab > kp ? LD + lab + (long)kp * ld : LD + kp + (long)lab * ld, rawk);
      if (lab == kk) st_s(LD + kp + (long)kp * ld, rawk);
      // W of row kk moves to row kp
      if (rank == 0 && w == 0 && lane < j) st_s(Wp + kp + (long)lane * ldw, Wt[(kk - k0) * LW + lane]);
      const bool taker = lab == kk;  // the panel row's thread that takes label kp
      auto follow = [&](int c, double& x) {
        if (c >= n || c >= k0 + NB) return;
        if (c == kp) {
          x = rawk;
        } else if (c < kp && rank == 0 && w == 0) {
          const unsigned long long src = __ballot(lab == c);
          const double y = src ? lane_f64(rawk, __ffsll((long long)src) - 1) : 0.0;
          if (taker) x = y;
        }
      };
      if (kstep == 1) follow(k + 1, c1);
      follow(k + 2, c2);
      follow(k + 3, c3);
      // the two rows' threads exchange labels
      const int o = lab;
      lab = o == kk ? kp : (o == kp ? kk : o);
    }
    stored = swap;
    const bool below = lab > kk && lab < n;
    if (below) {
      st_s(Wp + lab + (long)j * ldw, av);
      if (kstep == 2) st_s(Wp + lab + (long)(j + 1) * ldw, b);
    }
    if (lab >= k && lab <= kk) wlim = j;  // this row became a pivot
    // (rows that are done take values that nothing reads)
    put_panel<NB>(L, j, -l1);
    if (kstep == 2) put_panel<NB>(L, j + 1, -l2);
    c0 = kstep == 1 ? c1 : c2;
    c1 = kstep == 1 ? c2 : c3;
    // ---- every workgroup's copy of the panel rows' W
    if (cand) {
      if (w == 0) {
        if (swap && kp < k0 + NB) {  // row kp takes row kk's W
          const double x0 = Wt[(kk - k0) * LW + min(lane, NB - 1)];
          if (lane < NB && lane <= j + 1) Wt[(kp - k0) * LW + lane] = x0;
        }
        __builtin_amdgcn_wave_barrier();
        if (kstep == 1 && lane < NB) {
          const double x1 = Wt[lane * LW + j + 1];
          if (swap) Wt[lane * LW + j] = x1;
          Wt[lane * LW + j + 1] = 0.0;
        }
      }
      barrier_lds();
    }
    if (rank == 0 && tid == NT - 1) {
      sw[k] = kstep == 1 ? kp : k;
      LD[k + (long)k * ld] = d11;
      colpanel[k] = P;
      if (kstep == 1) {
        blk[k] = 1;
        if (d11 < 0.0)
          ++neg;
        else if (d11 > 0.0)
          ++pos;
        else
          ++zer;
      } else {
        sw[k + 1] = kp;
        LD[k + 1 + (long)k * ld] = d21;
        LD[k + 1 + (long)(k + 1) * ld] = d22;
        blk[k] = 2;
        blk[k + 1] = 0;
        colpanel[k + 1] = P;
        const double det = d11 * d22 - d21 * d21;
        const double tr = d11 + d22;
        if (det < 0.0) {
          ++neg;
          ++pos;
        } else if (det > 0.0) {
          if (tr < 0.0)
            neg += 2;
          else
            pos += 2;
        } else {
          ++zer;
          if (tr < 0.0)
            ++neg;
          else if (tr > 0.0)
            ++pos;
          else
            ++zer;
        }
      }
    }
    j += kstep;
  }
  // ---- L and the permutation under the final labels
  if (lab < n) {
    const bool accepted = lab < k0 + jstart;  // a pivot of the accepted columns
    const int lim = accepted ? lab - k0 : (wlim >= 0 ? wlim : j);
#pragma unroll
    for (int p = 0; p < NB; ++p)
      if (p < lim) LD[lab + (long)(k0 + p) * ld] = -L[p];
    if (accepted) {
      LD[lab + (long)lab * ld] = Dv[lim];
      blk[lab] = 1;
      colpanel[lab] = P;
    }
    if (lab != first) perm[lab] = pv;
  }
  if (rank == 0 && tid == NT - 1) {
    panel_done(st, n, nb, min(nb, rem), k0, j, jstart, P, a.defer);
    st->neg += neg;
    st->zero += zer;
    st->pos += pos;
    global_ptr(a.pstarts[s])[P] = k0;
  }
}

// C22 -= L21 W21^T on the lower triangle of the trailing matrix of every shift.
// 64x64 tile per 256-thread workgroup; each wavefront owns a 32x32 quarter as
// 2x2 v_mfma_f64_16x16x4 blocks.  The A operand is -W (tile columns), the B
// operand is L (tile rows), so that accumulator element r of lane l is
// C(i0 + l%16, j0 + l/16 + 4r): sixteen consecutive rows of one column per
// register.  The tile of C is loaded straight into the accumulators, every
// operand of the panel's K <= 64 columns is issued from global memory up front
// (no LDS, no barrier: occupancy is bounded by registers only), and the
// accumulators are stored back: one read and one write of C per panel.
__global__ __launch_bounds__(256) void k_trailing_update(int n, double* const* LDs, long ldld,
                                                         double* const* Wps, long ldw,
                                                         const FactorState* states) {
  constexpr int KS = kMaxNb / 4;  // k-steps of 4
  const int s = blockIdx.y;
  const int k0 = states[s].k0, kb = states[s].kb;
  const int k1 = k0 + kb;
  if (kb <= 0 || k1 >= n) return;
  const int T = (n - k1 + 63) / 64;
  const int lin = blockIdx.x;
  if (lin >= T * (T + 1) / 2) return;
  int ti = (int)((sqrt(8.0 * lin + 1.0) - 1.0) * 0.5);
  while (ti * (ti + 1) / 2 > lin) --ti;
  while ((ti + 1) * (ti + 2) / 2 <= lin) ++ti;
  const int tj = lin - ti * (ti + 1) / 2;
  const int row0 = k1 + ti * 64, col0 = k1 + tj * 64;
  double* LD = global_ptr(LDs[s]);
  const double* Wp = global_ptr(Wps[s]);
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int wi = (w & 1) * 32, wj = (w >> 1) * 32;
  const int lr = l & 15, lk = l >> 4;
  const int nks = (kb + 3) >> 2;
  // tile rows / columns of this lane (clamped for the loads, masked for the stores)
  int ri[2], cj[2];
#pragma unroll
  for (int x = 0; x < 2; ++x) ri[x] = row0 + wi + 16 * x + lr;
#pragma unroll
  for (int y = 0; y < 2; ++y) cj[y] = col0 + wj + 16 * y + lr;
  d4 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = min(ri[x], n - 1), j = min(col0 + wj + 16 * y + lk + 4 * r, n - 1);
        acc[x][y][r] = LD[i + (long)j * ldld];
      }
  // operands in chunks of 4 k-steps, double-buffered: the loads of chunk c + 1 are
  // in flight while chunk c feeds the MFMAs (registers stay low enough for several
  // resident wavefronts per SIMD)
  constexpr int CK = 4;
  const int nch = (nks + CK - 1) / CK;
  double lop[2][CK][2], wop[2][CK][2];
  auto load_chunk = [&](int ch, double (&lb)[CK][2], double (&wb)[CK][2]) {
#pragma unroll
    for (int u = 0; u < CK; ++u) {
      const int k = 4 * (CK * ch + u) + lk;
      const bool kv = k < kb;
      const int kc = kv ? k : 0;
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const double v = LD[min(ri[x], n - 1) + (long)(k0 + kc) * ldld];
        lb[u][x] = kv ? v : 0.0;
      }
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        const double v = Wp[min(cj[y], n - 1) + (long)kc * ldw];
        wb[u][y] = kv ? -v : 0.0;
      }
    }
  };
  auto mfma_chunk = [&](const double (&lb)[CK][2], const double (&wb)[CK][2]) {
#pragma unroll
    for (int u = 0; u < CK; ++u)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = mfma16x16x4(wb[u][y], lb[u][x], acc[x][y]);
  };
  load_chunk(0, lop[0], wop[0]);
#pragma unroll
  for (int ch = 0; ch < KS / CK; ch += 2) {
    if (ch < nch) {
      if (ch + 1 < nch) load_chunk(ch + 1, lop[1], wop[1]);
      mfma_chunk(lop[0], wop[0]);
    }
    if (ch + 1 < nch) {
      if (ch + 2 < nch) load_chunk(ch + 2, lop[0], wop[0]);
      mfma_chunk(lop[1], wop[1]);
    }
  }
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int i = ri[x];
#pragma unroll
    for (int y = 0; y < 2; ++y) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int jc = col0 + wj + 16 * y + lk + 4 * r;
        if (i < n && jc < n && i >= jc) LD[i + (long)jc * ldld] = acc[x][y][r];
      }
    }
  }
}

// The same update on 128x128 tiles for large trailing matrices, one 1024-thread
// workgroup per tile.  Each of the 16 wavefronts owns a 32x32 block of the tile as
// 2x2 v_mfma_f64_16x16x4 blocks, so a wavefront needs at most 64 registers (asked for) and
// a CU keeps two workgroups (eight wavefronts per SIMD) in flight; the C tile is read and
// written once per 128x128.  The operand panels of the tile (128 rows of L and 128
// rows of W, 16 k-columns per chunk) are fetched once per workgroup with coalesced
// 1 KB column runs into double-buffered LDS (70 KB), and the next chunk is in
// flight while the wavefronts run the current one's MFMAs: nothing touches the fetched
// values before they go to LDS (a sign or a select there waits for them, 30 TF/s).
// Layout per chunk and operand: [k][row], rows padded to 136 doubles (132 and 144: 2% more
// per update of many columns).
//
// What bounds it: at 64 columns the C stream, 2 x 8 bytes per 128 flops (4.0 TB/s of the
// 4.6 a copy reaches).  So a panel that the pivot-free path accepted whole updates the next
// panel's columns only, one column of tiles, and up to kDeferPanels of them go into C
// together; then the matrix instructions bound it (50 TF/s; 68 without the staging).  When
// a panel is not whole, those waiting are caught up first (`auxs` given: the panel's masks
// decide), since pivoting may look at any column.  The order of the sums is the same either
// way, so the factors are the same bits.  17 shifts of order 4096, 384 columns: 1.75 ms, in
// six updates of 64 3.2.
constexpr int kUpdK = 16;           // k-columns per staged chunk
constexpr int kUpdLd = 128 + 8;     // padded row count per k-column
template <bool STREAM>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8))) void k_trailing_update_lds(
    int n, double* const* LDs, long ldld, double* const* Wps, long ldw, const FactorState* states,
    const double* const* auxs, int nb, int groups) {
  constexpr int TB = 128;
  __shared__ double sL[2][kUpdK * kUpdLd];
  __shared__ double sW[2][kUpdK * kUpdLd];
  __shared__ int sh;
  const int s = blockIdx.y;
  const FactorState st = states[s];
  int k0 = st.u_k0, kb = st.u_kb, w0 = st.u_w0, k1 = st.u_c0, c1 = st.u_c1;
  int nbe = 0;
  if (auxs) {  // the panel before, for the columns past the present one's
    k1 = st.k0 + st.kb;
    if (st.done || st.pend == 0 || k1 >= n) return;
    nbe = min(nb, n - k1);
    k0 = k1 - st.pend;
    kb = st.pend;
    w0 = 0;
    k1 += nbe;
    c1 = n;
  }
  if (kb <= 0 || k1 >= n) return;
  const int T = (n - k1 + TB - 1) / TB;
  const int lin = blockIdx.x;
  const bool strip = c1 - k1 <= TB;  // one column of tiles
  if (lin >= (strip ? T : T * (T + 1) / 2)) return;
  if (auxs && accepted_columns(global_ptr(auxs[s]), nb, nbe, groups, &sh) == nbe) return;
  int ti = (int)((sqrt(8.0 * lin + 1.0) - 1.0) * 0.5);
  while (ti * (ti + 1) / 2 > lin) --ti;
  while ((ti + 1) * (ti + 2) / 2 <= lin) ++ti;
  int tj = lin - ti * (ti + 1) / 2;
  if (strip) {
    ti = lin;
    tj = 0;
  }
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int wi = (w & 3) * 32, wj = (w >> 2) * 32;
  // on a diagonal tile the blocks above the diagonal store nothing, but their
  // wavefronts still help stage the operands
  const int row0 = k1 + ti * TB, col0 = k1 + tj * TB;
  const bool active = !(ti == tj && wi + 31 < wj) && col0 + wj < c1;
  double* LD = global_ptr(LDs[s]);
  const double* Wp = global_ptr(Wps[s]) + w0 * ldw;
  const int lr = l & 15, lk = l >> 4;
  const int nch = (kb + kUpdK - 1) / kUpdK;  // staged chunks
  // staging: thread t fetches row (t % 128) of columns (t / 128) + 8j, j < 2
  const int sr = tid & 127, sc = w >> 1;
  const unsigned lrow = min(row0 + sr, n - 1), wrow = min(col0 + sr, n - 1);
  double stL[kUpdK / 8], stW[kUpdK / 8];
  // (a column past kb is the last one again, and zero when it goes to LDS: the loads are not
  // touched before the MFMAs of the chunk at hand)
  auto fetch = [&](int ch) {
#pragma unroll
    for (int j = 0; j < kUpdK / 8; ++j) {
      const int k = min(ch * kUpdK + sc + 8 * j, kb - 1);
      stL[j] = (LD + (long)(k0 + k) * ldld)[lrow];
      stW[j] = (Wp + (long)k * ldw)[wrow];
    }
  };
  auto stage = [&](int buf, int ch) {
#pragma unroll
    for (int j = 0; j < kUpdK / 8; ++j) {
      const bool kv = ch * kUpdK + sc + 8 * j < kb;
      sL[buf][(sc + 8 * j) * kUpdLd + sr] = kv ? stL[j] : 0.0;
      sW[buf][(sc + 8 * j) * kUpdLd + sr] = kv ? -stW[j] : 0.0;
    }
  };
  fetch(0);
  d4 acc[2][2];
  if (active) {
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int i = min(row0 + wi + 16 * x + lr, n - 1);
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int j = min(col0 + wj + 16 * y + lk + 4 * r, n - 1);
          acc[x][y][r] = STREAM ? __builtin_nontemporal_load(LD + i + (long)j * ldld)
                                : LD[i + (long)j * ldld];
        }
    }
  }
  stage(0, 0);
  __syncthreads();
  for (int ch = 0; ch < nch; ++ch) {
    const int buf = ch & 1;
    if (ch + 1 < nch) fetch(ch + 1);
    if (active) {
      const double* L0 = sL[buf] + wi + lr;
      const double* W0 = sW[buf] + wj + lr;
      // (k-steps past kb meet zeros)
#pragma unroll
      for (int u = 0; u < kUpdK / 4; ++u) {
        const int kk = (4 * u + lk) * kUpdLd;
        double lo[2], wo[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) lo[x] = L0[kk + 16 * x];
#pragma unroll
        for (int y = 0; y < 2; ++y) wo[y] = W0[kk + 16 * y];
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y) acc[x][y] = mfma16x16x4(wo[y], lo[x], acc[x][y]);
      }
    }
    if (ch + 1 < nch) {
      stage(buf ^ 1, ch + 1);
      __syncthreads();
    }
  }
  if (!active) return;
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int i = row0 + wi + 16 * x + lr;
#pragma unroll
    for (int y = 0; y < 2; ++y) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int jc = col0 + wj + 16 * y + lk + 4 * r;
        if (i < n && jc < c1 && i >= jc) {
          if (STREAM)
            __builtin_nontemporal_store(acc[x][y][r], LD + i + (long)jc * ldld);
          else
            LD[i + (long)jc * ldld] = acc[x][y][r];
        }
      }
    }
  }
}

// Suffix compositions of the interchanges: for the panel ending at e, Q_e[v] is
// the final row of the entry found at row v (v >= e) when that panel finished.
//
// What bounds it: the interchanges are a chain, from the last column back.  One wavefront
// takes a panel's (at most 64) at once, lane l that of column t = hi - l with row p: in order
// each does q[t] = q[p], q[p] = t (q[t] is t until then).  A lane reads q[p] as it was before
// the panel unless an earlier one of its panel wrote that entry, and those are played
// through in registers, columns without interchange left out.  Order 4096, 17 shifts:
// 412 us by one thread, 79 so; order 1001: 100 and 27; order 200: 18 and 5.
__global__ __launch_bounds__(1024) void k_perm_suffix(int n, const int* const* swps,
                                                      const int* const* pstarts,
                                                      const FactorState* states, int* const* snaps) {
  extern __shared__ int q[];
  const int s = blockIdx.x, lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int* sw = global_ptr(swps[s]);
  const int* pstart = global_ptr(pstarts[s]);
  int* snap = global_ptr(snaps[s]);
  const int np = __builtin_amdgcn_readfirstlane(states[s].npanel);
  for (int v = threadIdx.x; v < n; v += blockDim.x) q[v] = v;
  int hi = n - 1;  // the panel's last column
  int e = np > 1 ? __builtin_amdgcn_readfirstlane(pstart[np - 1]) : 0;
  int p = sw[max(hi - lane, 0)];
  __syncthreads();
  for (int P = np - 1; P >= 1; --P) {
    const int e1 = P > 1 ? __builtin_amdgcn_readfirstlane(pstart[P - 1]) : 0;  // the panel before
    const int p1 = sw[max(e - 1 - lane, 0)];
    if (w == 0) {
      const int t = hi - lane;
      const bool moves = t >= e && p != t;
      int val = moves ? q[p] : t;
      bool last = moves;  // no later column of the panel has the same row
      for (unsigned long long m = __ballot(moves); m; m &= m - 1) {
        const int l = __ffsll((long long)m) - 1;
        const int tl = hi - l, pl = __builtin_amdgcn_readlane(p, l), vl = __builtin_amdgcn_readlane(val, l);
        const bool later = moves && lane > l;
        if (__ballot(later && p == pl) && lane == l) last = false;
        if (later && p == pl) val = tl;
        if (later && p == tl) val = vl;
      }
      if (moves) q[t] = val;
      __builtin_amdgcn_wave_barrier();
      if (last) q[p] = t;
    }
    __syncthreads();
    for (int v = e + threadIdx.x; v < n; v += blockDim.x) snap[(long)(P - 1) * n + v] = q[v];
    hi = e - 1;
    e = e1;
    p = p1;
    __syncthreads();
  }
}

// Apply the later panels' interchanges to the rows of each finished L column.
// The column is staged in LDS (up to n doubles), which allows one workgroup per
// CU: 1024 threads, each with four rows' loads in flight per round.
__global__ __launch_bounds__(1024) void k_left_gather(int n, double* const* LDs, long ldld,
                                                      const int* const* colpanels,
                                                      const int* const* pstarts,
                                                      const FactorState* states,
                                                      const int* const* snaps) {
  extern __shared__ double col[];
  const int c = blockIdx.x, s = blockIdx.y;
  const int P = global_ptr(colpanels[s])[c];
  const int np = states[s].npanel;
  if (P + 1 >= np) return;
  const int e = global_ptr(pstarts[s])[P + 1];
  if (e >= n) return;
  double* LD = global_ptr(LDs[s] + (long)c * ldld);
  const int* q = global_ptr(snaps[s] + (long)P * n);
  constexpr int U = 4;
  for (int v0 = e + threadIdx.x; v0 < n; v0 += U * 1024) {
    double x[U];
    int t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = v0 + u * 1024;
      x[u] = v < n ? LD[v] : 0.0;
      t[u] = v < n ? q[v] : e;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (v0 + u * 1024 < n) col[t[u] - e] = x[u];
  }
  __syncthreads();
  for (int i = e + threadIdx.x; i < n; i += 1024) LD[i] = col[i - e];
}

// ipiv in the documented format and the inertia triple of every shift.  A factorization that
// a wait's expiry spoiled, or whose steps ended before its columns, gets kSpoiledInertia or
// kUnfinishedInertia for a count, which the host reads with the inertias (check_factor).
__global__ __launch_bounds__(256) void k_factor_finalize(int n, const int* const* perms,
                                                         const int* const* blks, int* const* ipivs,
                                                         const FactorState* states,
                                                         int64_t* inertia, const unsigned* wait_err) {
  const int s = blockIdx.y;
  const int* perm = global_ptr(perms[s]);
  const int* blk = global_ptr(blks[s]);
  int* ipiv = global_ptr(ipivs[s]);
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const bool two = (blk[i] == 2) || (blk[i] == 0);
    ipiv[i] = two ? -(perm[i] + 1) : perm[i];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    inertia[3 * s + 0] = *wait_err ? kSpoiledInertia : (states[s].done ? states[s].neg : kUnfinishedInertia);
    inertia[3 * s + 1] = states[s].zero;
    inertia[3 * s + 2] = states[s].pos;
  }
}

// ------------------------------------------------------------------ host side

void factor_prepare() {
  static std::once_flag attr_set;
  std::call_once(attr_set, [] {
    SL_HIP(hipFuncSetAttribute((const void*)k_left_gather,
                               hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    SL_HIP(hipFuncSetAttribute((const void*)k_perm_suffix,
                               hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
  });
}

void factor_shift_form_launch(const FactorPlan& fp, hipStream_t st) {
  if (fp.nshift <= 0 || fp.n <= 0) return;
  SL_LAUNCH(k_shift_form, dim3(fp.n), dim3(256), 0, st, fp.n, fp.nshift, fp.A, fp.lda, fp.B, fp.ldb,
            fp.d_sigmas, fp.d_LD, fp.ldld);
  SL_LAUNCH_CHECK();
}

void factor_launch(const FactorPlan& fp, hipStream_t st) {
  factor_shift_form_launch(fp, st);
  factor_steps_launch(fp, st, true);
}

// The plan of shifts [s0, s0 + cnt): every per-shift device table offset.
static FactorPlan factor_subplan(const FactorPlan& fp, int s0, int cnt) {
  FactorPlan f = fp;
  f.nshift = cnt;
  f.d_sigmas = fp.d_sigmas ? fp.d_sigmas + s0 : nullptr;
  f.d_LD = fp.d_LD + s0;
  f.d_W = fp.d_W + s0;
  f.d_perm = fp.d_perm + s0;
  f.d_sw = fp.d_sw + s0;
  f.d_blk = fp.d_blk + s0;
  f.d_colpanel = fp.d_colpanel + s0;
  f.d_pstart = fp.d_pstart + s0;
  f.d_snap = fp.d_snap + s0;
  f.d_ipiv = fp.d_ipiv + s0;
  f.d_state = fp.d_state + s0;
  f.d_inertia = fp.d_inertia + 3 * (size_t)s0;
  f.d_aux = fp.d_aux ? fp.d_aux + s0 : nullptr;
  f.d_team = fp.d_team + (size_t)s0 * kTeamWords;
  return f;
}

// The pivoting panel of every shift.  rem_max bounds the rows of the least advanced shift;
// a team per shift must fit the device at once (seven eighths of it, shared by the shift
// groups), otherwise one workgroup a shift runs the panel from memory.
static bool panel_team(const FactorPlan& fp, long rem_max, long& need) {
  need = rem_max <= (fp.nb > 32 ? 512 : 1024) ? 1 : ceil_div(rem_max, 512);
  return fp.pivot &&
         (need <= 1 || (need <= kTeamMax && need * fp.nshift <= (long)fp.cus * 7 / 8 / fp.groups));
}

static void panel_launch(const FactorPlan& fp, hipStream_t st, long rem_max, int nbpiv, int groups, int defer) {
  const int n = fp.n, S = fp.nshift, nb = fp.nb;
  if (!fp.pivot) return;  // (k_fast_commit ends the panel)
  long need;
  if (panel_team(fp, rem_max, need)) {
    TeamArgs a{n, fp.d_LD, fp.ldld, fp.d_W, fp.ldw, fp.d_perm, fp.d_sw, fp.d_blk, fp.d_colpanel,
               fp.d_pstart, fp.d_state, fp.d_aux, fp.d_team, fp.wait_err, fp.wait_limit,
               fp.wait_limit < kTeamMinLimit ? 0u : kTeamGather, nb, nbpiv, groups, defer};
    // As few threads as hold the rows: a column's reductions, tests and barriers cost every
    // wavefront the same instructions, so a SIMD's wavefronts take turns at them.  Five
    // shifts at order 1001, all panels: 1.52 ms with 1024 threads to the end, 1.04 so.
    const dim3 team(need > 1 ? (unsigned)need : 1u, S);
    if (need > 1) {
      if (nb > 32)
        SL_LAUNCH((k_bk_team<64, 512, true>), team, dim3(512), 0, st, a);
      else
        SL_LAUNCH((k_bk_team<32, 512, true>), team, dim3(512), 0, st, a);
    } else if (rem_max <= 256) {
      if (nb > 32)
        SL_LAUNCH((k_bk_team<64, 256, false>), team, dim3(256), 0, st, a);
      else
        SL_LAUNCH((k_bk_team<32, 256, false>), team, dim3(256), 0, st, a);
    } else if (rem_max <= 512) {
      if (nb > 32)
        SL_LAUNCH((k_bk_team<64, 512, false>), team, dim3(512), 0, st, a);
      else
        SL_LAUNCH((k_bk_team<32, 512, false>), team, dim3(512), 0, st, a);
    } else {
      SL_LAUNCH((k_bk_team<32, 1024, false>), team, dim3(1024), 0, st, a);
    }
  } else {
    SL_LAUNCH(k_bk_panel, dim3(S), dim3(1024), 0, st, n, fp.d_LD, fp.ldld, fp.d_W, fp.ldw,
              fp.d_perm, fp.d_sw, fp.d_blk, fp.d_colpanel, fp.d_pstart, fp.d_state, nb, nbpiv, defer);
  }
  SL_LAUNCH_CHECK();
}

// The update on 128x128 tiles, one workgroup a tile, of at most `rem` rows; with groups > 0
// that of the panel before, where the present one is not whole.
static void update_tiles_launch(const FactorPlan& fp, hipStream_t st, long rem, int groups) {
  const long T = ceil_div(rem, 128);
  const double* const* auxs = groups > 0 ? (const double* const*)fp.d_aux : nullptr;
  const auto update = fp.stream_c ? k_trailing_update_lds<true> : k_trailing_update_lds<false>;
  SL_LAUNCH(update, dim3((unsigned)(T * (T + 1) / 2), fp.nshift), dim3(1024), 0, st, fp.n, fp.d_LD,
            fp.ldld, fp.d_W, fp.ldw, fp.d_state, auxs, fp.nb, groups);
  SL_LAUNCH_CHECK();
}

// One panel step of every shift of `fp` on stream `st`: the speculative
// pivot-free panel, the pivoting panel and the trailing update.  k0_lb is a lower
// bound on the step's first column (it sizes the update grid).  `after_panel`,
// when given, is recorded once the pivoting panel is enqueued.
// With `defer` > 0 a whole panel may leave its update to a later one (at most `defer` together);
// `pending` says that the step before was such a step.
static void factor_step(const FactorPlan& fp, hipStream_t st, long k0_lb, sislice_handle* ph,
                        hipEvent_t after_panel, int defer = 0, bool pending = false) {
  const int n = fp.n, S = fp.nshift, nb = fp.nb;
  const int nbpiv = fp.nbpiv;
  const int min_kb = factor_min_panel(nb, nbpiv);
  // one timed ticket per panel step: the pivot-free group and the pivoting panel are
  // consecutive launches of the panel class
  const int tpan = prof_begin(ph, kProfPanel, st);
  // a workgroup per 256 rows below the block, as many as run side by side (two a CU)
  const int groups = (int)std::max<long>(
      1, std::min<long>({ceil_div(n - k0_lb - 1, 256), (long)kSpecGroups, 2l * fp.cus / S}));
  const auto panel = nb > 32 ? (fp.pivot ? k_fast_panel<64, true> : k_fast_panel<64, false>)
                             : (fp.pivot ? k_fast_panel<32, true> : k_fast_panel<32, false>);
  SL_LAUNCH(panel, dim3((unsigned)groups, S), dim3(320), 0, st, n, (const double* const*)fp.d_LD,
            fp.ldld, fp.d_W, fp.ldw, fp.d_aux, fp.d_state, fp.d_team, nb);
  SL_LAUNCH_CHECK();
  long need;
  if (pending) update_tiles_launch(fp, st, n - k0_lb, groups);  // a panel that is not whole
  if (!panel_team(fp, n - k0_lb, need)) {
    SL_LAUNCH(fp.pivot ? k_fast_commit<true> : k_fast_commit<false>, dim3(nb, S), dim3(256), 0, st, n,
              fp.d_LD, fp.ldld, fp.d_W, fp.ldw, (const double* const*)fp.d_aux, fp.d_perm, fp.d_sw,
              fp.d_blk, fp.d_colpanel, fp.d_pstart, fp.d_state, fp.d_team, nb, nbpiv, groups);
    SL_LAUNCH_CHECK();
  }
  panel_launch(fp, st, n - k0_lb, nbpiv, groups, defer);
  prof_end(ph, tpan, st);
  if (after_panel) SL_HIP(hipEventRecord(after_panel, st));
  const long k1_lb = std::min<long>(n, k0_lb + min_kb);
  if (k1_lb >= n) return;
  const int tu = prof_begin(ph, kProfUpdate, st);
  if (defer || pending || n - k1_lb >= fp.wide_min) {
    update_tiles_launch(fp, st, n - k1_lb, 0);
  } else {
    const long T = ceil_div(n - k1_lb, 64);
    SL_LAUNCH(k_trailing_update, dim3((unsigned)(T * (T + 1) / 2), S), dim3(256), 0, st, n,
              fp.d_LD, fp.ldld, fp.d_W, fp.ldw, fp.d_state);
  }
  SL_LAUNCH_CHECK();
  prof_end(ph, tu, st);
}

// The deferred interchanges and the inertia of every shift of `fp`.
static void factor_tail(const FactorPlan& fp, hipStream_t st) {
  const int n = fp.n, S = fp.nshift;
  if (fp.pivot) {
    SL_LAUNCH(k_perm_suffix, dim3(S), dim3(1024), (size_t)n * sizeof(int), st, n, fp.d_sw,
              fp.d_pstart, fp.d_state, fp.d_snap);
    SL_LAUNCH_CHECK();
    SL_LAUNCH(k_left_gather, dim3(n, S), dim3(1024), (size_t)n * sizeof(double), st, n, fp.d_LD,
              fp.ldld, fp.d_colpanel, fp.d_pstart, fp.d_state, fp.d_snap);
    SL_LAUNCH_CHECK();
  }
  SL_LAUNCH(k_factor_finalize, dim3((unsigned)ceil_div(n, 256), S), dim3(256), 0, st, n, fp.d_perm,
            fp.d_blk, fp.d_ipiv, fp.d_state, fp.d_inertia, fp.wait_err);
  SL_LAUNCH_CHECK();
}

// Whether whole panels wait for one another with `rem` rows left: where the trailing
// triangles (half of 8 rem^2 bytes each) outgrow the 256 MB memory-side cache and an update
// is a pass over memory.  With every panel whole, in pairs and at once: order 4096, 17 shifts
// 19.1 and 21.4 ms; 8192, 24 shifts 137 and 165; 8192, 2 shifts 21.0 and 23.1; below, 4096,
// 4 shifts 8.30 and 8.20; 2048, 8 shifts 3.76 and 3.61 (a launch more a panel).
static bool defer_pays(long rem, int nb, int nshift) {
  return nb == kMaxNb && 4.0 * (double)rem * (double)rem * nshift >= (double)(256u << 20);
}
int factor_defers(int n, int nb, int nshift, bool pivot) {
  if (!pivot || n <= 0 || nshift <= 0 || !defer_pays(n, nb, nshift)) return 0;
  const double panel = 8.0 * (double)n * nb * nshift;  // bytes of W a panel
  const int p = (int)std::min<double>(kDeferPanels, 1.0 + (double)(4ull << 30) / panel);
  return p > 1 ? p : 0;
}

void factor_steps_launch(const FactorPlan& fp, hipStream_t st, bool readback) {
  const int n = fp.n, S = fp.nshift, nb = fp.nb;
  if (S <= 0 || n <= 0) return;
  factor_prepare();
  SL_LAUNCH(k_factor_init, dim3((unsigned)ceil_div(n, 256), S), dim3(256), 0, st, n,
                     fp.d_state, fp.d_perm, fp.d_sw, fp.d_team);
  SL_LAUNCH_CHECK();
  sislice_handle* ph = current_handle();
  const int min_kb = factor_min_panel(nb, fp.nbpiv);
  const int step_cap = factor_npanel_max(n, nb, fp.nbpiv);
  SL_CHECK_ARG(step_cap <= fp.npmax, "panel bookkeeping smaller than the step bound");
  if (!readback) {
    // a fixed sequence (for graph capture): every step up to the bound; steps
    // past a shift's end return at once
    for (int q = 0; q < step_cap; ++q)
      factor_step(fp, st, std::min<long>(n, (long)q * min_kb), ph, nullptr);
    factor_tail(fp, st);
    return;
  }
  // Panel widths depend on the pivots: launch chunks of steps and read the
  // per-shift progress back between chunks (kmin = least factored prefix of a
  // group).  The shifts run in G groups, each on its own stream, so that the
  // latency-bound panels of one group run while another group's updates use the
  // memory system; group g + 1 starts once group g's first pivoting panel is
  // enqueued, which staggers the groups by about one panel.
  const int G = ph ? std::max(1, std::min(fp.groups, S / 2)) : 1;
  std::vector<FactorPlan> sub(G);
  std::vector<hipStream_t> gs(G);
  std::vector<long> kmin(G, 0);
  std::vector<int> steps(G, 0);
  std::vector<char> launched(G, 0);
  // waiting updates: whether the last chunk's panels were mostly whole, the panels and whole
  // panels so far, and whether the step before deferred
  std::vector<char> mostly(G, 1), pending(G, 0);
  std::vector<long> panels(G, 0), whole(G, 0);
  for (int g = 0; g < G; ++g) {
    const int s0 = (int)((long)S * g / G), s1 = (int)((long)S * (g + 1) / G);
    sub[g] = factor_subplan(fp, s0, s1 - s0);
    if (G > 1) sub[g].stream_c = 1;
    gs[g] = g == 0 ? st : group_stream(ph, g - 1);
  }
  FactorState* hs = static_cast<FactorState*>(host_stage(ph, sizeof(FactorState) * S));
  if (G > 1) {
    if (ph->flush_fn) ph->flush_fn(ph->flush_ctx);  // staged tables reach the device first
    SL_HIP(hipEventRecord(group_event(ph, 0), st));
    for (int g = 1; g < G; ++g) SL_HIP(hipStreamWaitEvent(gs[g], group_event(ph, 0), 0));
  }
  constexpr int kChunk = 8;
  for (bool first = true;; first = false) {
    bool any = false;
    for (int g = 0; g < G; ++g) {
      launched[g] = kmin[g] < n && steps[g] < step_cap;
      if (!launched[g]) continue;
      any = true;
      for (int q = 0; q < kChunk && steps[g] < step_cap; ++q, ++steps[g]) {
        hipEvent_t mark = (first && q == 0 && g + 1 < G) ? group_event(ph, g + 1) : nullptr;
        const long lb = std::min<long>(n, kmin[g] + (long)q * min_kb);
        const int defer = mostly[g] && defer_pays(n - lb, nb, S) ? sub[g].defer : 0;
        factor_step(sub[g], gs[g], lb, ph, mark, defer, pending[g]);
        pending[g] = defer > 0;
        if (mark) SL_HIP(hipStreamWaitEvent(gs[g + 1], mark, 0));
      }
      const FactorPlan& f = sub[g];
      SL_HIP(hipMemcpyAsync(hs + (f.d_state - fp.d_state), f.d_state, sizeof(FactorState) * f.nshift,
                            hipMemcpyDeviceToHost, gs[g]));
    }
    if (!any) break;
    for (int g = 0; g < G; ++g) {
      if (!launched[g]) continue;
      SL_HIP(hipStreamSynchronize(gs[g]));
      const FactorPlan& f = sub[g];
      const FactorState* h0 = hs + (f.d_state - fp.d_state);
      long km = n;
      long np = 0, nw = 0;
      for (int q = 0; q < f.nshift; ++q) {
        km = std::min<long>(km, h0[q].done ? n : h0[q].k0 + h0[q].kb);
        np += h0[q].npanel;
        nw += h0[q].whole;
      }
      kmin[g] = km;
      mostly[g] = 4 * (nw - whole[g]) >= 3 * (np - panels[g]);
      panels[g] = np;
      whole[g] = nw;
    }
  }
  for (int g = 0; g < G; ++g)
    SL_CHECK_ARG(kmin[g] >= n, "factorization did not complete");
  for (int g = 0; g < G; ++g) factor_tail(sub[g], gs[g]);
  if (G > 1) {
    for (int g = 1; g < G; ++g) {
      SL_HIP(hipEventRecord(group_event(ph, g), gs[g]));
      SL_HIP(hipStreamWaitEvent(st, group_event(ph, g), 0));
    }
  }
}

}  // namespace sislice
