// Symmetric eigensolver of the solve path's iteration (Section 2.1: Lanczos matrices T, and
// the B-Gram matrices of Rayleigh-Ritz): Householder tridiagonalisation, divide and conquer
// and one step of refinement.
//
// The published methods: Householder's reduction (Wilkinson 1965), Cuppen's
// rank-one tearing (1981) with the deflation of Dongarra and Sorensen (1987), rational
// interpolation of the secular equation (Bunch, Nielsen and Sorensen 1978; Li 1993), the
// eigenvectors from the Loewner formula of Gu and Eisenstat (1994), orthogonal to working
// precision however close the eigenvalues lie, and the eigenvector refinement of Ogita and
// Aishima (2018).
//
// What bounds it and why this form (gfx950).  The problems are small (m <= 112) and few
// (one per probe), so the call is one chain of dependent steps on one CU; the length of
// that chain is what counts.  Cyclic Jacobi (eig.hip) takes about 9 sweeps x 111 rounds
// with a workgroup barrier each.  Here the reduction takes m - 2 steps of two barriers
// on a matrix held in registers, and the divide-and-conquer levels, about ten barriers
// each, have no serial part except rare deflating rotations:
//   1. reduction (149 us of 390 at order 112): four lanes share a row, so 8 wavefronts hold
//      the matrix; with 16 (eight lanes a row) the instructions every wavefront repeats
//      took 172 us.  A step publishes column k; every wavefront forms the norm for itself,
//      which is cheaper than waiting for one that does.
//   2. divide and conquer (about 120 us) from pairs up to the whole, the merges of a level
//      side by side.  A root of the secular equation is found by 4 lanes; Q in LDS is
//      multiplied by the eigenvectors of the rank-one problem on FP64 MFMA, whose B
//      operand is formed on the fly from the poles and roots.
//   3. back-transformation (18 us): four lanes share a column of Q in registers and apply
//      the reflectors from LDS, no barrier.
//   4. refinement (57 us): three products on FP64 MFMA, chained through registers.
// Measured per launch of 16 random matrices against Jacobi's two kernels: order 112
// 389 against 1579 us, 80 265 against 969, 56 156 against 542, 30 90 against 287.
//
// Accuracy against Jacobi (the same matrices): eigenvalues and residuals two to four times
// closer, orthogonality 2e-15 against 2e-14, and on Lanczos matrices after a restart
// (Ritz values from 3 to 5000) components of the small ones' vectors along each other
// 1e-16 against 9e-15.
#include <algorithm>
#include <cfloat>
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "eig.hpp"
#include "handle.hpp"

namespace sislice {

namespace {

constexpr int E = kEigMax;       // 112 rows and columns at most
constexpr double kEps = 2.220446049250313e-16;

template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(v >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// the sum over a quad of lanes (quad_perm xor 1, xor 2), the same bits in each
__device__ __forceinline__ double sum4(double x) {
  x += dpp<0xB1>(x);
  return x + dpp<0x4E>(x);
}
__device__ __forceinline__ double prod4(double x) {
  x *= dpp<0xB1>(x);
  return x * dpp<0x4E>(x);
}
__device__ __forceinline__ int sum4i(int x) {
  x += __builtin_amdgcn_mov_dpp(x, 0xB1, 0xf, 0xf, true);
  return x + __builtin_amdgcn_mov_dpp(x, 0x4E, 0xf, 0xf, true);
}
__device__ __forceinline__ double lane_value(double x, int lane) {
  const long long v = __double_as_longlong(x);
  const unsigned lo = __builtin_amdgcn_readlane((int)v, lane);
  const unsigned hi = __builtin_amdgcn_readlane((int)(v >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | lo);
}
__device__ __forceinline__ double sum_wave(double x) {
  x = sum4(x);
  x += dpp<0x141>(x);  // the mirrored half row of 8, then the mirrored row of 16
  x += dpp<0x140>(x);
  return (lane_value(x, 0) + lane_value(x, 16)) + (lane_value(x, 32) + lane_value(x, 48));
}
// 1 / x and 1 / sqrt(x) from the hardware approximations and two Newton steps
__device__ __forceinline__ double rcp2(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(y, fma(-x, y, 1.0), y);
  return fma(y, fma(-x, y, 1.0), y);
}
__device__ __forceinline__ double rsq2(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double hx = 0.5 * x;
  y = y * fma(-hx, y * y, 1.5);
  return y * fma(-hx, y * y, 1.5);
}

// f(0), f(1), ... f(N - 1) with compile-time arguments
template <class F, int... I>
__device__ __forceinline__ void static_for_(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_(f, std::make_integer_sequence<int, N>{});
}

// Segment i of the 2^lev segments of 0 .. m - 1 (halving: the segments of one level are
// pairs of segments of the next finer one).
__device__ __forceinline__ int seg(int i, int m, int lev) { return (i * m) >> lev; }
// the segment that holds element i
__device__ __forceinline__ int seg_of(int i, int m, int lev) {
  int g = (i << lev) / m;
  while (seg(g + 1, m, lev) <= i) ++g;
  return g;
}

// A workgroup barrier that orders LDS only: __syncthreads would also wait for the global
// stores in flight (the reflectors), half a microsecond a step.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

struct Shared {
  double xs[2][E], ps[E];                // reduction: column k (by parity), A u
  double hv[E];                          // its reflectors' 1 / h
  double d[E], e[E];                     // diagonal (then eigenvalue of column c), off-diagonal
  double dl[E], zl[E];                   // a merge's poles and weights, ascending
  double dk[E], zk[E];                   // the ones that are not deflated
  double mu[E], lam[E], zh[E], nrm[E];   // root - its pole, root, Loewner weight, 1 / norm
  double rc[E], rs[E];                   // deflating rotations
  double red[8];
  int ph[E], pk[E], org[E];              // column of a pole; of one not deflated; a root's pole
  int rp[E], rq[E];                      // columns of the rotations
  int up[E], lo[E];                      // poles whose column lies in the upper / lower segment
  int nd[E], cl[E];                      // pole not deflated; per merge: some poles nearly equal
  int nk[E], nup[E], nlo[E], nrot[E];    // per merge: poles, upper, lower, rotations
  int rank[E];
};

// One root of f(x) = 1/rho + sum_i zk_i^2 / (dk_i - x) by the 4 lanes of a quad (lane q takes
// the poles q + 4c): root t lies right of pole t.  x is an offset from the nearer pole, so
// that the distances to all poles stay accurate.  A step solves the two-pole model
// c - W0/x + W1/(D - x) = 0 with D the other pole of the gap (of the last root: pole t - 1).
// W0 is the nearer pole's own weight, W1 and c come from f' and f (Li's fixed weight); when
// a step shrinks f by less than ten, the next one takes both weights from the derivatives of
// the two sides (Bunch, Nielsen and Sorensen).  Steps out of the bracket, and every fourth
// one after the seventh, halve the bracket, by its exponent where it spans decades.
// Lanczos matrices after a restart need 3 steps on average, close pairs up to 25.
__device__ __forceinline__ void secular_root(const double* dk, const double* zk, int K, int t, int q,
                                             double rho, double& mu_out, int& org_out) {
  const double rinv = 1.0 / rho;
  const bool last = t == K - 1, only = K == 1;
  double gap;
  if (last) {
    double s = 0.0;
    for (int i = q; i < K; i += 4) s += zk[i] * zk[i];
    gap = rho * sum4(s);
  } else {
    gap = dk[t + 1] - dk[t];
  }
  int org = t;
  double x = 0.5 * gap, lo = 0.0, hi = gap, wp = 1e300;
  bool fixed = true;
  for (int it = 0; it < 100; ++it) {
    const double dorg = dk[org];
    double f = 0.0, fa = 0.0, df = 0.0, dl = 0.0;
#pragma unroll 4
    for (int i = q; i < K; i += 4) {
      const double z = zk[i], r = z * rcp2((dk[i] - dorg) - x), r2 = r * r;
      f = fma(z, r, f);
      fa += fabs(z * r);
      df += r2;
      dl += i <= t ? r2 : 0.0;
    }
    f = sum4(f);
    fa = sum4(fa);
    df = sum4(df);
    dl = sum4(dl);
    const double w = rinv + f;
    if (it == 0 && !last) {
      // the half that holds the root; offsets from the nearer pole from here on
      if (w > 0.0) {
        hi = x;
      } else {
        org = t + 1;
        x -= gap;
        lo = x;
        hi = 0.0;
      }
    } else if (w < 0.0) {
      lo = x;
    } else {
      hi = x;
    }
    if (!(fabs(w) > kEps * (8.0 * (rinv + fa) + fabs(x) * df))) break;
    const bool left = org == t;
    const double D = last ? (only ? 0.0 : dk[t - 1] - dk[t]) : (left ? gap : -gap), b = D - x;
    const double rx = rcp2(x), rb = only ? 0.0 : rcp2(b);
    double W0 = zk[org] * zk[org], W1 = fmax(df - W0 * rx * rx, 0.0) * b * b;
    if (!fixed && !last) {
      W0 = (left ? dl : df - dl) * x * x;
      W1 = (left ? df - dl : dl) * b * b;
    }
    if (only) W1 = 0.0;
    double c = w + W0 * rx - W1 * rb;
    // c y^2 - B y + W0 |D| = 0 in the offset's modulus y (of the last root: in x)
    const double B = fma(c, D, W0 + W1);
    double E0 = W0 * D;
    if (!left) {
      c = -c;
      E0 = -E0;
    }
    const double disc = fma(B, B, -4.0 * c * E0);
    const double rt = disc > 0.0 ? disc * rsq2(disc) : 0.0;
    const bool pos = last ? B >= 0.0 : B > 0.0, first = last == pos;  // (B +- rt) / 2c or 2 E0 / (B +- rt)
    const double sum = pos ? B + rt : B - rt;
    double xn = (first ? sum : 2.0 * E0) * rcp2(first ? 2.0 * c : sum);
    if (!left) xn = -xn;
    if (it > 0 && fabs(w) > 0.1 * wp) fixed = !fixed;
    wp = fabs(w);
    if (!(xn > lo && xn < hi) || (it > 6 && (it & 3) == 3)) {
      const double al = fmin(fabs(lo), fabs(hi)), ah = fmax(fabs(lo), fabs(hi));
      xn = copysign(fmax(sqrt(al * ah), ah * 0x1p-10), lo + hi);
      if (last || !(xn > lo && xn < hi)) xn = 0.5 * (lo + hi);
    }
    if (!(xn > lo && xn < hi) || fabs(xn - x) <= 2.0 * kEps * fabs(xn)) break;
    x = xn;
  }
  mu_out = x;
  org_out = org;
}

// P: the padded order (m <= P), a multiple of 16.  NT threads, four to a row.
template <int P, int NT>
__global__ __launch_bounds__(NT) void k_eig_dc(EigArgs a, double* __restrict__ refl, long rstride,
                                               int qdoubles) {
  constexpr int NB = P / 8;  // blocks of 8 columns; a lane holds columns 8c + 2q, 8c + 2q + 1
  constexpr int NW = NT / 64;
  extern __shared__ double sh[];
  double* Q = sh;  // column-major, ldq rows a column (odd); then the reflectors; then X
  Shared& S = *reinterpret_cast<Shared*>(sh + qdoubles);
  const int b = blockIdx.x, tid = threadIdx.x;
  const int m = a.m[b];
  if (m <= 0) return;
  const int ldq = m | 1;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int i = tid >> 2, q = tid & 3;  // row (reduction), element or column; lane of its quad
  double* U = refl + (long)b * rstride;  // reflector k at U + k * P
  const double* Ain = global_ptr(a.A[b]);
  const long lda = a.lda;

  // ---- 1. reduction to tridiagonal form
  double x[NB][2];
  double mx = 0.0;
#pragma unroll
  for (int c = 0; c < NB; ++c)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j = 8 * c + 2 * q + h;
      const int r = min(max(i, j), m - 1), cc = min(min(i, j), m - 1);
      const double v = Ain[r + (long)cc * lda];
      x[c][h] = (i < m && j < m) ? v : 0.0;
      mx = fmax(mx, fabs(x[c][h]) <= DBL_MAX ? fabs(x[c][h]) : INFINITY);
    }
  // An entry that is not finite makes every result NaN.  Otherwise the largest entry is brought
  // to between 1e-20 and 1e20 by a power of two: what is below 1e-100 then (squares leave the
  // range) is far below its rounding, and is dropped by the reduction and the deflation.
  mx = fmax(mx, dpp<0xB1>(mx));
  mx = fmax(mx, dpp<0x4E>(mx));
  mx = fmax(mx, dpp<0x141>(mx));
  mx = fmax(mx, dpp<0x140>(mx));
  if (lane == 0)
    S.red[w] = fmax(fmax(lane_value(mx, 0), lane_value(mx, 16)), fmax(lane_value(mx, 32), lane_value(mx, 48)));
  lds_barrier();
  mx = S.red[0];
  for (int k = 1; k < NW; ++k) mx = fmax(mx, S.red[k]);
  if (mx > DBL_MAX) {  // uniform
    for (int k = tid; k < m; k += NT) a.W[b][k] = NAN;
    for (int k = tid; k < m * m; k += NT) a.V[b][k % m + (long)(k / m) * a.ldv] = NAN;
    return;
  }
  int ex = 0;
  if (mx > 0.0 && (mx < 1e-20 || mx > 1e20)) {
    ex = ilogb(mx);
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int h = 0; h < 2; ++h) x[c][h] = ldexp(x[c][h], -ex);
  }
  // The code is unrolled for every 16 columns, so a step touches at most 15 finished ones
  // and the register indexes are static; finished rows and columns meet zeros.
  static_for<NB / 2>([&](auto gc) {
    constexpr int G = gc;
    const int kend = min(16 * G + 16, m - 2);
#pragma unroll 1
    for (int k = 16 * G; k < kend; ++k) {
      double* xs = S.xs[k & 1];
      const bool odd = k & 1, second = k & 8;
      const double y0 = second ? x[2 * G + 1][0] : x[2 * G][0];
      const double y1 = second ? x[2 * G + 1][1] : x[2 * G][1];
      const double y = odd ? y1 : y0;
      if (q == ((k >> 1) & 3) && i < E) {
        xs[i] = i > k ? y : 0.0;
        if (i == k) S.d[k] = y;
      }
      lds_barrier();
      const double alpha = xs[k + 1];
      const double v0 = lane < P ? xs[lane] : 0.0, v1 = lane + 64 < P ? xs[lane + 64] : 0.0;
      const bool live = i < P && 16 * w + 15 > k;  // some row of this wavefront is in play
      // A x without column k + 1, whose entry of u is known later
      double s = 0.0, s2 = 0.0, ak = 0.0;
      double2 ur[NB];
      if (live) {
#pragma unroll
        for (int c = 2 * G; c < NB; ++c) ur[c] = *reinterpret_cast<const double2*>(xs + 8 * c + 2 * q);
#pragma unroll
        for (int c = 2 * G; c < NB; ++c) {
          const int j = 8 * c + 2 * q;
          if (c <= 2 * G + 2) {
            const bool h0 = j == k + 1, h1 = j + 1 == k + 1;
            ak = h0 ? x[c][0] : (h1 ? x[c][1] : ak);
            ur[c].x = h0 ? 0.0 : ur[c].x;
            ur[c].y = h1 ? 0.0 : ur[c].y;
          }
          s = fma(x[c][0], ur[c].x, s);
          s2 = fma(x[c][1], ur[c].y, s2);
        }
      }
      const double sig = sum_wave((lane > k + 1 ? v0 * v0 : 0.0) + (lane + 64 > k + 1 ? v1 * v1 : 0.0));
      // H = I - u u^T / h maps the column to beta e_{k+1}; u = the column with alpha - beta
      double beta = alpha, hinv = 0.0;
      if (sig > 1e-200) {
        const double n2 = fma(alpha, alpha, sig), nr = n2 * rsq2(n2);
        beta = -copysign(nr, alpha);
        hinv = rcp2(fma(nr, fabs(alpha), n2));
      }
      const double u1 = alpha - beta;
      if (live) {
        s = sum4(fma(ak, u1, s + s2));
        if (q == 0) S.ps[i] = i > k ? s * hinv : 0.0;
      } else if (i < P && q == 0) {
        S.ps[i] = 0.0;
      }
      lds_barrier();
      if (tid < P) U[(long)k * P + tid] = tid == k + 1 ? u1 : xs[tid];
      if (tid == 0) {
        S.e[k] = beta;
        S.hv[k] = hinv;
      }
      if (live) {
        const double f0 = lane == k + 1 ? u1 : v0, f1 = lane + 64 == k + 1 ? u1 : v1;
        const double g0 = lane < P ? S.ps[lane] : 0.0, g1 = lane + 64 < P ? S.ps[lane + 64] : 0.0;
        double2 pr[NB];
#pragma unroll
        for (int c = 2 * G; c < NB; ++c) pr[c] = *reinterpret_cast<const double2*>(S.ps + 8 * c + 2 * q);
        const double ui = i == k + 1 ? u1 : xs[i], pi = S.ps[i];
        const double kq = 0.5 * hinv * sum_wave(f0 * g0 + f1 * g1);
        const double qi = pi - kq * ui;
#pragma unroll
        for (int c = 2 * G; c < NB; ++c) {
          const int j = 8 * c + 2 * q;
          if (c <= 2 * G + 2) {
            ur[c].x = j == k + 1 ? u1 : ur[c].x;
            ur[c].y = j + 1 == k + 1 ? u1 : ur[c].y;
          }
          x[c][0] -= fma(ui, fma(-kq, ur[c].x, pr[c].x), qi * ur[c].x);
          x[c][1] -= fma(ui, fma(-kq, ur[c].y, pr[c].y), qi * ur[c].y);
        }
      }
    }
  });
#pragma unroll
  for (int c = 0; c < NB; ++c)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j = 8 * c + 2 * q + h;
      if (i == j && i < m && i + 2 >= m) S.d[i] = x[c][h];
      if (i == m - 1 && j == m - 2) S.e[m - 2] = x[c][h];
    }
  for (int k = tid; k < m * ldq; k += NT) Q[k] = 0.0;
  lds_barrier();

  // ---- 2. divide and conquer, from leaves of one or two elements
  int lev = 0;
  while ((2 << lev) < m) ++lev;
  if (tid < E) {  // valid columns everywhere, also where NaNs leave places unranked
    S.ph[tid] = S.pk[tid] = tid < m ? tid : 0;
    S.org[tid] = 0;
  }
  if (tid < (1 << lev)) {
    const int c0 = seg(tid, m, lev), c1 = seg(tid + 1, m, lev);
    if (c1 > c0) {
      // torn at both ends: the borders lose the off-diagonal's modulus
      double d0 = S.d[c0], d1 = S.d[c1 - 1];
      const double eb = c0 > 0 ? fabs(S.e[c0 - 1]) : 0.0, ea = c1 < m ? fabs(S.e[c1 - 1]) : 0.0;
      if (c1 == c0 + 1) {
        S.d[c0] = d0 - eb - ea;
        Q[c0 * ldq + c0] = 1.0;
      } else {
        d0 -= eb;
        d1 -= ea;
        // the 2x2 rotation with tan of the smaller angle
        const double e = S.e[c0], dd = d1 - d0, hyp = hypot(dd, 2.0 * e);
        const double t = e == 0.0 ? 0.0 : copysign(2.0 * fabs(e) / (fabs(dd) + hyp), dd < 0.0 ? -e : e);
        const double c = 1.0 / sqrt(fma(t, t, 1.0)), sn = t * c;
        S.d[c0] = d0 - t * e;
        S.d[c1 - 1] = d1 + t * e;
        Q[c0 * ldq + c0] = c;
        Q[c0 * ldq + c0 + 1] = -sn;
        Q[(c0 + 1) * ldq + c0] = sn;
        Q[(c0 + 1) * ldq + c0 + 1] = c;
      }
    }
  }
  lds_barrier();
  for (int lv = lev - 1; lv >= 0; --lv) {
    const int nm = 1 << lv;
    // the merge of element (and place) i, its segments [s0, s1) and [s1, s2)
    int s0 = 0, s1 = 0, s2 = 0;
    if (i < m) {
      const int g = seg_of(i, m, lv);
      s0 = seg(g, m, lv);
      s1 = seg(2 * g + 1, m, lv + 1);
      s2 = seg(g + 1, m, lv);
    }
    const bool merging = s0 < s1 && s1 < s2;
    const double beta = merging ? S.e[s1 - 1] : 0.0, rho = 2.0 * fabs(beta);
    // poles in ascending order: the rank of element i in its merge
    if (merging) {
      const double di = S.d[i];
      int r = 0;
#pragma unroll 4
      for (int j = s0 + q; j < s2; j += 4) {
        const double dj = S.d[j];
        r += (dj < di) || (dj == di && j < i);
      }
      r = s0 + sum4i(r);
      if (q == 0) {
        const double zi = i < s1 ? Q[i * ldq + s1 - 1] : copysign(1.0, beta) * Q[i * ldq + s1];
        S.dl[r] = di;
        S.zl[r] = zi * 0.70710678118654752440;
        S.ph[r] = i;
      }
    }
    lds_barrier();
    // deflation: poles without weight, then neighbours so close that a rotation decouples
    // one of them (rare: one wavefront walks such a merge in order)
    double tol = 0.0;
    bool nd = false;
    if (merging) {
      tol = 8.0 * kEps * fmax(fmax(fabs(S.dl[s0]), fabs(S.dl[s2 - 1])), fmax(rho, 1e-120));
      nd = rho * fabs(S.zl[i]) > tol;
      if (q == 0) {
        S.nd[i] = nd ? 1 : 0;
        if (i == s0) {
          S.cl[i] = 0;
          S.nrot[i] = 0;
        }
      }
    }
    lds_barrier();
    if (nd) {
      int pr = i - 1;
      while (pr >= s0 && !S.nd[pr]) --pr;
      if (pr >= s0) {
        const double z1 = S.zl[i], z0 = S.zl[pr];
        if (fabs((S.dl[i] - S.dl[pr]) * z1 * z0) <= tol * (z1 * z1 + z0 * z0)) S.cl[s0] = 1;
      }
    }
    lds_barrier();
    for (int g = w; g < nm; g += NW) {
      const int t0 = seg(g, m, lv), t1 = seg(2 * g + 1, m, lv + 1), t2 = seg(g + 1, m, lv);
      if (!(t0 < t1 && t1 < t2) || !S.cl[t0]) continue;  // uniform
      const double rg = 2.0 * fabs(S.e[t1 - 1]);
      const double tg = 8.0 * kEps * fmax(fmax(fabs(S.dl[t0]), fabs(S.dl[t2 - 1])), fmax(rg, 1e-120));
      // each rotation changes the next test; every lane follows the same steps, lane 0 writes
      int pr = -1, nr = 0;
      for (int p = t0; p < t2; ++p) {
        if (!S.nd[p]) continue;
        if (pr >= 0) {
          const double z1 = S.zl[p], z0 = S.zl[pr], d1 = S.dl[p], d0 = S.dl[pr], zz = z1 * z1 + z0 * z0;
          if (fabs((d1 - d0) * z1 * z0) <= tg * zz) {
            const double tau = sqrt(zz), c = z1 / tau, s = z0 / tau;
            __builtin_amdgcn_wave_barrier();
            if (lane == 0) {
              S.zl[p] = tau;
              S.zl[pr] = 0.0;
              S.dl[pr] = d0 * c * c + d1 * s * s;
              S.dl[p] = d0 * s * s + d1 * c * c;
              S.rc[t0 + nr] = c;
              S.rs[t0 + nr] = s;
              S.rp[t0 + nr] = S.ph[pr];
              S.rq[t0 + nr] = S.ph[p];
              S.nd[pr] = 0;
            }
            __builtin_amdgcn_wave_barrier();
            ++nr;
          }
        }
        pr = p;
      }
      if (lane == 0) S.nrot[t0] = nr;
    }
    lds_barrier();
    // the poles that stay, and those of the upper and of the lower segment; rotated
    // columns may reach into both, so after a rotation both lists hold every pole
    if (merging) {
      const int nr = S.nrot[s0];
      const bool stay = S.nd[i] != 0;
      const int col = S.ph[i];
      int k = 0, ku = 0, kl = 0, kt = 0, ut = 0, lt = 0;
#pragma unroll 4
      for (int j = s0 + q; j < s2; j += 4) {
        const int one = S.nd[j], cj = S.ph[j];
        const int u = one && (nr || cj < s1), l = one && (nr || cj >= s1);
        kt += one;
        ut += u;
        lt += l;
        if (j < i) {
          k += one;
          ku += u;
          kl += l;
        }
      }
      k = sum4i(k);
      ku = sum4i(ku);
      kl = sum4i(kl);
      if (q == 0) {
        if (stay) {
          S.dk[s0 + k] = S.dl[i];
          S.zk[s0 + k] = S.zl[i];
          S.pk[s0 + k] = col;
          if (nr || col < s1) S.up[s0 + ku] = k;
          if (nr || col >= s1) S.lo[s0 + kl] = k;
        } else {
          S.d[col] = S.dl[i];
        }
      }
      if (i == s0) {
        kt = sum4i(kt);
        ut = sum4i(ut);
        lt = sum4i(lt);
        if (q == 0) {
          S.nk[s0] = kt;
          S.nup[s0] = ut;
          S.nlo[s0] = lt;
        }
      }
      // deflating rotations: row i of its merge's columns
      if (q == 0)
        for (int r = 0; r < nr; ++r) {
          double* u = Q + S.rp[s0 + r] * ldq + i;
          double* v = Q + S.rq[s0 + r] * ldq + i;
          const double c = S.rc[s0 + r], s = S.rs[s0 + r], y0 = *u, y1 = *v;
          *u = c * y0 - s * y1;
          *v = s * y0 + c * y1;
        }
    }
    lds_barrier();
    // the roots
    const int K = merging ? S.nk[s0] : 0, t = i - s0;
    const bool root = merging && t < K;
    double mu = 0.0;
    int org = 0;
    if (root) {
      secular_root(S.dk + s0, S.zk + s0, K, t, q, rho, mu, org);
      if (q == 0) {
        S.mu[i] = mu;
        S.org[i] = org;
        S.lam[i] = S.dk[s0 + org] + mu;
      }
    }
    lds_barrier();
    // Loewner weights: the rank-one problem whose roots these are exactly
    if (root) {
      const double di = S.dk[s0 + t];
      double p = 1.0;
#pragma unroll 4
      for (int j = q; j < K; j += 4) {
        const double lj = (S.dk[s0 + S.org[s0 + j]] - di) + S.mu[s0 + j];
        const double den = j < t ? S.dk[s0 + j] - di : (j < K - 1 ? S.dk[s0 + j + 1] - di : 1.0);
        p *= lj * rcp2(den);
      }
      p = prod4(p);
      if (q == 0) S.zh[i] = copysign(sqrt(fabs(p)), S.zk[s0 + t]);
    }
    lds_barrier();
    if (root) {
      const double dorg = S.dk[s0 + org];
      double s = 0.0;
#pragma unroll 4
      for (int j = q; j < K; j += 4) {
        const double u = S.zh[s0 + j] * rcp2((S.dk[s0 + j] - dorg) - mu);
        s = fma(u, u, s);
      }
      s = sum4(s);
      if (q == 0) S.nrm[i] = 1.0 / sqrt(s);
    }
    lds_barrier();
    // Q(:, stay) <- Q(:, stay) U
    const int most = (m + nm - 1) >> lv;  // rows of the largest merge
    if (most <= 8) {
      // lane q forms roots q and q + 4 of row i
      double y[2] = {0.0, 0.0};
      if (merging)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int j = q + 4 * h;
          if (j < K) {
            const double dorg = S.dk[s0 + S.org[s0 + j]], mj = S.mu[s0 + j], nj = S.nrm[s0 + j];
            for (int k = 0; k < K; ++k)
              y[h] = fma(Q[S.pk[s0 + k] * ldq + i], S.zh[s0 + k] * rcp2((S.dk[s0 + k] - dorg) - mj) * nj, y[h]);
          }
        }
      lds_barrier();
      if (merging)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          if (q + 4 * h < K) Q[S.pk[s0 + q + 4 * h] * ldq + i] = y[h];
    } else {
      // A task is one half of the rows (a merge of at most 16 rows: all of them) x 16 roots
      // of one merge.  A level has at most 2 NW tasks, so every wavefront takes its two
      // and all of them have read their columns before any is written.
      const int nct = (most + 15) >> 4, nh = most > 16 ? 2 : 1;
      const int tasks = nm * nh * nct;
      const int lr = lane & 15, lg = lane >> 4;
      d4 acc[2][4];
      int rb[2], re[2], oc[2];  // rows, and the column this lane writes (-1: none)
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const int tk = w + NW * v;
        const int g = tk / (nh * nct), half = nh == 2 ? (tk / nct) & 1 : 2, ct = tk % nct;
        const int t0 = seg(g, m, lv), t1 = seg(2 * g + 1, m, lv + 1), t2 = seg(g + 1, m, lv);
        const bool real = tk < tasks && t0 < t1 && t1 < t2;
        const int Kg = real ? S.nk[t0] : 0;
        rb[v] = half == 1 ? t1 : t0;
        re[v] = half == 0 ? t1 : t2;
        oc[v] = -1;
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[v][u] = d4{0.0, 0.0, 0.0, 0.0};
        if (16 * ct < Kg) {
          const int nrt = (re[v] - rb[v] + 15) >> 4;
          const int j = 16 * ct + lr;  // root
          const bool jv = j < Kg;
          const int cnt = half == 2 ? Kg : (half == 0 ? S.nup[t0] : S.nlo[t0]);
          const int* list = half == 0 ? S.up + t0 : S.lo + t0;
          const int jc = t0 + (jv ? j : 0);
          if (jv) oc[v] = S.pk[jc];
          const double dorg = S.dk[t0 + S.org[jc]], mj = S.mu[jc], nj = S.nrm[jc];
          // two steps of four poles at a time: the loads of both go out together
          for (int k0 = 0; k0 < cnt; k0 += 8) {
            double uv[2], av[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int kl = min(k0 + 4 * h + lg, cnt - 1);
              const int k = t0 + (half == 2 ? kl : list[kl]);
              const double* col = Q + S.pk[k] * ldq;
              const double u0 = S.zh[k] * rcp2((S.dk[k] - dorg) - mj) * nj;
              uv[h] = k0 + 4 * h + lg < cnt && jv ? u0 : 0.0;
#pragma unroll
              for (int u = 0; u < 4; ++u)
                if (u < nrt) av[h][u] = col[min(rb[v] + 16 * u + lr, re[v] - 1)];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
              for (int u = 0; u < 4; ++u)
                if (u < nrt) acc[v][u] = mfma16x16x4(av[h][u], uv[h], acc[v][u]);
          }
        }
      }
      lds_barrier();
#pragma unroll
      for (int v = 0; v < 2; ++v)
        if (oc[v] >= 0) {
          double* col = Q + oc[v] * ldq;
#pragma unroll
          for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int row = rb[v] + 16 * u + lg + 4 * r;
              if (row < re[v]) col[row] = acc[v][u][r];
            }
        }
    }
    if (root && q == 0) S.d[S.pk[i]] = S.lam[i];
    lds_barrier();
  }

  // ---- 3. back-transformation: a quad holds column i of Q, rows 8r + 2q, 8r + 2q + 1
#pragma unroll
  for (int r = 0; r < NB; ++r)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int row = 8 * r + 2 * q + h;
      const double v = Q[min(i, m - 1) * ldq + min(row, m - 1)];
      x[r][h] = row < m ? v : 0.0;
    }
  __syncthreads();
  for (int k = tid; k < (m - 2) * P; k += NT) Q[k] = U[k];
  __syncthreads();
  static_for<NB / 2>([&](auto gc) {
    constexpr int G = NB / 2 - 1 - gc;
    const int k1 = min(16 * G + 15, m - 3);
    if (k1 < 16 * G) return;  // uniform
    // reflector k has zeros up to row k: the blocks from 2G on; the next one is loaded
    // while this one is applied
    double2 un[NB];
    auto load = [&](int k) {
#pragma unroll
      for (int r = 2 * G; r < NB; ++r) un[r] = *reinterpret_cast<const double2*>(Q + k * P + 8 * r + 2 * q);
    };
    load(k1);
#pragma unroll 1
    for (int k = k1; k >= 16 * G; --k) {
      double2 ur[NB];
#pragma unroll
      for (int r = 2 * G; r < NB; ++r) ur[r] = un[r];
      const double hk = S.hv[k];
      load(max(k - 1, 16 * G));
      double s = 0.0, s2 = 0.0;
#pragma unroll
      for (int r = 2 * G; r < NB; ++r) {
        s = fma(ur[r].x, x[r][0], s);
        s2 = fma(ur[r].y, x[r][1], s2);
      }
      s = sum4(s + s2) * hk;
#pragma unroll
      for (int r = 2 * G; r < NB; ++r) {
        x[r][0] = fma(-s, ur[r].x, x[r][0]);
        x[r][1] = fma(-s, ur[r].y, x[r][1]);
      }
    }
  });

  // ---- 4. one step of refinement (Ogita and Aishima): with r_j = A x_j - d_j x_j and
  // G = X^T R, X <- X (I + E), E_ij = G_ij / (d_j - d_i), d_j <- d_j + G_jj.  The steps above
  // are accurate to rounding of ||A||; a Lanczos matrix near a shift mixes Ritz values of
  // very different size, and this restores the accuracy of the small ones' vectors
  // (components along each other 30 times smaller on such matrices, below Jacobi's).
  // Pairs whose gap the residual does not resolve are left as they are.
  constexpr int ldx = P + 1;
  constexpr int TL = P / 16;   // column tiles: one a wavefront
  // 16 columns of A, [k][row]; later two 16x16 tiles a wavefront
  double* Tc = sh + qdoubles + (sizeof(Shared) + 15) / 16 * 2;
  lds_barrier();
#pragma unroll
  for (int r = 0; r < NB; ++r)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (i < P) Q[i * ldx + 8 * r + 2 * q + h] = i < m ? x[r][h] : 0.0;
  const int lr = lane & 15, lg = lane >> 4, j = 16 * w + lr;  // this wavefront's column of X
  const bool tile = w < TL;
  d4 y[TL];
#pragma unroll
  for (int rt = 0; rt < TL; ++rt) y[rt] = d4{0.0, 0.0, 0.0, 0.0};
  constexpr int TE = (16 * P + NT - 1) / NT;
  double tn[TE];
  auto load_a = [&](int k0) {
#pragma unroll
    for (int t = 0; t < TE; ++t) {
      const int e = tid + NT * t, r = e % P, k = k0 + e / P;
      const int ra = min(max(r, k), m - 1), ca = min(min(r, k), m - 1);
      const double v = Ain[ra + (long)ca * lda];
      tn[t] = r < m && k < m ? v : 0.0;
    }
  };
  load_a(0);
  for (int k0 = 0; k0 < m; k0 += 16) {
    lds_barrier();
#pragma unroll
    for (int t = 0; t < TE; ++t) {
      const int e = tid + NT * t;
      if (e < 16 * P) Tc[(e / P) * ldx + e % P] = ex ? ldexp(tn[t], -ex) : tn[t];
    }
    lds_barrier();
    load_a(k0 + 16);
    if (tile)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double xv = Q[j * ldx + k0 + 4 * u + lg];
#pragma unroll
        for (int rt = 0; rt < TL; ++rt) y[rt] = mfma16x16x4(Tc[(4 * u + lg) * ldx + 16 * rt + lr], xv, y[rt]);
      }
  }
  // accumulator element r of tile rt is row 16 rt + lg + 4 r: the B operand of the products
  // that follow takes it as it is
  const double dj = j < m ? S.d[j] : 0.0;
  d4 e[TL];
  if (tile) {
#pragma unroll
    for (int rt = 0; rt < TL; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) y[rt][r] = fma(-dj, Q[j * ldx + 16 * rt + lg + 4 * r], y[rt][r]);
#pragma unroll
    for (int it = 0; it < TL; ++it) {
      e[it] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int rt = 0; rt < TL; ++rt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          e[it] = mfma16x16x4(Q[(16 * it + lr) * ldx + 16 * rt + lg + 4 * r], y[rt][r], e[it]);
    }
  }
  double dnew = dj;
#pragma unroll
  for (int it = 0; it < TL; ++it)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (16 * it + lg + 4 * r == j) dnew = dj + e[it][r];
  // G_ij and G_ji are rounded separately; E from their mean is antisymmetric to the last
  // bit, so X stays as orthogonal as it is.  Tile (it, w) meets tile (w, it) of wavefront
  // it through LDS, the tiles at distance s at a time.
#pragma unroll
  for (int st = 0; st <= TL / 2; ++st) {
    lds_barrier();
#pragma unroll
    for (int it = 0; it < TL; ++it) {
      const int fw = (w + st) % TL == it, bw = (w + TL - st) % TL == it;  // uniform
      if (tile && (fw || bw)) {
        double* t = Tc + (2 * w + (fw ? 0 : 1)) * 16 * 17;
#pragma unroll
        for (int r = 0; r < 4; ++r) t[(lg + 4 * r) * 17 + lr] = e[it][r];
      }
    }
    lds_barrier();
#pragma unroll
    for (int it = 0; it < TL; ++it) {
      const int fw = (w + st) % TL == it, bw = (w + TL - st) % TL == it;
      if (tile && (fw || bw)) {
        // the partner wrote its tile for rows w forward if it lies behind, and so on
        const bool pf = (it + st) % TL == w;
        const double* t = Tc + (2 * it + (pf ? 0 : 1)) * 16 * 17;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * it + lg + 4 * r;
          const double gap = dj - (row < m ? S.d[row] : 0.0), gv = 0.5 * (e[it][r] + t[lr * 17 + lg + 4 * r]);
          const bool fit = row < m && j < m && row != j && fabs(gv) < 0x1p-25 * fabs(gap);
          e[it][r] = fit ? gv * rcp2(gap) : 0.0;
        }
      }
    }
  }
  if (tile) {
#pragma unroll
    for (int rt = 0; rt < TL; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) y[rt][r] = Q[j * ldx + 16 * rt + lg + 4 * r];
#pragma unroll
    for (int it = 0; it < TL; ++it)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int rt = 0; rt < TL; ++rt)
          y[rt] = mfma16x16x4(Q[(16 * it + lg + 4 * r) * ldx + 16 * rt + lr], e[it][r], y[rt]);
  }
  lds_barrier();
  if (tile) {
#pragma unroll
    for (int rt = 0; rt < TL; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) Q[j * ldx + 16 * rt + lg + 4 * r] = y[rt][r];
    if (j < m && (j & 3) == lg && dnew == dnew) S.d[j] = dnew;  // (the lane that held the diagonal)
  }
  lds_barrier();
  if (i < m) {
    const double di = S.d[i];
    int r = 0;
    for (int c = q; c < m; c += 4) {
      const double dc = S.d[c];
      r += (dc < di) || (dc == di && c < i);
    }
    r = sum4i(r);
    if (q == 0) {
      S.rank[i] = r;
      a.W[b][r] = ldexp(di, ex);
    }
  }
  lds_barrier();
  double* Vo = global_ptr(a.V[b]);
  for (int c = w; c < m; c += NW) {
    double* v = Vo + (long)S.rank[c] * a.ldv;
    for (int r = lane; r < m; r += 64) v[r] = Q[c * ldx + r];
  }
}

}  // namespace

// Reflectors of a launch stay near this size however large the batch is.
constexpr size_t kReflChunkBytes = size_t(64) << 20;

template <int P, int NT>
static void eig_go(const EigArgs& a, int batch, int mmax, hipStream_t st) {
  static std::once_flag attr;
  std::call_once(attr, [] {
    SL_HIP(hipFuncSetAttribute((const void*)k_eig_dc<P, NT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               160 * 1024));
  });
  sislice_handle* h = current_handle();
  SL_CHECK_ARG(h != nullptr, "no current handle for the eigensolver workspace");
  const int qdoubles = P * (P + 1);
  const size_t lds = sizeof(double) * (qdoubles + std::max(16 * (P + 1), 2 * (P / 16) * 16 * 17)) + (sizeof(Shared) + 15) / 16 * 16;
  const long rstride = (long)P * P;
  const int chunk =
      (int)std::max<size_t>(1, std::min<size_t>(batch, kReflChunkBytes / (rstride * sizeof(double))));
  double* refl = static_cast<double*>(ws_get(h, kBufEigRefl, (size_t)chunk * rstride * sizeof(double)));
  const int tk = prof_begin(h, kProfEig, st);
  for (int c0 = 0; c0 < batch; c0 += chunk) {
    EigArgs c = a;
    c.m = a.m + c0;
    c.A = a.A + c0;
    c.W = a.W + c0;
    c.V = a.V + c0;
    SL_LAUNCH((k_eig_dc<P, NT>), dim3(std::min(chunk, batch - c0)), dim3(NT), lds, st, c, refl,
              rstride, qdoubles);
    SL_LAUNCH_CHECK();
  }
  prof_end(h, tk, st);
}

void eig_launch(const EigArgs& a, int batch, int mmax, hipStream_t st) {
  SL_CHECK_ARG(mmax <= kEigMax, "projected problem too large for the LDS eigensolver");
  if (batch <= 0 || mmax <= 0) return;
  // the kernel of the smallest padded order that holds the batch: fewer wavefronts repeat
  // the reduction's scalar part, and fewer padded columns are carried
  if (mmax <= 32)
    eig_go<32, 128>(a, batch, mmax, st);
  else if (mmax <= 64)
    eig_go<64, 256>(a, batch, mmax, st);
  else if (mmax <= 96)
    eig_go<96, 512>(a, batch, mmax, st);
  else
    eig_go<112, 512>(a, batch, mmax, st);
}

}  // namespace sislice
