// Device-resident Newton step of the reduced-space interior-point iteration.
//
// After the closed-form elimination of y, the slack and the multipliers
// (Eq. 2 with the barrier terms), each Newton step is one dense symmetric
// positive definite solve in x:
//     M = H + diag(d) + s a a^T + delta I,      M dx = r,
// with H the Hessian of the Lagrangian that nnc_eval_hess_lag leaves in HBM.
// Solving it on the GPU keeps the n x n Hessian on the device (only dx
// returns to the host), the step the paper names as future work.
//
// Dense Cholesky M = L L^T in FP64, blocked with 64-column panels; B
// independent systems per call (grid dimension x, so that with a multiple of
// 8 systems each stays on one XCD and its L2).  One launch per panel:
//   * kkt_panel (launch k): the workgroups of panel k first take the update by
//     panel k - 1 of their own 64 x 64 block and of the diagonal block, factor
//     the diagonal block (each workgroup for itself: no launch in between) and
//     solve L_ik = A_ik L_kk^-T; the remaining workgroups apply panel k - 1 to
//     the tiles right of panel k, which the factorisation does not wait for.
//     M is never assembled: launches 0 and 1 read their blocks of A from H and
//     the diagonal and rank-one terms (lower triangle only).
//   * The right-hand side rides along as one more row of the matrix, so y
//     (L y = r) is there after the last panel.
//   * kkt_back: L^T x = y, one workgroup per system.
// A pivot that is not positive (or not finite) stops that system with info =
// its global order (LAPACK's convention: the leading minor of that order is
// not positive definite).  Every sum runs in a fixed order: identical inputs
// give identical bits.
//
// What bounds it: the chain of n / 64 panels, each with 64 dependent pivots;
// the products (n^3 / 3 flops per system) run on v_mfma_f64_16x16x4_f64
// beside it.  16 systems of 784: 557 us, where assembling M and three launches
// per panel took 3,370 us.
#include <math.h>

#include <algorithm>

#include "../../include/nnc.h"
#include "nnc_device.h"
#include "nnc_internal.h"

namespace nnc {

constexpr int KB = 64;          // panel width
constexpr int kKktMaxN = 2048;  // the back substitution keeps y in LDS
constexpr int KP = KB + 2;      // LDS row pitch (doubles) of the diagonal block

// One call's arguments.  The workspace holds the matrix padded to whole
// panels with an identity (np = n rounded up to 64; rows ld apart), so no
// block is ragged; L the factor's blocks below the diagonal ones, D per panel
// the factored diagonal block with its 16 x 16 diagonal blocks inverted (and as
// they are in blocks above the diagonal, kkt_diag_row / kkt_diag_col), R the
// right-hand side as it is reduced and Y its solved blocks.
struct KktArgs {
  const double *H, *d, *a, *s, *delta, *r;
  double *L, *D, *R, *Y;
  int* info;
  int n, np, ld;
};

// N entries (i_e, j_e) of M = H + diag(d) + s a a^T + delta I, read from its
// lower triangle; identity past n.  All loads go out before any is waited for
// (the optional terms are uniform branches around whole groups).
template <int N>
__device__ __forceinline__ void kkt_entries(const KktArgs& g, int b, const int (&i)[N], const int (&j)[N],
                                            double (&v)[N]) {
  const long long bn = (long long)b * g.n;
  const int last = g.n - 1;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const int r = min(max(i[e], j[e]), last), c = min(min(i[e], j[e]), last);
    v[e] = g.H[(bn + r) * g.n + c];
  }
  double t[N];
  if (g.d) {
#pragma unroll
    for (int e = 0; e < N; ++e) t[e] = g.d[bn + min(i[e], last)];
#pragma unroll
    for (int e = 0; e < N; ++e) v[e] = i[e] == j[e] ? v[e] + t[e] : v[e];
  }
  if (g.delta) {
    const double dl = g.delta[b];
#pragma unroll
    for (int e = 0; e < N; ++e) v[e] = i[e] == j[e] ? v[e] + dl : v[e];
  }
  if (g.a) {
    const double sb = g.s[b];
    double u[N];
#pragma unroll
    for (int e = 0; e < N; ++e) {
      t[e] = g.a[bn + min(max(i[e], j[e]), last)];
      u[e] = g.a[bn + min(min(i[e], j[e]), last)];
    }
#pragma unroll
    for (int e = 0; e < N; ++e) v[e] += sb * t[e] * u[e];
  }
#pragma unroll
  for (int e = 0; e < N; ++e)
    if (i[e] > last || j[e] > last) v[e] = i[e] == j[e] ? 1.0 : 0.0;
}

// The same entries of A as panel k finds it: M before the first update has
// been written (k < 2), the workspace after.
template <int N>
__device__ __forceinline__ void kkt_load(const KktArgs& g, int b, int k, const int (&i)[N], const int (&j)[N],
                                         double (&v)[N]) {
  if (k >= 2) {
    const double* Lb = g.L + (long long)b * g.np * g.ld;
#pragma unroll
    for (int e = 0; e < N; ++e) v[e] = Lb[i[e] * g.ld + j[e]];
  } else {  // in four parts, for the registers
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      int ih[N / 4], jh[N / 4];
      double vh[N / 4];
#pragma unroll
      for (int e = 0; e < N / 4; ++e) {
        ih[e] = i[h * (N / 4) + e];
        jh[e] = j[h * (N / 4) + e];
      }
      kkt_entries<N / 4>(g, b, ih, jh, vh);
#pragma unroll
      for (int e = 0; e < N / 4; ++e) v[h * (N / 4) + e] = vh[e];
    }
  }
}

__device__ __forceinline__ doublex4 mma64(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Where a panel's stored diagonal block keeps its diagonal sub-block s.
__device__ __forceinline__ constexpr int kkt_diag_row(int s) { return s == 3 ? 16 : 0; }
__device__ __forceinline__ constexpr int kkt_diag_col(int s) { return s == 3 ? 32 : 16 * (s + 1); }

__device__ __forceinline__ double readlane_d(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// 1 / v and 1 / sqrt(v) of a positive, finite v: Newton's iteration on the
// mantissa from the hardware's estimate (24 bits; each step doubles them), the
// exponent put back, so that the whole FP64 range goes one branch-free way and
// a pivot's wait can be filled with the updates of the step before (the
// full-range division took four times as long).
__device__ __forceinline__ double recip(double v) {
  const double m = __builtin_amdgcn_frexp_mant(v);
  double r = __builtin_amdgcn_rcp(m);
  r = fma(fma(-m, r, 1.0), r, r);
  return __builtin_amdgcn_ldexp(fma(fma(-m, r, 1.0), r, r), -__builtin_amdgcn_frexp_exp(v));
}
__device__ __forceinline__ double recip_sqrt(double v) {
  const int e = __builtin_amdgcn_frexp_exp(v);
  // an even exponent: mantissa in [1/2, 2)
  const double m = __builtin_amdgcn_ldexp(__builtin_amdgcn_frexp_mant(v), e & 1);
  double r = __builtin_amdgcn_rsq(m);
#pragma unroll
  for (int i = 0; i < 2; ++i) r = fma(0.5 * r, fma(-m * r, r, 1.0), r);
  return __builtin_amdgcn_ldexp(r, -((e - (e & 1)) / 2));
}

// Products of this kernel are accumulated transposed: register e of lane l
// holds X[l % 16][4 e + l / 16] of a 16 x 16 block X (row, column), which is
// at once the B operand of K step e of a following product with X^T, so
// chained products need no move between lanes.

// Rows row0 .. row0 + 15 of panel k, column blocks 0 .. nj - 1 of 16: z[jb] =
// A - (update by panel k - 1).  xr: the rows' own elements of panel k - 1
// (kkt_row), Pk: those of rows 64 k .. 64 k + 63.  Lane group q takes columns
// 16 q .. 16 q + 15 of panel k - 1 in both (a fixed order of the sum).
__device__ __forceinline__ void kkt_row(const KktArgs& g, int b, int k, int row0, int lane, double2 (&xr)[8]) {
  const double* p = g.L + ((long long)b * g.np + row0 + (lane & 15)) * g.ld + (k - 1) * KB + 16 * (lane >> 4);
#pragma unroll
  for (int t = 0; t < 8; ++t) xr[t] = *(const double2*)(p + 2 * t);
}

__device__ __forceinline__ void kkt_block(const KktArgs& g, int b, int k, int row0, int nj, int lane,
                                          const double (*Pk)[KP], const double2 (&xr)[8], const double (&av)[16],
                                          doublex4 (&z)[4]) {
  const int c16 = lane & 15, q = lane >> 4;
#pragma unroll
  for (int jb = 0; jb < 4; ++jb) {
    doublex4 acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
    if (k > 0 && jb < nj) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const double2 xk = *(const double2*)&Pk[jb * 16 + c16][16 * q + 2 * t];
        acc[0] = mma64(xk.x, xr[t].x, acc[0]);
        acc[1] = mma64(xk.y, xr[t].y, acc[1]);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) z[jb][e] = av[4 * jb + e] - (acc[0][e] + acc[1][e]);
  }
}

// A's entries of 16 rows from row0, 64 columns of panel k, in z's layout.
__device__ __forceinline__ void kkt_rows_of_a(const KktArgs& g, int b, int k, int row0, int lane, double (&av)[16]) {
  int ii[16], jj[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    ii[e] = row0 + (lane & 15);
    jj[e] = k * KB + 4 * e + (lane >> 4);
  }
  kkt_load<16>(g, b, k, ii, jj, av);
}

// Factor the 16 x 16 block at columns 16 s of S by one wave: lane c < 16 holds
// column c, lane 16 + c column c of the identity, and each pivot step is the
// same row operation on both (multipliers broadcast with readlane), leaving
// D L_u^T and L_u^-1 of the unit-triangular factor L_u.  Writes L = L_u sqrt(D)
// to S and L^-1 to inv; returns 0 or the 1-based order of the first pivot that
// is not positive and finite.
//
// A product with L^-1 is off by L's condition number, which a substitution is
// not.  Whoever multiplies by it corrects the product once with what L leaves of
// the right-hand side, x += L^-1 (b - L x), and has the substitution's residual
// again at the price of two more short products: 256 unknowns of condition
// 1e9, residual relative to |M| |x| 6e-15 without, 4e-17 with (a row-wise
// substitution: 4e-17).  16 systems of 784: 511 -> 564 us.
template <int PITCH>
__device__ __forceinline__ int kkt_factor16(double (*S)[PITCH], int s, double (*inv)[18], int lane) {
  const int c = lane & 15;
  double a[16];
#pragma unroll
  for (int i = 0; i < 16; ++i)
    a[i] = lane < 16 ? S[16 * s + max(i, c)][16 * s + min(i, c)] : (lane < 32 && i == c ? 1.0 : 0.0);
  // The reciprocal of a pivot below 2^-1022 is past the range, and so may be its
  // multiples: a block with a diagonal that small is eliminated with its rows
  // and columns scaled by powers of two, exactly, to diagonals of about 1 (the
  // look at the diagonal: 564 -> 569 us for 16 systems of 784; eliminating again
  // only where a pivot came out small spilled registers, 580 to 612).
  const double dg = S[16 * s + c][16 * s + c];
  const bool tiny = __ballot(dg < 0x1p-900 && dg > 0.0) != 0;
  int h = 0;  // exponent of this column's scale
  if (tiny) {
    h = dg > 0.0 && dg < INFINITY ? -(__builtin_amdgcn_frexp_exp(dg) >> 1) : 0;
    if (lane < 16) {
#pragma unroll
      for (int i = 0; i < 16; ++i) a[i] = __builtin_amdgcn_ldexp(a[i], h + __builtin_amdgcn_readlane(h, i));
    }
  }
  // the next pivot is brought up to date first, and the multipliers are all
  // read before the first is used: its reciprocal, the chain, runs beside them.
  // Multipliers and factor come from the same entries, row j from the diagonal
  // on: (i, c) and (c, i) round differently, and a factor other than the one
  // that was eliminated with is off by the block's condition number.
  double r = recip(readlane_d(a[0], 0));
#pragma unroll
  for (int j = 0; j < 15; ++j) {
    double u[16];
#pragma unroll
    for (int i = j + 1; i < 16; ++i) u[i] = readlane_d(a[j], i);
    const double p = a[j] * r;
    a[j + 1] = fma(-u[j + 1], p, a[j + 1]);
    r = recip(readlane_d(a[j + 1], j + 1));
#pragma unroll
    for (int i = j + 2; i < 16; ++i) a[i] = fma(-u[i], p, a[i]);
  }
  double piv = a[0];  // lane j: pivot j
#pragma unroll
  for (int j = 1; j < 16; ++j) piv = lane == j ? a[j] : piv;
  piv = lane < 16 ? piv : 1.0;
  const unsigned long long bad = __ballot(!(piv > 0.0) || !isfinite(piv));
  const double rs = recip_sqrt(piv);
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    double v = a[j] * readlane_d(rs, j);
    if (tiny) v = __builtin_amdgcn_ldexp(v, lane < 16 ? -h : h);
    if (lane < 16) {
      S[16 * s + c][16 * s + j] = j <= c ? v : 0.0;
    } else if (lane < 32) {
      inv[j][c] = j >= c ? v : 0.0;
    }
  }
  return bad ? __ffsll(bad) : 0;
}

// L^T x = y of one panel's diagonal block by one wave, 16 unknowns at a time:
// lane l holds unknown l.  at(i, s): row 16 s + i of the block in this lane's
// column, the inverted 16 x 16 blocks on the diagonal; diag(i, s): row i of the
// diagonal sub-block s itself in this lane's column of it; only the first `subs`
// sub-blocks hold unknowns.
template <typename At, typename Diag>
__device__ __forceinline__ void kkt_back_block(At at, Diag diag, int subs, int lane, double& yi) {
#pragma unroll
  for (int s = 3; s >= 0; --s) {
    if (s >= subs) continue;
    double xs[16];  // y of sub-block s, x as its product with the inverse, what that leaves of y, then x
    auto dot = [&](auto m) {
      double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i & 3] = fma(m(i, s), xs[i], v[i & 3]);
      return (v[0] + v[1]) + (v[2] + v[3]);
    };
#pragma unroll
    for (int i = 0; i < 16; ++i) xs[i] = readlane_d(yi, 16 * s + i);
    double x0 = 0.0;
    if (lane >> 4 == s) x0 = dot(at);
#pragma unroll
    for (int i = 0; i < 16; ++i) xs[i] = readlane_d(x0, 16 * s + i);
    double left = 0.0;
    if (lane >> 4 == s) left = yi - dot(diag);
#pragma unroll
    for (int i = 0; i < 16; ++i) xs[i] = readlane_d(left, 16 * s + i);
    if (lane >> 4 == s) yi = x0 + dot(at);
    if (s == 0) break;
#pragma unroll
    for (int i = 0; i < 16; ++i) xs[i] = readlane_d(yi, 16 * s + i);
    if (lane < 16 * s) yi -= dot(at);
  }
}

// Launch k (see the head of the file).  gridDim = (B, P + tiles): the first
// P = max(1, panels below k) workgroups of a system factor panel k (workgroup
// y owns row block k + 1 + y), the others take the lower block triangle of
// tiles (I, J), I >= J > k, row by row.
//
// A panel's workgroup: wave 0 factors the diagonal block 16 columns at a time,
// a chain of 64 pivots that everything waits for; waves 1 to 4 (16 rows of the
// diagonal block and 16 of the workgroup's own block each) work beside it:
// the own block's update by panel k - 1 during the first 16 pivots, its
// columns of L during the others'.  Wave 0 brings the next 16 x 16 block up to
// date itself, so that only the solve with the block just factored stands
// between two runs of pivots.  16 systems of 784: 42 us a panel when four waves
// did both in turn, 34 us then; 36 with the corrections of kkt_factor16's products.
//
// ONE: a single panel, solved here too (no panel before it to read).
constexpr int kPanelThreads = 320;
template <bool ONE>
__global__ void __launch_bounds__(kPanelThreads, 3) kkt_panel_kernel(KktArgs g, int panel, double* __restrict__ x) {
  __shared__ __attribute__((aligned(16))) double S[KB + 1][KP];
  __shared__ __attribute__((aligned(16))) double Pk[ONE ? 1 : KB][KP];
  __shared__ double inv[4][16][18];
  __shared__ int s_fail;
  const int b = blockIdx.x;
  const int k = ONE ? 0 : panel;
  if (k > 0 && g.info[b] != 0) return;
  const int nblk = ONE ? 1 : g.np / KB;
  const int below = nblk - k - 1;
  const int P = max(1, below);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int c16 = lane & 15, q = lane >> 4;
  double* Lb = g.L + (long long)b * g.np * g.ld;
  const int kb = k * KB;

  if (!ONE && (int)blockIdx.y >= P) {  // A_IJ -= L_I,k-1 L_J,k-1^T, a 32 x 32 quadrant per wave
    if (wave == 4) return;
    const int t = blockIdx.y - P;
    int ti = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while (ti > 0 && ti * (ti + 1) / 2 > t) --ti;
    while ((ti + 1) * (ti + 2) / 2 <= t) ++ti;
    const int tj = t - ti * (ti + 1) / 2;
    const int i0 = (k + 1 + ti) * KB + 32 * (wave >> 1), j0 = (k + 1 + tj) * KB + 32 * (wave & 1);
    const double* pi = Lb + (long long)(i0 + c16) * g.ld + kb - KB + 16 * q;
    const double* pj = Lb + (long long)(j0 + c16) * g.ld + kb - KB + 16 * q;
    int ii[16], jj[16];
    double av[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      ii[e] = i0 + 16 * (e >> 3) + 4 * (e & 3) + q;
      jj[e] = j0 + 16 * ((e >> 2) & 1) + c16;
    }
    kkt_load<16>(g, b, k, ii, jj, av);
    doublex4 acc[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v) acc[u][v] = doublex4{0, 0, 0, 0};
#pragma unroll 4
    for (int c = 0; c < 16; c += 2) {
      double2 xi[2], xj[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        xi[u] = *(const double2*)(pi + (long long)u * 16 * g.ld + c);
        xj[u] = *(const double2*)(pj + (long long)u * 16 * g.ld + c);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          acc[u][v] = mma64(xi[u].x, xj[v].x, acc[u][v]);
          acc[u][v] = mma64(xi[u].y, xj[v].y, acc[u][v]);
        }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int t = 8 * u + 4 * v + e;
          Lb[ii[t] * g.ld + jj[t]] = av[t] - acc[u][v][e];
        }
    return;
  }

  // rows 64 k .. 64 k + 63 of panel k - 1, the diagonal block's and the
  // right-hand side's entries: all loads before the first wait
  const int gw = wave - 1;  // row group of waves 1 to 4
  double2 pre[7], xr[8];
  double av[16];
  if (k > 0) {
#pragma unroll
    for (int u = 0; u < 7; ++u) {
      const int t = tid + u * kPanelThreads;  // row t / 32, elements 2 (t % 32) and the next
      if (t < KB * 32) pre[u] = *(const double2*)(Lb + (long long)(kb + t / 32) * g.ld + kb - KB + 2 * (t % 32));
    }
  }
  if (wave > 0) {
    if (k > 0) kkt_row(g, b, k, kb + 16 * gw, lane, xr);
    kkt_rows_of_a(g, b, k, kb + 16 * gw, lane, av);
  } else {
    const int i = kb + lane;
    S[KB][lane] = k > 0 ? g.R[(long long)b * g.np + i] : (i < g.n ? g.r[(long long)b * g.n + i] : 0.0);
    if (lane == 0) s_fail = 0;
  }
  if (k > 0) {
#pragma unroll
    for (int u = 0; u < 7; ++u) {
      const int t = tid + u * kPanelThreads;
      if (t < KB * 32) *(double2*)&Pk[t / 32][2 * (t % 32)] = pre[u];
    }
  }
  __syncthreads();
  doublex4 z[4];
  if (wave > 0) {
    kkt_block(g, b, k, kb + 16 * gw, gw + 1, lane, Pk, xr, av, z);
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
      if (jb <= gw) {
#pragma unroll
        for (int e = 0; e < 4; ++e) S[16 * gw + c16][16 * jb + 4 * e + q] = z[jb][e];
      }
  }
  __syncthreads();
  const int row0 = (k + 1 + blockIdx.y) * KB + 16 * gw;  // this wave's rows of the own block
  double dot = 0.0;                                      // this lane's part of (L_ik y_k)
  // X^T = L_ss^-1 B^T for 16 rows of B in z's layout, corrected once
  auto solve16 = [&](int s, const doublex4& w) {
    doublex4 xs = {0, 0, 0, 0}, lx = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < 4; ++e) xs = mma64(inv[s][c16][4 * e + q], w[e], xs);
#pragma unroll
    for (int e = 0; e < 4; ++e) lx = mma64(S[16 * s + c16][16 * s + 4 * e + q], xs[e], lx);
    const doublex4 left = w - lx;
#pragma unroll
    for (int e = 0; e < 4; ++e) xs = mma64(inv[s][c16][4 * e + q], left[e], xs);
    return xs;
  };
  // X_s^T = L_ss^-1 (A_s^T - sum_{t < s} L_st X_t^T) of the own rows
  auto own_columns = [&](int s) {
    doublex4 acc = {0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < 3; ++t)
      if (t < s) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = mma64(S[16 * s + c16][16 * t + 4 * e + q], z[t][e], acc);
      }
    const doublex4 w = (s == 0 ? z[0] : s == 1 ? z[1] : s == 2 ? z[2] : z[3]) - acc;
    const doublex4 xs = solve16(s, w);
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (t == s) z[t] = xs;
    double* o = Lb + (long long)(row0 + c16) * g.ld + kb + 16 * s + q;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[4 * e] = xs[e];
      dot = fma(xs[e], S[KB][16 * s + 4 * e + q], dot);
    }
  };
  // S[row][16 j ..] -= (column block s of row) (column block s of block row j)^T
  auto trail = [&](int s, int i, int j) {
    const bool rhs = i == 4;
    const int row = rhs ? KB : 16 * i + c16;
    doublex4 acc = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double bv = !rhs || c16 == 0 ? S[row][16 * s + 4 * e + q] : 0.0;
      acc = mma64(S[16 * j + c16][16 * s + 4 * e + q], bv, acc);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (!rhs || c16 == 0) S[row][16 * j + 4 * e + q] -= acc[e];
  };
  const int subs = min(4, (g.n - kb + 15) / 16);  // sub-blocks that are not all padding
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if (wave == 0) {
      const int f = kkt_factor16(S, s, inv[s], lane);
      if (f && lane == 0) s_fail = kb + 16 * s + f;
    } else if (below > 0) {
      if (s == 0) {
        if (k > 0) kkt_row(g, b, k, row0, lane, xr);
        kkt_rows_of_a(g, b, k, row0, lane, av);
        kkt_block(g, b, k, row0, 4, lane, Pk, xr, av, z);
      } else {
        own_columns(s - 1);
      }
    }
    __syncthreads();
    if (s_fail) {
      if (blockIdx.y == 0 && tid == 0) g.info[b] = s_fail;
      if (ONE && tid < g.n) x[(long long)b * g.n + tid] = 0.0;
      return;
    }
    // blocks below (row group i > s; wave 0: the right-hand side): X = A L_ss^-T
    const bool rhs = wave == 0;
    if (rhs || gw > s) {
      const int row = rhs ? KB : 16 * gw + c16;
      doublex4 bv;
#pragma unroll
      for (int e = 0; e < 4; ++e) bv[e] = !rhs || c16 == 0 ? S[row][16 * s + 4 * e + q] : 0.0;
      const doublex4 xs = solve16(s, bv);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (!rhs || c16 == 0) S[row][16 * s + 4 * e + q] = xs[e];
    }
    __syncthreads();
    if (s == 3 || s + 1 == subs) break;
    // block (s + 1, s + 1) by wave 0, the others (i = 4: the right-hand side) by the row groups
    if (wave == 0) {
      trail(s, s + 1, s + 1);
    } else {
      int id = 0;
#pragma unroll
      for (int j = s + 1; j < 4; ++j)
#pragma unroll
        for (int i = j; i <= 4; ++i) {
          if (i == s + 1 && j == s + 1) continue;
          if ((id++ & 3) == gw) trail(s, i, j);
        }
    }
  }
  if (blockIdx.y == 0) {
    if constexpr (!ONE) {
      double* Dk = g.D + ((long long)b * nblk + k) * KB * KB;
      for (int idx = tid; idx < KB * KB; idx += kPanelThreads) {
        const int i = idx / KB, j = idx % KB;
        if (i / 16 == j / 16) {
          Dk[idx] = i / 16 < subs ? inv[i / 16][i % 16][j % 16] : i == j ? 1.0 : 0.0;
          Dk[(kkt_diag_row(i / 16) + i % 16) * KB + kkt_diag_col(i / 16) + j % 16] = S[i][j];
        } else if (i > j) {
          Dk[idx] = S[i][j];
        }
      }
      if (tid < KB) g.Y[(long long)b * g.np + kb + tid] = S[KB][tid];
    } else if (wave == 0) {  // one panel: L^T x = y here
      double yi = S[KB][lane];
      kkt_back_block([&](int i, int s) { return lane >> 4 == s ? inv[s][i][c16] : S[16 * s + i][lane]; },
                     [&](int i, int s) { return S[16 * s + i][16 * s + c16]; }, subs, lane, yi);
      if (lane < g.n) x[(long long)b * g.n + lane] = yi;
    }
    if (k == 0 && tid == 0) g.info[b] = 0;
  }
  if (wave == 0 || below == 0) return;
  own_columns(3);
  dot += __shfl_xor(dot, 16, 64);
  dot += __shfl_xor(dot, 32, 64);
  if (q == 0) {
    const int i = row0 + c16;
    double* R = g.R + (long long)b * g.np + i;
    const double rv = k > 0 ? *R : (i < g.n ? g.r[(long long)b * g.n + i] : 0.0);
    *R = rv - dot;
  }
}

// Up to 16 unknowns: a wave per system, four systems per workgroup.  A panel's
// workgroup would factor one 16 x 16 block of its four with one wave of its five.
// 20,000 systems of 2, 8 and 16 unknowns: 1,587 us each there, 51 here.
constexpr int kKktSmall = 16;
__global__ void __launch_bounds__(256) kkt_small_kernel(KktArgs g, int B, double* __restrict__ x) {
  __shared__ double Sall[4][16][18], invall[4][16][18];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = lane & 15;
  double (*S)[18] = Sall[wave];
  double (*inv)[18] = invall[wave];
  const bool live = (int)blockIdx.x * 4 + wave < B;
  const int b = min((int)blockIdx.x * 4 + wave, B - 1);
  int ii[4], jj[4];
  double v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    ii[e] = 4 * e + (lane >> 4);
    jj[e] = c;
  }
  kkt_entries<4>(g, b, ii, jj, v);
  const double r = lane < g.n ? g.r[(long long)b * g.n + lane] : 0.0;
#pragma unroll
  for (int e = 0; e < 4; ++e) S[ii[e]][c] = v[e];
  __syncthreads();
  const int f = kkt_factor16(S, 0, inv, lane);
  __syncthreads();
  auto dot = [&](auto m, double y) {  // sum over i of m(i) and lane i's y
    double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 16; ++i) t[i & 3] = fma(m(i), readlane_d(y, i), t[i & 3]);
    return (t[0] + t[1]) + (t[2] + t[3]);
  };
  auto row = [&](int i) { return S[c][i]; };
  auto col = [&](int i) { return S[i][c]; };
  auto irow = [&](int i) { return inv[c][i]; };
  auto icol = [&](int i) { return inv[i][c]; };
  double y = dot(irow, r);
  y += dot(irow, r - dot(row, y));
  double xv = dot(icol, y);
  xv += dot(icol, y - dot(col, xv));
  if (!live) return;
  if (lane == 0) g.info[b] = f;
  if (lane < g.n) x[(long long)b * g.n + lane] = f ? 0.0 : xv;
}

// L^T x = y, one workgroup of 16 waves per system: wave 0 solves a panel's 64
// unknowns from the diagonal block in LDS (16 at a time through the inverted
// 16 x 16 blocks), then all threads take them out of the unknowns above,
// reading the panel's rows of L once, along the rows.  Bound by what one CU
// reads (half of the matrix) and the n / 64 panels in turn.
__global__ void __launch_bounds__(1024) kkt_back_kernel(KktArgs g, double* __restrict__ x) {
  __shared__ double y[kKktMaxN];
  __shared__ double D[KB][KB + 1];
  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  double* xb = x + (long long)b * g.n;
  if (g.info[b] != 0) {
    for (int i = tid; i < g.n; i += 1024) xb[i] = 0.0;
    return;
  }
  const int nblk = g.np / KB;
  const double* Lb = g.L + (long long)b * g.np * g.ld;
  for (int i = tid; i < g.np; i += 1024) y[i] = g.Y[(long long)b * g.np + i];
  double dreg[4];
  auto load_diag = [&](int k) {
    const double* Dk = g.D + ((long long)b * nblk + k) * KB * KB;
#pragma unroll
    for (int u = 0; u < 4; ++u) dreg[u] = Dk[u * 1024 + tid];
  };
  load_diag(nblk - 1);
  for (int k = nblk - 1; k >= 0; --k) {
    const int kb = k * KB;
#pragma unroll
    for (int u = 0; u < 4; ++u) D[(u * 1024 + tid) / KB][tid % KB] = dreg[u];
    __syncthreads();
    if (k > 0) load_diag(k - 1);
    // this thread's column of the panel's first rows, on the way meanwhile
    constexpr int PF = 16;
    const double* p = Lb + (long long)kb * g.ld + tid;
    double pre[PF];
#pragma unroll
    for (int i = 0; i < PF; ++i) pre[i] = tid < kb ? p[(long long)i * g.ld] : 0.0;
    if (tid < 64) {
      double yi = y[kb + lane];
      kkt_back_block([&](int i, int s) { return D[16 * s + i][lane]; },
                     [&](int i, int s) { return D[kkt_diag_row(s) + i][kkt_diag_col(s) + (lane & 15)]; }, 4, lane, yi);
      y[kb + lane] = yi;
      if (kb + lane < g.n) xb[kb + lane] = yi;
    }
    __syncthreads();
    if (tid < kb) {
      double v = 0.0;
      double rest[KB - PF];
#pragma unroll
      for (int i = PF; i < KB; ++i) rest[i - PF] = p[(long long)i * g.ld];
#pragma unroll
      for (int i = 0; i < PF; ++i) v = fma(pre[i], y[kb + i], v);
#pragma unroll
      for (int i = PF; i < KB; ++i) v = fma(rest[i - PF], y[kb + i], v);
      y[tid] -= v;
    }
    for (int j = 1024 + tid; j < kb; j += 1024) {
      const double* pj = Lb + (long long)kb * g.ld + j;
      double v = 0.0;
#pragma unroll 32
      for (int i = 0; i < KB; ++i) v = fma(pj[(long long)i * g.ld], y[kb + i], v);
      y[j] -= v;
    }
    // the next round's barrier stands between these updates and wave 0's read
  }
}

struct Kkt {
  int n = 0, maxB = 0;
  int np = 0, ld = 0;
  int wsB = 0;          // systems the workspace holds
  double* L = nullptr;  // one allocation: L, D, R, Y of KktArgs (NULL for one panel)
};

// Doubles of one system's workspace (KktArgs): rows of L 16 doubles past a
// multiple of 64 apart, so that the rows of a tile spread over the channels.
inline size_t kkt_words(const Kkt* k) { return (size_t)k->np * k->ld + (size_t)k->np * KB + 2 * (size_t)k->np; }

void free_kkts(Ctx* c) {
  for (void* p : c->kkts) {
    Kkt* k = (Kkt*)p;
    if (!k) continue;
    hipFree(k->L);
    delete k;
  }
  c->kkts.clear();
}

}  // namespace nnc

using namespace nnc;

namespace {
int kkt_fail(Ctx* c, int code, const char* msg) {
  if (c) c->err = msg;
  return code;
}
}  // namespace

extern "C" {

int nnc_kkt_create(nnc_ctx ctx, int n, int max_B, int* kkt) {
  Ctx* c = (Ctx*)ctx;
  if (!c || !kkt) return kkt_fail(c, NNC_E_ARG, "null argument");
  if (n < 1 || n > kKktMaxN || max_B < 1) return kkt_fail(c, NNC_E_SHAPE, "n outside 1..2048 or max_B < 1");
  if (hipSetDevice(c->device) != hipSuccess) return kkt_fail(c, NNC_E_HIP, "hipSetDevice failed");
  Kkt* k = new Kkt();
  k->n = n;
  k->maxB = max_B;
  k->np = (n + KB - 1) / KB * KB;
  k->ld = k->np + 16;
  // One panel is factored and solved in LDS.  Otherwise the workspace is up to
  // six times H (65 unknowns): where it does not fit for all systems, it holds
  // as many as do and a call takes them in turn.
  k->wsB = max_B;
  while (k->np > KB && hipMalloc(&k->L, (size_t)k->wsB * kkt_words(k) * sizeof(double)) != hipSuccess) {
    (void)hipGetLastError();
    k->L = nullptr;
    if (k->wsB == 1) {
      delete k;
      return kkt_fail(c, NNC_E_NOMEM, "KKT factor workspace");
    }
    k->wsB = (k->wsB + 1) / 2;
  }
  c->kkts.push_back(k);
  *kkt = (int)c->kkts.size() - 1;
  return NNC_OK;
}

int nnc_kkt_destroy(nnc_ctx ctx, int kkt) {
  Ctx* c = (Ctx*)ctx;
  if (!c || kkt < 0 || kkt >= (int)c->kkts.size() || !c->kkts[kkt]) return kkt_fail(c, NNC_E_ARG, "invalid KKT handle");
  Kkt* k = (Kkt*)c->kkts[kkt];
  hipStreamSynchronize(c->stream);
  hipFree(k->L);
  delete k;
  c->kkts[kkt] = nullptr;
  return NNC_OK;
}

int nnc_kkt_solve(nnc_ctx ctx, int kkt, int B, const double* H, const double* d, const double* a, const double* s,
                  const double* delta, const double* r, double* dx, int* info) {
  Ctx* c = (Ctx*)ctx;
  if (!c || kkt < 0 || kkt >= (int)c->kkts.size() || !c->kkts[kkt]) return kkt_fail(c, NNC_E_ARG, "invalid KKT handle");
  Kkt* k = (Kkt*)c->kkts[kkt];
  if (B < 0 || B > k->maxB) return kkt_fail(c, NNC_E_SHAPE, "B outside [0, max_B]");
  if (B == 0) return NNC_OK;
  if (!H || !r || !dx || !info) return kkt_fail(c, NNC_E_ARG, "null H, r, dx or info");
  if ((a == nullptr) != (s == nullptr)) return kkt_fail(c, NNC_E_ARG, "a and s must be given together");
  if (hipSetDevice(c->device) != hipSuccess) return kkt_fail(c, NNC_E_HIP, "hipSetDevice failed");
  const int n = k->n;
  const long long total = (long long)B * n * n;
  if ((total + 255) / 256 > 0x7fffffffLL) return kkt_fail(c, NNC_E_SHAPE, "B * n * n too large");
  ProfRec pr;
  prof_begin(c, NNC_KC_OTHER, &pr);
  const int nblk = k->np / KB;
  for (int b0 = 0, nb = 0; b0 < B; b0 += nb) {
    nb = std::min(k->wsB, B - b0);
    const long long o = (long long)b0 * n;
    KktArgs g;
    g.H = H + o * n;
    g.d = d ? d + o : nullptr;
    g.a = a ? a + o : nullptr;
    g.s = s ? s + b0 : nullptr;
    g.delta = delta ? delta + b0 : nullptr;
    g.r = r + o;
    g.info = info + b0;
    g.n = n;
    g.np = k->np;
    g.ld = k->ld;
    g.L = k->L;
    g.D = nblk > 1 ? g.L + (size_t)nb * k->np * k->ld : nullptr;
    g.R = nblk > 1 ? g.D + (size_t)nb * k->np * KB : nullptr;
    g.Y = nblk > 1 ? g.R + (size_t)nb * k->np : nullptr;
    if (n <= kKktSmall) {
      hipLaunchKernelGGL(kkt_small_kernel, dim3((nb + 3) / 4), dim3(256), 0, c->stream, g, nb, dx + o);
      continue;
    }
    if (nblk == 1) {
      hipLaunchKernelGGL(kkt_panel_kernel<true>, dim3(nb), dim3(kPanelThreads), 0, c->stream, g, 0, dx + o);
      continue;
    }
    for (int p = 0; p < nblk; ++p) {
      const int below = nblk - p - 1;
      const int tiles = p > 0 ? below * (below + 1) / 2 : 0;
      hipLaunchKernelGGL(kkt_panel_kernel<false>, dim3(nb, (below > 0 ? below : 1) + tiles), dim3(kPanelThreads), 0,
                         c->stream, g, p, dx + o);
    }
    hipLaunchKernelGGL(kkt_back_kernel, dim3(nb), dim3(1024), 0, c->stream, g, dx + o);
  }
  const hipError_t e = hipGetLastError();
  prof_end(c, &pr);
  if (e != hipSuccess) {
    c->err = std::string("KKT kernels: ") + hipGetErrorString(e);
    return NNC_E_HIP;
  }
  return NNC_OK;
}

}  // extern "C"
