// Overlap, log-determinant and Green's function of every (walker, path) pair
// (Sec. III.A, Eqs. ratio-update-phi and sign-path; Theta feeds Eq. local-obs).
//
// One wavefront handles two paths, both spins of each, 16 lanes (rows) apiece:
//  1. A^s = Phi_T^T phi^s (N x N complex) on the FP64 matrix cores, one path after the
//     other, operands read straight from HBM (real trial times the re / im parts of phi);
//  2. elimination with partial pivoting, one lane per row, pivot rows found by a
//     16-lane max over DPP moves and a ballot (largest |a|^2, lowest row on ties)
//     and broadcast by lane shuffles instead of swapped;
//     det = parity(perm) prod u_kk, accumulated as a scaled complex product;
//  3. with Theta or the Green's function diagonal requested the elimination is
//     Gauss-Jordan in place, which leaves X^s = (A^s)^{-1} in the rows: X^s goes to LDS,
//     Theta^s = phi^s X^s runs on the matrix cores (four real products per
//     spin), is stored as whole 16-byte complex entries along each row, and the
//     diagonal Re (G_up + G_dn)_mm = Re sum_s sum_n Theta^s_mn Phi_T,mn is summed from
//     its tiles.
// A zero pivot marks the path singular: l = -inf + 0i and Theta = 0, diag = 0.
// A non-finite overlap entry gives l = NaN + NaN i (Theta and diag 0).
//
// FP32 contexts' Theta (the FP32 contraction rounds it to FP32, see k_overlap_lu.hip) comes
// from an LU factorisation and triangular solves instead, unrolled over rows and columns: lane
// (path, spin, j) solves z U = e_j, v L = z, X[j][perm[k]] = v[k].  With a workgroup per path
// (k_overlap_lu) and here: M = 24, N = 6, 4000 paths 67 and 27 us; M = 48, N = 12, 4000 paths 108 and
// 58; M = 64, N = 16, 4096 paths 138 and 76, but 120 paths 35 and 49: calls that leave the chip
// part empty run there for N > 8 (overlap_lu_wide).  Both give the same bits.
//
// The elimination is a loop: after a step every row moves up one register, so that the
// pivot column is always register 0 and one step's code serves all.  Unrolled over columns
// and steps it was 82 KB of code, past the instruction cache (64 KB for two CUs), and the
// passes over it set the time; now 5 to 11 KB.  Two paths fill the wavefront's 64 lanes.
// Bound by the serial chain of a step (pivot search, reciprocal, broadcasts), with Theta also
// by its writes.  Measured, before and now, log-overlaps / with Theta: M = 64, N = 16, 4096
// paths 58 -> 40 / 111 -> 79 us; M = 48, N = 12, 4000 paths 49 -> 28 / 85 -> 55; M = 16,
// N = 8, 300 paths 16 -> 10 / 24 -> 14; M = 8, N = 2, 512 paths 9.6 -> 9.8 / 13.2 -> 10.6.
#include "afqmc_internal.h"
#include "dev_common.h"

namespace {

constexpr int OV_WAVES = 4;

// Elimination with partial pivoting of four matrices, 16 lanes (rows) each: the pivots'
// product as log|det| and its argument, whether a pivot was zero, the step that took this
// lane's row as its pivot row (-1: none) and 1 / its pivot; INV: the rows of the inverse
// (unscaled).
template <int NC, bool INV>
__device__ __forceinline__ void eliminate(cplx (&a)[NC], int N, int lane, int& mystep, cplx& scale,
                                          double& logabs, double& argsum, bool& singular) {
  const int i = lane & 15;
  bool used = i >= N;
  mystep = -1;
  scale = cmk(0.0, 0.0);
  // det = prod of pivots, kept as a complex mantissa times 2^pexp so that it
  // neither overflows nor needs a logarithm per step
  cplx pprod = cmk(1.0, 0.0);
  int pexp = 0, inv = 0;
  unsigned done = 0;  // pivot rows so far
  singular = false;
  // step k on the first W registers.  INV: Gauss-Jordan in place; column k of the
  // inverse takes the place of the pivot column, and pivot rows stay unscaled (row
  // `scale` times the registers) as every update is linear in the row it changes.
  auto step = [&](auto WW, int k) {
    constexpr int W = decltype(WW)::value;
    // NaN entries count as zero so that the order is total and every lane of the
    // group agrees on the pivot
    double v = used ? -1.0 : cabs2(a[0]);
    if (!used && !(v >= 0.0)) v = 0.0;
    double vm = fmax(v, dpp_f64<0xB1>(v));
    vm = fmax(vm, dpp_f64<0x4E>(vm));
    vm = fmax(vm, dpp_f64<0x141>(vm));
    vm = fmax(vm, dpp_f64<0x140>(vm));
    const unsigned cand = (unsigned)(__ballot(!used && v == vm) >> (lane & 48)) & 0xffffu;
    const int prow = __builtin_ctz(cand | 0x10000u) & 15;  // uniform within the group
    inv += __builtin_popcount(done >> prow);
    done |= 1u << prow;
    const int src = (lane & 48) + prow;
    const cplx piv = cmk(__shfl(a[0].re, src, 64), __shfl(a[0].im, src, 64));
    if (!(vm > 0.0)) singular = true;
    const bool mine = i == prow;
    if (mine) {
      used = true;
      mystep = k;
    }
    pprod = cmul(pprod, piv);
    const double mx = fmax(fabs(pprod.re), fabs(pprod.im));
    if (mx > 0.0 && isfinite(mx)) {
      const int ex = ilogb(mx);
      pprod = cscale(pprod, ldexp(1.0, -ex));
      pexp += ex;
    }
    const cplx rp = crecip(piv);  // the pivot's reciprocal: one real division
    if (INV && mine) scale = rp;
    cplx l = cmul(a[0], rp);
    if (mine || singular || (!INV && used)) l = cmk(0.0, 0.0);
#pragma unroll
    for (int j = 0; j + 1 < W; ++j) {
      const cplx pj = cmk(__shfl(a[j + 1].re, src, 64), __shfl(a[j + 1].im, src, 64));
      a[j] = cfms(a[j + 1], l, pj);
    }
    if (INV) a[W - 1] = mine ? cmk(1.0, 0.0) : cmk(-l.re, -l.im);
  };
  if constexpr (INV) {
#pragma unroll 1
    for (int k = 0; k < N; ++k) step(std::integral_constant<int, NC>{}, k);
  } else {
    int k = 0;
    unrolled<NC / 8>([&](auto I) {  // N - k columns are left: W, W - 8
      constexpr int W = NC - 8 * decltype(I)::value;
#pragma unroll 1
      for (; k < N - W + 8; ++k) step(std::integral_constant<int, W>{}, k);
    });
  }
  logabs = 0.5 * log(cabs2(pprod)) + (double)pexp * M_LN2;
  argsum = atan2(pprod.im, pprod.re) + ((inv & 1) ? M_PI : 0.0);
}

// LU factors in place with partial pivoting of four matrices, 16 lanes (rows) each, the pivots,
// their product, mystep and singular as eliminate's: the row of step k holds U from column k
// on and L's multipliers before it
template <int NC>
__device__ __forceinline__ void factor(cplx (&a)[NC], int N, int lane, int& mystep, double& logabs,
                                       double& argsum, bool& singular) {
  const auto mul = [](cplx x, cplx y) {
    return cmk(fma(x.re, y.re, -(x.im * y.im)), fma(x.im, y.re, x.re * y.im));
  };
  const auto abs2 = [](cplx x) { return fma(x.re, x.re, x.im * x.im); };
  const auto recip = [](cplx x) {  // crecip
    const double m = fmax(fabs(x.re), fabs(x.im));
    const int e = (m > 0.0 && isfinite(m)) ? ilogb(m) : 0;
    const double r = ldexp(x.re, -e), t = ldexp(x.im, -e);
    const double d = 1.0 / fma(r, r, t * t);
    return cmk(ldexp(r * d, -e), ldexp(-t * d, -e));
  };
  const int i = lane & 15;
  bool used = i >= N;
  mystep = -1;
  cplx pprod = cmk(1.0, 0.0);
  int pexp = 0, inv = 0;
  unsigned done = 0;
  singular = false;
  unrolled<NC>([&](auto K) {
    constexpr int k = decltype(K)::value;
    if (k >= N) return;
    double v = used ? -1.0 : abs2(a[k]);
    if (!used && !(v >= 0.0)) v = 0.0;
    double vm = fmax(v, dpp_f64<0xB1>(v));
    vm = fmax(vm, dpp_f64<0x4E>(vm));
    vm = fmax(vm, dpp_f64<0x141>(vm));
    vm = fmax(vm, dpp_f64<0x140>(vm));
    const unsigned cand = (unsigned)(__ballot(!used && v == vm) >> (lane & 48)) & 0xffffu;
    const int prow = __builtin_ctz(cand | 0x10000u) & 15;  // uniform within the group
    inv += __builtin_popcount(done >> prow);
    done |= 1u << prow;
    const int src = (lane & 48) + prow;
    const cplx piv = cmk(__shfl(a[k].re, src, 64), __shfl(a[k].im, src, 64));
    if (!(vm > 0.0)) singular = true;
    if (i == prow) {
      used = true;
      mystep = k;
    }
    pprod = mul(pprod, piv);
    const double mx = fmax(fabs(pprod.re), fabs(pprod.im));
    if (mx > 0.0 && isfinite(mx)) {
      const int ex = ilogb(mx);
      pprod = cscale(pprod, ldexp(1.0, -ex));
      pexp += ex;
    }
    const bool live = !used && !singular;
    cplx l = cmk(0.0, 0.0);
    if (live) {
      l = mul(a[k], recip(piv));  // the pivot's reciprocal: one real division
      a[k] = l;
    }
#pragma unroll
    for (int j = k + 1; j < NC; ++j) {
      const cplx pj = cmk(__shfl(a[j].re, src, 64), __shfl(a[j].im, src, 64));
      if (live) a[j] = cfms(a[j], l, pj);
    }
  });
  logabs = fma((double)pexp, M_LN2, 0.5 * log(abs2(pprod)));
  argsum = atan2(pprod.im, pprod.re) + ((inv & 1) ? M_PI : 0.0);
}

enum { OV_DET = 0, OV_INV = 1, OV_LU = 2 };

// NC: columns of a row in registers (N <= NC).  MODE: log-overlaps only, or with Theta or the
// diagonal from the inverse (OV_INV) or Theta from LU factors (OV_LU)
template <int NC, int MODE>
__global__ void __launch_bounds__(OV_WAVES * 64, 2)
k_overlap(int n_samples, int P, int M, int N, const double* __restrict__ phi,
          const double* __restrict__ phiT, double* __restrict__ logov, double* __restrict__ theta,
          double* __restrict__ gdiag) {
  __shared__ double s_lu[OV_WAVES][4][NC][NC + 1][2];  // [path, spin]: A, then X
  __shared__ int s_perm[OV_WAVES][4][NC];

  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, c = lane & 15;
  const int s0 = (blockIdx.x * OV_WAVES + wave) * 2;
  if (s0 >= n_samples) return;  // no block-level barriers below
  const auto fence = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  };

  // 1. A^s: tiles (re up, im up, re dn, im dn); lane holds A[g+4r][c].  A lone last path
  // takes both places.
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    const int s = min(s0 + h, n_samples - 1);
    const double* pT = phiT + (size_t)s * M * N;
    const double* pw = phi + (size_t)(s / P) * 2 * M * N * 2;
    dx4 acc[4] = {dx4_zero(), dx4_zero(), dx4_zero(), dx4_zero()};
#pragma unroll 4
    for (int q = 0; q < (M + 3) / 4; ++q) {
      const int m = 4 * q + g;
      const bool ok = m < M && c < N;
      const size_t e = (size_t)min(m, M - 1) * N + min(c, N - 1);
      const double a = keep_if(pT[e], ok);
#pragma unroll
      for (int sp = 0; sp < 2; ++sp) {
        const double2 x = *reinterpret_cast<const double2*>(pw + ((size_t)sp * M * N + e) * 2);
        acc[2 * sp] = mfma_f64(a, keep_if(x.x, ok), acc[2 * sp]);
        acc[2 * sp + 1] = mfma_f64(a, keep_if(x.y, ok), acc[2 * sp + 1]);
      }
    }
#pragma unroll
    for (int sp = 0; sp < 2; ++sp)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (NC == 16 || (g + 4 * r < NC && c < NC)) {
          s_lu[wave][2 * h + sp][g + 4 * r][c][0] = acc[2 * sp][r];
          s_lu[wave][2 * h + sp][g + 4 * r][c][1] = acc[2 * sp + 1][r];
        }
  }
  fence();

  // 2. elimination: lane = (path, spin, row i)
  const int i = c;
  cplx a[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    a[j] = cmk(s_lu[wave][g][min(i, NC - 1)][j][0], s_lu[wave][g][min(i, NC - 1)][j][1]);
    if (NC < 16 && i >= NC) a[j] = cmk(0.0, 0.0);
  }
  fence();
  // a non-finite entry of either spin's overlap matrix makes l NaN (a
  // numerical event, not a singular path)
  double nf = 0.0;
#pragma unroll
  for (int j = 0; j < NC; ++j) nf = fma(a[j].re, 0.0, fma(a[j].im, 0.0, nf));
  const bool nf_any = ((__ballot(nf != 0.0) >> (lane & 32)) & 0xffffffffull) != 0;  // the path's
  int mystep;
  cplx scale;
  double logabs, argsum;
  bool singular;
  if constexpr (MODE == OV_LU)
    factor<NC>(a, N, lane, mystep, logabs, argsum, singular);
  else
    eliminate<NC, MODE == OV_INV>(a, N, lane, mystep, scale, logabs, argsum, singular);

  // both spins' results to the lanes of the path's first spin
  const double la_dn = __shfl(logabs, (lane & 32) + 16, 64);
  const double ar_dn = __shfl(argsum, (lane & 32) + 16, 64);
  const bool sing_any =
      (__shfl((int)singular, lane & 32, 64) | __shfl((int)singular, (lane & 32) + 16, 64)) != 0;
  if ((lane & 31) == 0 && s0 + (lane >> 5) < n_samples) {
    double* o = logov + (size_t)(s0 + (lane >> 5)) * 2;
    if (nf_any) {
      o[0] = __builtin_nan("");
      o[1] = __builtin_nan("");
    } else if (sing_any) {
      o[0] = neg_inf();
      o[1] = 0.0;
    } else {
      o[0] = logabs + la_dn;
      o[1] = argsum + ar_dn;
    }
  }
  if constexpr (MODE == OV_DET) return;

  // 3. X^s = (A^s)^{-1}: the row of step k is X's row k, and register NC - N + m its column
  //    perm[m]; the rest is zero
  const unsigned long long deadm = __ballot(sing_any || nf_any);
  if (mystep >= 0) s_perm[wave][g][mystep] = i;
  if constexpr (MODE == OV_LU) {
    if (mystep >= 0)
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        s_lu[wave][g][mystep][j][0] = a[j].re;
        s_lu[wave][g][mystep][j][1] = a[j].im;
      }
    fence();
    auto lu = [&](int k, int j) { return cmk(s_lu[wave][g][k][j][0], s_lu[wave][g][k][j][1]); };
#pragma unroll
    for (int j = 0; j < NC; ++j) a[j] = cmk(j == i ? 1.0 : 0.0, 0.0);
#pragma unroll
    for (int j = 0; j < NC; ++j)
      if (j < N) {
#pragma unroll
        for (int k = 0; k < j; ++k) a[j] = cfms(a[j], a[k], lu(k, j));
        a[j] = cdiv(a[j], lu(j, j));
      }
#pragma unroll
    for (int j = NC - 1; j >= 0; --j)
      if (j < N)
#pragma unroll
        for (int k = j + 1; k < NC; ++k)
          if (k < N) a[j] = cfms(a[j], a[k], lu(k, j));
    fence();  // the factors are read
  }
  if (i < NC)
#pragma unroll
    for (int j = 0; j < NC; ++j) s_lu[wave][g][i][j][0] = s_lu[wave][g][i][j][1] = 0.0;
  fence();
  if constexpr (MODE == OV_LU) {
    if (i < N)
#pragma unroll
      for (int k = 0; k < NC; ++k)
        if (k < N) {
          const int col = s_perm[wave][g][k] & (NC - 1);
          s_lu[wave][g][i][col][0] = a[k].re;
          s_lu[wave][g][i][col][1] = a[k].im;
        }
  } else if (mystep >= 0) {
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int m = j - (NC - N);
      if (m >= 0) {
        const cplx x = cmul(a[j], scale);
        const int col = s_perm[wave][g][m];
        s_lu[wave][g][mystep][col][0] = x.re;
        s_lu[wave][g][mystep][col][1] = x.im;
      }
    }
  }
  fence();
  // 4. Theta^s = phi^s X^s on the matrix cores: A[c][g] = phi[16t + c][4q + g],
  //    B[g][c] = X[4q + g][c]; the lane holds Theta[16t + g + 4r][c]
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    const int s = s0 + h;
    if (s >= n_samples) break;
    double* th = theta ? theta + (size_t)s * 2 * M * N * 2 : nullptr;
    double* gd = gdiag ? gdiag + (size_t)s * M : nullptr;
    if ((deadm >> (32 * h)) & 1) {
      if (th)
        for (int q = lane; q < 2 * M * N * 2; q += 64) th[q] = 0.0;
      if (gd)
        for (int q = lane; q < M; q += 64) gd[q] = 0.0;
      continue;
    }
    const double* pT = phiT + (size_t)s * M * N;
    const double* pw = phi + (size_t)(s / P) * 2 * M * N * 2;
    double xr[2][NC / 4], xi[2][NC / 4];
#pragma unroll
    for (int sp = 0; sp < 2; ++sp)
#pragma unroll
      for (int q = 0; q < NC / 4; ++q) {  // columns from N on are not used
        xr[sp][q] = s_lu[wave][2 * h + sp][4 * q + g][min(c, NC - 1)][0];
        xi[sp][q] = s_lu[wave][2 * h + sp][4 * q + g][min(c, NC - 1)][1];
      }
#pragma unroll 1
    for (int t = 0; t < (M + 15) / 16; ++t) {
      double gs[4] = {0.0, 0.0, 0.0, 0.0};
      const int m = 16 * t + c;
      double2 v[2][NC / 4];
#pragma unroll
      for (int sp = 0; sp < 2; ++sp)
#pragma unroll
        for (int q = 0; q < NC / 4; ++q) {
          const int n = 4 * q + g;
          const double2 e = *reinterpret_cast<const double2*>(
              pw + ((size_t)(sp * M + min(m, M - 1)) * N + min(n, N - 1)) * 2);
          const bool ok = m < M && n < N;
          v[sp][q] = make_double2(keep_if(e.x, ok), keep_if(e.y, ok));
        }
#pragma unroll
      for (int sp = 0; sp < 2; ++sp) {
        dx4 tr = dx4_zero(), ti = dx4_zero();
#pragma unroll
        for (int q = 0; q < NC / 4; ++q) {
          tr = mfma_f64(v[sp][q].x, xr[sp][q], tr);
          tr = mfma_f64(-v[sp][q].y, xi[sp][q], tr);
          ti = mfma_f64(v[sp][q].x, xi[sp][q], ti);
          ti = mfma_f64(v[sp][q].y, xr[sp][q], ti);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int mo = 16 * t + g + 4 * r;
          if (mo < M && c < N) {
            if (th)
              *reinterpret_cast<double2*>(th + ((size_t)(sp * M + mo) * N + c) * 2) =
                  make_double2(tr[r], ti[r]);
            if (gd) gs[r] = fma(tr[r], pT[(size_t)mo * N + c], gs[r]);
          }
        }
      }
      if (gd)  // sum over the columns: the 16 lanes of a row
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double x = gs[r];
          x += dpp_f64<0xB1>(x);
          x += dpp_f64<0x4E>(x);
          x += dpp_f64<0x141>(x);
          x += dpp_f64<0x140>(x);
          const int mo = 16 * t + g + 4 * r;
          if (c == 0 && mo < M) gd[mo] = x;
        }
    }
  }
}

// One Metropolis sweep of Ising single-spin flips with diagonal generators: per flip the
// proposed y', its determinant (row m of Phi_0 scaled by exp(c sum_k y'_k A_k[m][m])), the
// log-overlap as in k_overlap, and the acceptance, in one launch for all K flips.  Two paths
// per wavefront; lane k holds y_k (K <= 64).  One flip is a chain of four kernels otherwise,
// each of a few us that its launch sets, and moves Phi_T through memory three times.  Whole
// steps, before and now: M = 8, N = 2, K = 4, 512 paths 153 -> 105 us; K = 8: M = 64, N = 16,
// 18000 paths 5.8 -> 4.0 ms, M = 16, N = 4, 18000 paths 1.54 -> 0.66 ms.
template <int NC>
__global__ void __launch_bounds__(OV_WAVES * 64, 2)
k_ising_sweep(int n_samples, int P, int M, int N, int K, double coupling,
              const double* __restrict__ Adiag, const double* __restrict__ phi0,
              const double* __restrict__ phi, double* __restrict__ y, double* __restrict__ phiT,
              double* __restrict__ logov, int* __restrict__ nacc, uint64_t seed, uint64_t step,
              const uint64_t* __restrict__ dstep, int sweep) {
  __shared__ double s_a[OV_WAVES][4][NC][NC + 1][2];  // [path, spin]: A
  __shared__ double s_e[OV_WAVES][2][64];             // row scales
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, c = lane & 15;
  const int s0 = (blockIdx.x * OV_WAVES + wave) * 2;
  if (s0 >= n_samples) return;  // no block-level barriers below
  if (dstep != nullptr) step = *dstep;
  const auto fence = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  };
  // a lone last path takes both places; the second does not write
  const int s1 = min(s0 + 1, n_samples - 1);
  double yk[2];
  yk[0] = lane < K ? y[(size_t)s0 * K + lane] : 0.0;
  yk[1] = lane < K ? y[(size_t)s1 * K + lane] : 0.0;
  // this half of the wavefront's path: its log-overlap, acceptances
  const int h = lane >> 5, sm = h ? s1 : s0;
  double lre = logov[(size_t)sm * 2], lim = logov[(size_t)sm * 2 + 1];
  int count = 0;
  const int mc = min(lane, M - 1);
  auto scales = [&](int flip) {  // lane m: exp(c sum_k y_k A_k[m][m]), y_flip negated
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      double u = 0.0;
      for (int k = 0; k < K; ++k) {
        const double x = readlane_f64(yk[q], k);
        u = fma(k == flip ? -x : x, Adiag[(size_t)k * M + mc], u);
      }
      s_e[wave][q][lane] = exp(coupling * u);
    }
    fence();
  };
#pragma unroll 1
  for (int f = 0; f < K; ++f) {
    scales(f);
#pragma unroll 1
    for (int q2 = 0; q2 < 2; ++q2) {
      const double* pw = phi + (size_t)((q2 ? s1 : s0) / P) * 2 * M * N * 2;
      dx4 acc[4] = {dx4_zero(), dx4_zero(), dx4_zero(), dx4_zero()};
#pragma unroll 4
      for (int q = 0; q < (M + 3) / 4; ++q) {
        const int m = 4 * q + g;
        const bool ok = m < M && c < N;
        const size_t e = (size_t)min(m, M - 1) * N + min(c, N - 1);
        const double a = keep_if(s_e[wave][q2][min(m, M - 1)] * phi0[e], ok);
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) {
          const double2 x = *reinterpret_cast<const double2*>(pw + ((size_t)sp * M * N + e) * 2);
          acc[2 * sp] = mfma_f64(a, keep_if(x.x, ok), acc[2 * sp]);
          acc[2 * sp + 1] = mfma_f64(a, keep_if(x.y, ok), acc[2 * sp + 1]);
        }
      }
#pragma unroll
      for (int sp = 0; sp < 2; ++sp)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (NC == 16 || (g + 4 * r < NC && c < NC)) {
            s_a[wave][2 * q2 + sp][g + 4 * r][c][0] = acc[2 * sp][r];
            s_a[wave][2 * q2 + sp][g + 4 * r][c][1] = acc[2 * sp + 1][r];
          }
    }
    fence();
    cplx a[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      a[j] = cmk(s_a[wave][g][min(c, NC - 1)][j][0], s_a[wave][g][min(c, NC - 1)][j][1]);
      if (NC < 16 && c >= NC) a[j] = cmk(0.0, 0.0);
    }
    fence();
    double nf = 0.0;
#pragma unroll
    for (int j = 0; j < NC; ++j) nf = fma(a[j].re, 0.0, fma(a[j].im, 0.0, nf));
    const bool nf_any = ((__ballot(nf != 0.0) >> (lane & 32)) & 0xffffffffull) != 0;
    int mystep;
    cplx scale;
    double logabs, argsum;
    bool singular;
    eliminate<NC, false>(a, N, lane, mystep, scale, logabs, argsum, singular);
    const int up = lane & 32, dn = up + 16;
    const bool sing = (__shfl((int)singular, up, 64) | __shfl((int)singular, dn, 64)) != 0;
    double nre = __shfl(logabs, up, 64) + __shfl(logabs, dn, 64);
    double nim = __shfl(argsum, up, 64) + __shfl(argsum, dn, 64);
    if (nf_any) {
      nre = nim = __builtin_nan("");
    } else if (sing) {
      nre = neg_inf();
      nim = 0.0;
    }
    double la = nre - lre;
    const double u = stream_uniform(seed, sm / P, step, rng_word3(AFQMC_TAG_ACCEPT, sweep, sm % P),
                                    (uint32_t)f);
    if (__builtin_isnan(la)) la = neg_inf();
    const bool acc = (la >= 0.0) || (u < exp(fmin(la, 0.0)));
    if (acc) {
      lre = nre;
      lim = nim;
      ++count;
    }
    const unsigned long long am = __ballot(acc);
    if (lane == f) {
      if (am & 1) yk[0] = -yk[0];
      if (am >> 32) yk[1] = -yk[1];
    }
  }
  // the accepted state: y, its determinant and log-overlap
  scales(-1);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int s = s0 + q;
    const int n = __builtin_amdgcn_readlane(count, 32 * q);
    if (s >= n_samples || n == 0) continue;
    if (lane < K) y[(size_t)s * K + lane] = yk[q];
    for (int e = lane; e < M * N; e += 64)
      phiT[(size_t)s * M * N + e] = s_e[wave][q][e / N] * phi0[e];
    if (lane == 32 * q) {
      logov[(size_t)s * 2] = lre;
      logov[(size_t)s * 2 + 1] = lim;
      if (nacc != nullptr) atomicAdd(nacc + s / P, n);
    }
  }
}

template <int NC>
hipError_t launch_nc(const afqmc_ctx_s* c, int nw, const double* phi, const double* phiT,
                     double* logov, double* theta, double* gdiag) {
  const int n = nw * c->P;
  auto kern = theta == nullptr && gdiag == nullptr ? k_overlap<NC, OV_DET>
              : overlap_by_lu(c, theta, gdiag)     ? k_overlap<NC, OV_LU>
                                                   : k_overlap<NC, OV_INV>;
  hipLaunchKernelGGL(kern, dim3((n + 2 * OV_WAVES - 1) / (2 * OV_WAVES)), dim3(OV_WAVES * 64), 0,
                     c->stream, n, c->P, c->M, c->N, phi, phiT, logov, theta, gdiag);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_overlap(const afqmc_ctx_s* c, int nw, const double* phi, const double* phiT,
                          double* logov, double* theta, double* gdiag) {
  if (nw <= 0) return hipSuccess;
  if (c->N > 16) return hipErrorInvalidValue;
  return c->N <= 8 ? launch_nc<8>(c, nw, phi, phiT, logov, theta, gdiag)
                   : launch_nc<16>(c, nw, phi, phiT, logov, theta, gdiag);
}

// Sweeps of single-spin flips with diagonal generators, for the small systems of this file.
bool ising_sweep_takes(const afqmc_ctx_s* c) {
  return c->small && !c->ctrial && c->hidden_kind == AFQMC_HIDDEN_ISING && c->d_Adiag != nullptr &&
         c->K <= 64;
}

hipError_t launch_ising_sweep(const afqmc_ctx_s* c, int nw, const double* phi, double* y,
                              double* phiT, double* logov, int* nacc, uint64_t seed, uint64_t step,
                              int sweep) {
  if (nw <= 0) return hipSuccess;
  const int n = nw * c->P;
  auto kern = c->N <= 8 ? k_ising_sweep<8> : k_ising_sweep<16>;
  hipLaunchKernelGGL(kern, dim3((n + 2 * OV_WAVES - 1) / (2 * OV_WAVES)), dim3(OV_WAVES * 64), 0,
                     c->stream, n, c->P, c->M, c->N, c->K, c->coupling, c->d_Adiag, c->d_phi0, phi,
                     y, phiT, logov, nacc, seed, step, c->dstep, sweep);
  return hipGetLastError();
}
