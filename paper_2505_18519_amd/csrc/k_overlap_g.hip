// Overlap, log-determinant and Green's function for larger systems (N <= 40,
// M <= 160); same quantities and conventions as k_overlap (Sec. III.A, Eqs.
// ratio-update-phi and sign-path).  One workgroup of two wavefronts per path,
// wavefront s handling spin s:
//  1. A^s = Phi_T^T phi^s on the FP64 matrix cores (NTC x NTC tiles of 16),
//     operand loads clamped and bit-masked so that four k steps are in flight;
//  2. elimination with partial pivoting, one lane per row (N <= 40 lanes): the
//     pivot (largest |a|^2, lowest row on ties) by DPP moves and a ballot, the
//     pivot row broadcast by readlane (the pivot is uniform over the wavefront);
//     det = parity prod of pivots, accumulated as a scaled complex product;
//  3. with Theta or the Green's function diagonal requested the elimination is
//     Gauss-Jordan in place, which leaves X^s = (A^s)^{-1} in the rows: X^s goes to
//     LDS, Theta^s = phi^s X^s runs on the matrix cores (four real products per
//     tile), is stored as whole 16-byte complex entries along each row, and the
//     diagonal Re (G_up + G_dn)_mm = Re sum_s sum_n Theta^s_mn Phi_T,mn is summed
//     from its tiles.
// The two spins' log-determinants and diagonals are added through LDS.  A
// zero pivot gives l = -inf + 0i, a non-finite overlap entry l = NaN + NaN i
// (Theta and the diagonal 0 in both cases).
// CT: complex trial determinants (multi-slice trials), A^s = Phi_T^T phi^s
// with both factors complex (no conjugation: the bilinear overlap of Eq.
// ratio-update-phi); the Green's-function diagonal is then not formed.
//
// The elimination is a loop: after step k every row moves up one column, so that the
// pivot column is always register 0 and the code of a step is the same.  Unrolled over
// columns and steps it was 240 KB of code at N = 32 and 500 KB at N = 40, past the
// instruction cache (64 KB for two CUs), and every wavefront's pass over it set the time;
// now 4 to 19 KB.  What bounds it now: the matrix-core products (padded to 16 columns), the
// vector unit (a broadcast and four FP64 operations per row, column and step), each step's
// serial chain, and with Theta its writes.  Measured, before and now: M = 72, N = 18, 2800
// paths, log-overlaps only 187 -> 89 us; with Theta M = 96, N = 24, 8192 paths 959 -> 556 us,
// M = 128, N = 32, 4096 paths 711 -> 534 us; with the diagonal M = 96, N = 24, 2048 paths
// 285 -> 170 us.
#include "afqmc_internal.h"
#include "dev_common.h"

namespace {

// NC: columns of a row in registers, N rounded up to 8; INV: Theta or the diagonal
// requested (of one kernel's two eliminations each would keep its own copy of the rows)
template <int NC, bool CT, bool INV>
__global__ void __launch_bounds__(128, NC <= 16 ? 4 : NC <= 24 ? 3 : 2)
k_overlap_g(int n_samples, int P, int M, int N, const double* __restrict__ phi,
            const double* __restrict__ phiT, double* __restrict__ logov, double* __restrict__ theta,
            double* __restrict__ gdiag) {
  constexpr int NTC = (NC + 15) / 16, NT = 16 * NTC;
  __shared__ double s_lu[2][NC][NC + 1][2];
  __shared__ int s_perm[2][NC];
  __shared__ double s_res[2][3];
  __shared__ double s_gd[2][160];  // M <= 160

  // workgroup b takes walker 8 (b / 8P) + b % 8 and its path (b / 8) % P: the
  // P paths of a walker, which read the same phi, run 8 launches apart on one
  // XCD (workgroups go round-robin over the 8) and share that XCD's L2
  const int s = (8 * ((int)blockIdx.x / (8 * P)) + ((int)blockIdx.x & 7)) * P +
                ((int)blockIdx.x >> 3) % P;
  const int sp = threadIdx.x >> 6;  // spin of this wavefront
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, c = lane & 15;
  if (s >= n_samples) return;  // whole block
  const int w = s / P;
  const double* pT = phiT + (size_t)s * M * N * (CT ? 2 : 1);
  const double* pw = phi + ((size_t)w * 2 + sp) * M * N * 2;

  // 1. A^sp tiles (it, jt): A[i][j] = sum_m Phi_T[m][i] phi[m][j]
  dx4 acc[NTC][NTC][2];
#pragma unroll
  for (int it = 0; it < NTC; ++it)
#pragma unroll
    for (int jt = 0; jt < NTC; ++jt) acc[it][jt][0] = acc[it][jt][1] = dx4_zero();
#pragma unroll 4
  for (int q = 0; q < (M + 3) / 4; ++q) {
    const int m = 4 * q + g;
    const bool okm = m < M;
    const int mc = min(m, M - 1);
    double a[NTC], ai[NTC], br[NTC], bi[NTC];
#pragma unroll
    for (int t = 0; t < NTC; ++t) {
      const int n = 16 * t + c;
      const bool ok = okm && n < N;
      const size_t e = (size_t)mc * N + min(n, N - 1);
      if (CT) {
        const double2 v = *reinterpret_cast<const double2*>(pT + e * 2);
        a[t] = keep_if(v.x, ok);
        ai[t] = keep_if(v.y, ok);
      } else {
        a[t] = keep_if(pT[e], ok);
        ai[t] = 0.0;
      }
      const double2 x = *reinterpret_cast<const double2*>(pw + e * 2);
      br[t] = keep_if(x.x, ok);
      bi[t] = keep_if(x.y, ok);
    }
#pragma unroll
    for (int it = 0; it < NTC; ++it)
#pragma unroll
      for (int jt = 0; jt < NTC; ++jt) {
        acc[it][jt][0] = mfma_f64(a[it], br[jt], acc[it][jt][0]);
        acc[it][jt][1] = mfma_f64(a[it], bi[jt], acc[it][jt][1]);
        if (CT) {
          acc[it][jt][0] = mfma_f64(-ai[it], bi[jt], acc[it][jt][0]);
          acc[it][jt][1] = mfma_f64(ai[it], br[jt], acc[it][jt][1]);
        }
      }
  }
#pragma unroll
  for (int it = 0; it < NTC; ++it)
#pragma unroll
    for (int jt = 0; jt < NTC; ++jt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * it + g + 4 * r, col = 16 * jt + c;
        if (NC == NT || (row < NC && col < NC)) {
          s_lu[sp][row][col][0] = acc[it][jt][0][r];
          s_lu[sp][row][col][1] = acc[it][jt][1][r];
        }
      }
  __syncthreads();

  // 2. elimination, lane i = row i (i < N)
  const int i = lane;
  cplx a[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j)
    a[j] = (i < NC) ? cmk(s_lu[sp][i][j][0], s_lu[sp][i][j][1]) : cmk(0.0, 0.0);
  __syncthreads();
  // a non-finite entry of either spin's overlap matrix makes l NaN (a
  // numerical event, not a singular path)
  double nf = 0.0;
#pragma unroll
  for (int j = 0; j < NC; ++j) nf = fma(a[j].re, 0.0, fma(a[j].im, 0.0, nf));
  const bool nonfinite = __ballot(nf != 0.0) != 0;  // NaN
  bool used = i >= N;
  int mystep = -1;
  cplx scale = cmk(0.0, 0.0);  // 1 / pivot of this lane's row
  cplx pprod = cmk(1.0, 0.0);
  int pexp = 0, inv = 0;
  unsigned long long done = 0;  // pivot rows so far
  bool singular = false;
  // step k on the first W registers.  INV: Gauss-Jordan in place; column k of the
  // inverse takes the place of the pivot column, and pivot rows stay unscaled (row
  // `scale` times the registers) as every update is linear in the row it changes.
  auto step = [&](auto WW, int k) {
    constexpr int W = decltype(WW)::value;
    // NaN entries count as zero so that the order is total and every lane
    // agrees on the pivot
    double v = used ? -1.0 : cabs2(a[0]);
    if (!used && !(v >= 0.0)) v = 0.0;
    double mv = fmax(v, dpp_f64<0xB1>(v));
    mv = fmax(mv, dpp_f64<0x4E>(mv));
    mv = fmax(mv, dpp_f64<0x141>(mv));
    mv = fmax(mv, dpp_f64<0x140>(mv));
    // lanes past NC are all used
    double vm = readlane_f64(mv, 0);
    if (NTC > 1) vm = fmax(vm, readlane_f64(mv, 16));
    if (NTC > 2) vm = fmax(vm, readlane_f64(mv, 32));
    const int prow = __builtin_ctzll(__ballot(!used && v == vm));
    inv += __builtin_popcountll(done >> prow);
    done |= 1ull << prow;
    const cplx piv = cmk(readlane_f64(a[0].re, prow), readlane_f64(a[0].im, prow));
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
      const cplx pj = cmk(readlane_f64(a[j + 1].re, prow), readlane_f64(a[j + 1].im, prow));
      a[j] = cfms(a[j + 1], l, pj);
      asm volatile("" : "+v"(a[j].re), "+v"(a[j].im));  // in order: no second set of registers
    }
    if (INV) a[W - 1] = mine ? cmk(1.0, 0.0) : cmk(-l.re, -l.im);
  };
  if constexpr (INV) {
#pragma unroll 1
    for (int k = 0; k < N; ++k) step(std::integral_constant<int, NC>{}, k);
  } else {
    int k = 0;
    unrolled<NC / 8>([&](auto I) {  // N - k columns are left: W, W - 8, ..
      constexpr int W = NC - 8 * decltype(I)::value;
#pragma unroll 1
      for (; k < N - W + 8; ++k) step(std::integral_constant<int, W>{}, k);
    });
  }
  if (lane == 0) {
    s_res[sp][0] = 0.5 * log(cabs2(pprod)) + (double)pexp * M_LN2;
    s_res[sp][1] = atan2(pprod.im, pprod.re) + ((inv & 1) ? M_PI : 0.0);
    s_res[sp][2] = nonfinite ? 2.0 : singular ? 1.0 : 0.0;
  }
  if constexpr (INV) {
    if (mystep >= 0) s_perm[sp][mystep] = i;
    if (lane < NC)
#pragma unroll
      for (int j = 0; j < NC; ++j) s_lu[sp][lane][j][0] = s_lu[sp][lane][j][1] = 0.0;
  }
  __syncthreads();
  const bool sing_any = s_res[0][2] != 0.0 || s_res[1][2] != 0.0;
  const bool nf_any = s_res[0][2] == 2.0 || s_res[1][2] == 2.0;
  if (threadIdx.x == 0) {
    double* o = logov + (size_t)s * 2;
    const double nan = __builtin_nan("");
    o[0] = nf_any ? nan : sing_any ? neg_inf() : s_res[0][0] + s_res[1][0];
    o[1] = nf_any ? nan : sing_any ? 0.0 : s_res[0][1] + s_res[1][1];
  }
  if constexpr (!INV) return;
  double* th = theta ? theta + ((size_t)s * 2 + sp) * M * N * 2 : nullptr;
  double* gd = gdiag ? gdiag + (size_t)s * M : nullptr;
  if (sing_any) {
    if (th)
      for (int q = lane; q < M * N * 2; q += 64) th[q] = 0.0;
    if (gd && sp == 0)
      for (int q = lane; q < M; q += 64) gd[q] = 0.0;
    return;
  }
  // 3. X = (A^sp)^{-1}: the row of step k is X's row k, and register NC - N + m its column
  //    perm[m]; the rest stays zero
  if (mystep >= 0) {
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int m = j - (NC - N);
      if (m >= 0) {
        const cplx x = cmul(a[j], scale);
        const int col = s_perm[sp][m];
        s_lu[sp][mystep][col][0] = x.re;
        s_lu[sp][mystep][col][1] = x.im;
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  // 4. Theta^sp = phi^sp X on the matrix cores: A[c][g] = phi[16t + c][4q + g],
  //    B[g][c] = X[4q + g][16ct + c]; the lane holds Theta[16t + g + 4r][16ct + c]
  double xr[NC / 4][NTC], xi[NC / 4][NTC];
#pragma unroll
  for (int q = 0; q < NC / 4; ++q)
#pragma unroll
    for (int ct = 0; ct < NTC; ++ct) {
      const int col = min(16 * ct + c, NC - 1);  // columns from N on are not used
      xr[q][ct] = s_lu[sp][4 * q + g][col][0];
      xi[q][ct] = s_lu[sp][4 * q + g][col][1];
    }
  for (int t = 0; t < (M + 15) / 16; ++t) {
    const int m = 16 * t + c;
    const int mc = min(m, M - 1);
    double2 v[NC / 4];
#pragma unroll
    for (int q = 0; q < NC / 4; ++q) {
      const int n = 4 * q + g;
      const double2 e =
          *reinterpret_cast<const double2*>(pw + ((size_t)mc * N + min(n, N - 1)) * 2);
      const bool ok = m < M && n < N;
      v[q] = make_double2(keep_if(e.x, ok), keep_if(e.y, ok));
    }
    dx4 tr[NTC], ti[NTC];
#pragma unroll
    for (int ct = 0; ct < NTC; ++ct) tr[ct] = ti[ct] = dx4_zero();
#pragma unroll
    for (int q = 0; q < NC / 4; ++q)
#pragma unroll
      for (int ct = 0; ct < NTC; ++ct) {
        tr[ct] = mfma_f64(v[q].x, xr[q][ct], tr[ct]);
        tr[ct] = mfma_f64(-v[q].y, xi[q][ct], tr[ct]);
        ti[ct] = mfma_f64(v[q].x, xi[q][ct], ti[ct]);
        ti[ct] = mfma_f64(v[q].y, xr[q][ct], ti[ct]);
      }
    double gs[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ct = 0; ct < NTC; ++ct)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int mo = 16 * t + g + 4 * r, col = 16 * ct + c;
        if (mo < M && col < N) {
          if (th)
            *reinterpret_cast<double2*>(th + ((size_t)mo * N + col) * 2) =
                make_double2(tr[ct][r], ti[ct][r]);
          if (!CT && gd) gs[r] = fma(tr[ct][r], pT[(size_t)mo * N + col], gs[r]);
        }
      }
    if (!CT && gd) {  // sum over the columns: the 16 lanes of a row
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double x = gs[r];
        x += dpp_f64<0xB1>(x);
        x += dpp_f64<0x4E>(x);
        x += dpp_f64<0x141>(x);
        x += dpp_f64<0x140>(x);
        const int mo = 16 * t + g + 4 * r;
        if (c == 0 && mo < M) s_gd[sp][mo] = x;
      }
    }
  }
  if (!CT && gd) {  // block-uniform
    __syncthreads();
    for (int m = threadIdx.x; m < M; m += 128) gd[m] = s_gd[0][m] + s_gd[1][m];
  }
}

template <int NC>
hipError_t launch_g(const afqmc_ctx_s* c, int nw, const double* phi, const double* phiT,
                    double* logov, double* theta, double* gdiag) {
  const int n = nw * c->P;
  const dim3 grid(8 * c->P * ((nw + 7) / 8));  // walkers padded to 8 (see the kernel)
  if (c->ctrial && gdiag != nullptr) return hipErrorInvalidValue;
  const bool inv = theta != nullptr || gdiag != nullptr;
  auto kern = c->ctrial ? (inv ? k_overlap_g<NC, true, true> : k_overlap_g<NC, true, false>)
                        : (inv ? k_overlap_g<NC, false, true> : k_overlap_g<NC, false, false>);
  hipLaunchKernelGGL(kern, grid, dim3(128), 0, c->stream, n, c->P, c->M, c->N, phi, phiT, logov,
                     theta, gdiag);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_overlap_g(const afqmc_ctx_s* c, int nw, const double* phi, const double* phiT,
                            double* logov, double* theta, double* gdiag) {
  if (nw <= 0) return hipSuccess;
  switch ((c->N + 7) / 8) {
    case 1: return launch_g<8>(c, nw, phi, phiT, logov, theta, gdiag);
    case 2: return launch_g<16>(c, nw, phi, phiT, logov, theta, gdiag);
    case 3: return launch_g<24>(c, nw, phi, phiT, logov, theta, gdiag);
    case 4: return launch_g<32>(c, nw, phi, phiT, logov, theta, gdiag);
    case 5: return launch_g<40>(c, nw, phi, phiT, logov, theta, gdiag);
    default: return hipErrorInvalidValue;
  }
}
