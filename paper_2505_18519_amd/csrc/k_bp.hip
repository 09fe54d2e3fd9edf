// Back-propagated one-body density matrix (App. B, Measurement; Eqs.
// AFQMC_Metropolis_measure and AFQMC_Metropolis_measure2).  The projectors of
// the restored steps reuse the propagator's kernels (k_vbuild, and k_taylor_g or
// k_taylor_q with one block per path, the walker's V shared by its paths); the overlap
// with the saved walker reuses the complex-trial overlap kernel.  Here: the
// field history, and the path-weighted density per walker and its weighted
// sum over walkers.
#include <algorithm>

#include "afqmc_internal.h"
#include "dev_common.h"

namespace {

// hist_xi[w][slot][g] = xi[w][g], hist_xbar[w][slot][g] = xbar[w][g] (complex)
__global__ void k_bp_record(int nw, int h, int slot, int G, const double* __restrict__ xi,
                            const double* __restrict__ xbar, double* __restrict__ hxi,
                            double* __restrict__ hxb) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)nw * G) return;
  const size_t w = idx / G, g = idx % G;
  const size_t d = (w * h + slot) * G + g;
  hxi[d] = xi[idx];
  hxb[2 * d] = xbar[2 * idx];
  hxb[2 * d + 1] = xbar[2 * idx + 1];
}

__global__ void k_real_to_complex(size_t n, const double* __restrict__ src, double* __restrict__ dst) {
  for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < n;
       q += (size_t)gridDim.x * blockDim.x) {
    dst[2 * q] = src[q];
    dst[2 * q + 1] = 0.0;
  }
}

// One workgroup per walker.  Path weights a_p = exp(lt_p - Re l_p - max_p) (lt =
// log <Phi~_p|phi_mid>, l = log O_p at the measurement step; singular paths 0);
// R_k[i][j] = sum_p a_p sum_s sum_n Theta_p^s[i][n] Phi~_p[j][n] / sum_p a_p.  ok[k] = 1
// when the walker has a live path and a finite R_k.
// The sum over (p, n) is a complex M x M product of inner length P N on the FP64
// matrix cores: lane (g, c) supplies a_p (Theta^up + Theta^dn)[16 it + c][4 t + g] and
// Phi~[16 jt + c][4 t + g], and a wavefront takes NJ column tiles of one row tile.
// Bound by the reads of Theta and Phi~ (a path's are read once per tile row or column,
// mostly from L2).  M = 64, N = 16, 8 paths, 128 walkers: 655 us with one thread per entry,
// 48 now.
template <int NJ>
__global__ void __launch_bounds__(1024)
k_bp_density(int nw, int P, int M, int N, const double* __restrict__ theta,
             const double* __restrict__ phit, const double* __restrict__ lt,
             const double* __restrict__ lend, double* __restrict__ rho, int* __restrict__ ok) {
  __shared__ double s_x[64];
  __shared__ double s_a[64][2];
  __shared__ double s_den[2];
  __shared__ int s_bad;
  const int k = blockIdx.x, tid = threadIdx.x;
  // path weights, one lane each (P <= 64)
  double x = -__builtin_huge_val(), arg = 0.0;
  if (tid < P) {
    const double* a = lt + ((size_t)k * P + tid) * 2;
    const double* b = lend + ((size_t)k * P + tid) * 2;
    arg = a[1];
    if (__builtin_isfinite(a[0]) && __builtin_isfinite(b[0])) x = a[0] - b[0];
    s_x[tid] = x;
  }
  if (tid == 0) s_bad = 0;
  __syncthreads();
  if (tid < P) {
    double mx = -__builtin_huge_val();
    for (int p = 0; p < P; ++p) mx = fmax(mx, s_x[p]);
    double ar = 0.0, ai = 0.0;
    if (!__builtin_isinf(x)) {
      const double mag = exp(x - mx);
      double sn, cs;
      sincos(arg, &sn, &cs);
      ar = mag * cs;
      ai = mag * sn;
    }
    s_a[tid][0] = ar;
    s_a[tid][1] = ai;
  }
  __syncthreads();
  if (tid == 0) {
    double dr = 0.0, di = 0.0;
    for (int p = 0; p < P; ++p) {
      dr += s_a[p][0];
      di += s_a[p][1];
    }
    s_den[0] = dr;
    s_den[1] = di;
  }
  __syncthreads();
  const double dr = s_den[0], di = s_den[1];
  const double dd = dr * dr + di * di;
  const int wave = tid >> 6, lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int KT = (M + 15) / 16, JC = (KT + NJ - 1) / NJ, NQ = (N + 3) / 4;
  for (int task = wave; task < KT * JC; task += blockDim.x >> 6) {
    const int it = task / JC, jc = task % JC;
    const size_t MN = (size_t)M * N;
    const double* T = theta + ((size_t)k * P * 2 * MN + (size_t)min(16 * it + c, M - 1) * N) * 2;
    const double* X[NJ];
#pragma unroll
    for (int b = 0; b < NJ; ++b)
      X[b] = phit + ((size_t)k * P * MN + (size_t)min(16 * (jc * NJ + b) + c, M - 1) * N) * 2;
    dx4 re[NJ], im[NJ];
#pragma unroll
    for (int b = 0; b < NJ; ++b) re[b] = im[b] = dx4{0.0, 0.0, 0.0, 0.0};
    for (int p = 0; p < P; ++p) {
      const double wr = s_a[p][0], wi = s_a[p][1];
      if (wr == 0.0 && wi == 0.0) continue;  // the same on every lane
      const double* Tp = T + (size_t)p * 4 * MN;
#pragma unroll 4
      for (int t = 0; t < NQ; ++t) {
        const bool in = 4 * t + g < N;
        const int n = min(4 * t + g, N - 1);
        const double2 u = *reinterpret_cast<const double2*>(Tp + 2 * n);
        const double2 d = *reinterpret_cast<const double2*>(Tp + 2 * MN + 2 * n);
        double2 v[NJ];
#pragma unroll
        for (int b = 0; b < NJ; ++b)
          v[b] = *reinterpret_cast<const double2*>(X[b] + (size_t)p * 2 * MN + 2 * n);
        const double tr = u.x + d.x, ti = u.y + d.y;
        const double ar = keep_if(wr * tr - wi * ti, in), ai = keep_if(wr * ti + wi * tr, in);
#pragma unroll
        for (int b = 0; b < NJ; ++b) {
          const double xr = keep_if(v[b].x, in), xi = keep_if(v[b].y, in);
          re[b] = mfma_f64(ar, xr, re[b]);
          im[b] = mfma_f64(ar, xi, im[b]);
          re[b] = mfma_f64(-ai, xi, re[b]);
          im[b] = mfma_f64(ai, xr, im[b]);
        }
      }
    }
    bool bad = false;
#pragma unroll
    for (int b = 0; b < NJ; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * it + g + 4 * r, j = 16 * (jc * NJ + b) + c;
        if (i >= M || j >= M) continue;
        const double ar = re[b][r], ai = im[b][r];
        double2 o = make_double2(0.0, 0.0);
        if (dd > 0.0) o = make_double2((ar * dr + ai * di) / dd, (ai * dr - ar * di) / dd);
        *reinterpret_cast<double2*>(rho + ((size_t)k * M * M + (size_t)i * M + j) * 2) = o;
        bad = bad || !__builtin_isfinite(o.x);
      }
    if (bad) s_bad = 1;  // benign race: any writer sets 1
  }
  __syncthreads();
  if (tid == 0) ok[k] = (dd > 0.0 && s_bad == 0) ? 1 : 0;
}

// error-free transformation a + b = s + e
__device__ __forceinline__ void two_sum_bp(double a, double b, double& s, double& e) {
  s = a + b;
  const double bb = s - a;
  e = (a - (s - bb)) + (b - bb);
}

// out[e] = sum_k ok_k W_k Re R_k[e] for e < M^2, out[M^2] = sum_k ok_k W_k;
// thread e runs over the walkers in order (compensated), RB walkers' entries read at a
// time (M = 64, 128 walkers: 47 us one at a time, 18 now)
constexpr int RB = 16;
__global__ void __launch_bounds__(64)
k_bp_reduce(int nw, int MM, const double* __restrict__ w, const double* __restrict__ rho,
            const int* __restrict__ ok, double* __restrict__ out) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e > MM) return;
  const double* r = rho + (size_t)min(e, MM - 1) * 2;
  double s = 0.0, c = 0.0;
  for (int k0 = 0; k0 < nw; k0 += RB) {
    double x[RB], wk[RB];
    int live[RB];
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      const int k = min(k0 + q, nw - 1);
      x[q] = r[(size_t)k * MM * 2];
      wk[q] = w[k];
      live[q] = k0 + q < nw ? ok[k] : 0;
    }
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      const double v = (e == MM) ? wk[q] : wk[q] * x[q];
      double t, err;
      two_sum_bp(s, v, t, err);
      s = live[q] ? t : s;
      c = live[q] ? c + err : c;
    }
  }
  out[e] = s + c;
}

}  // namespace

hipError_t launch_bp_record(const afqmc_ctx_s* c, int nw, int h, int slot, const double* xi,
                            const double* xbar, double* hxi, double* hxb) {
  const size_t total = (size_t)nw * c->G;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(k_bp_record, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, c->stream,
                     nw, h, slot, c->G, xi, xbar, hxi, hxb);
  return hipGetLastError();
}

hipError_t launch_real_to_complex(const afqmc_ctx_s* c, size_t n, const double* src, double* dst) {
  if (n == 0) return hipSuccess;
  const unsigned blocks = (unsigned)std::min<size_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_real_to_complex, dim3(blocks), dim3(256), 0, c->stream, n, src, dst);
  return hipGetLastError();
}

hipError_t launch_bp_density(const afqmc_ctx_s* c, int nw, const double* theta, const double* phit,
                             const double* lt, const double* lend, double* rho, int* ok) {
  if (nw <= 0) return hipSuccess;
  const int KT = (c->M + 15) / 16;
  // a tile per wavefront up to the sixteen of a workgroup, then two
  auto kern = KT <= 4 ? k_bp_density<1> : k_bp_density<2>;
  hipLaunchKernelGGL(kern, dim3(nw), dim3(KT <= 4 ? 64 * KT * KT : 1024), 0, c->stream, nw, c->P,
                     c->M, c->N, theta, phit, lt, lend, rho, ok);
  return hipGetLastError();
}

hipError_t launch_bp_reduce(const afqmc_ctx_s* c, int nw, const double* w, const double* rho,
                            const int* ok, double* out) {
  const int MM = c->M * c->M;
  hipLaunchKernelGGL(k_bp_reduce, dim3((MM + 1 + 63) / 64), dim3(64), 0, c->stream, nw, MM, w,
                     rho, ok, out);
  return hipGetLastError();
}
