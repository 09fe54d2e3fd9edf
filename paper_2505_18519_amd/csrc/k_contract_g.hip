// Cholesky-vector contraction of complex (multi-slice) trials with FP32 matrix-core
// products (real trials with FP32 products run k_contract_f32, FP64 contexts
// k_contract and k_contract_q).  Same
// quantities as k_contract (Sec. III.A, Eq. local-obs; Eq. shift1):
//   Y_g = Phi_T^T L_g,  f_g^s = Y_g Theta^s,  vb_g = sum_s tr f_g^s,
//   E_p = sum_s tr(Phi_T^T h1' Theta^s) + 1/2 sum_g [vb_g^2 - sum_s tr(f_g^s f_g^s)].
//
// Layout: one workgroup per path with 2 * NTC wavefronts (NTC = ceil(N/16)),
// compiled per exact number of 16-row tiles KT = M/16 rounded up.  Wavefront
// w = (spin s = w % 2, column tile jt = w / 2) keeps Theta^s[:, jt] in
// registers for the whole loop over g.  Stage 1 (Y_g^T = L_g Phi_T) is split
// over all wavefronts by row tile so every element of L_g is read once per
// path (straight from L2; L is shared by all paths) through one software
// pipeline over all (row tile, k tile) steps whose loads run up to three steps
// ahead and continue into the next vector across the barrier; its result goes
// through LDS.  It runs on the real M x 2N matrix [Re Phi_T | Im Phi_T], giving
// Y_a = Re Phi_T^T L_g and Y_b = Im Phi_T^T L_g as column tiles that share every L
// operand.  Stage 2 forms Y_a Theta and Y_b Theta and combines
// f = Y_a Theta + i Y_b Theta for each wavefront's f^s[:, jt]; f is transposed
// through LDS for tr(f f).  Phi_T, Theta and L enter the products as FP32 with
// FP32 accumulation over m; per-vector traces, vb_g^2 and the sums over g are
// carried in FP64.
#include "afqmc_internal.h"
#include "dev_common.h"

namespace {

template <int KT, int NTC>
__global__ void __launch_bounds__(128 * NTC)
k_contract_g(int n_samples, int M, int N, int G, int MT, const float* __restrict__ Lpad,
             const double* __restrict__ phiT, const double* __restrict__ theta,
             const double* __restrict__ logov, double* __restrict__ vb, double* __restrict__ ep) {
  typedef float T;
  typedef ::MM<float> MM;
  typedef MM::acc_t acc_t;
  constexpr int KTMAX = KT;
  constexpr int NWV = 2 * NTC;             // wavefronts
  constexpr int NT = 16 * NTC;
  constexpr int NTC2 = 2 * NTC;            // stage-1 column tiles (re and im parts)
  constexpr int NT2 = 16 * NTC2;
  constexpr int S1MAX = (KT + NWV - 1) / NWV;  // stage-1 row tiles per wavefront
  constexpr int NS = S1MAX * KT;               // stage-1 (row tile, k tile) steps
  // L operand ring: loads run RING - 1 steps ahead; a depth that divides NS
  // leaves the next vector's first steps in slots 0 .. RING - 2 (no moves of
  // registers whose loads are still in flight)
  constexpr int RING = (NS % 4 == 0) ? 4 : (NS % 3 == 0) ? 3 : 2;
  extern __shared__ double smem[];
  T* sY = reinterpret_cast<T*>(smem);                        // [MT][NT2]
  double* sF = smem + (MT * NT2 * sizeof(T) + 7) / 8;         // [2][NT][NT+1][2]
  double* sD = sF + 2 * NT * (NT + 1) * 2;                    // [16][NWV*16][2]

  const int s = blockIdx.x;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = lane >> 4, c = lane & 15;
  const int sp = wave & 1, jt = wave >> 1;
  if (s >= n_samples) return;  // whole block exits together
  const bool active = !__builtin_isinf(logov[2 * s]);

  // Phi_T B operands for stage 1 (all column tiles), Theta^sp[:, jt] for stage 2.
  // Loads clamped in range and unconditional (masked afterwards), so that they are in
  // flight together rather than one branch and conversion at a time
  T bT[NTC2][KTMAX][4];
  T th[2][KTMAX][4];
#pragma unroll
  for (int t = 0; t < KTMAX; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = 16 * t + 4 * r + g;
      const bool okm = active && m < M;
      const int n = 16 * jt + c;
      const int mc = min(m, M - 1);
#pragma unroll
      for (int ct = 0; ct < NTC2; ++ct) {
        const int nb = 16 * (ct % NTC) + c, part = ct / NTC;
        const size_t e = ((size_t)s * M + mc) * N + min(nb, N - 1);
        bT[ct][t][r] = (T)keep_if(phiT[2 * e + part], okm && nb < N);
      }
      const double2 x2 = *reinterpret_cast<const double2*>(
          theta + ((((size_t)s * 2 + sp) * M + mc) * N + min(n, N - 1)) * 2);
      th[0][t][r] = (T)keep_if(x2.x, okm && n < N);
      th[1][t][r] = (T)keep_if(x2.y, okm && n < N);
    }

  // stage-1 step k = (q = k / KT, t = k % KT) reads L_g rows 16 t + 4 r + g of
  // column tile tp(q) = wave + NWV q (row tiles past KT are skipped)
  auto lrow = [&](const T* Lg, int k, int r) -> T {
    const int q = k / KT, t = k % KT;
    const int tp = min(wave + NWV * q, KT - 1);  // clamped: in bounds for every wave
    return Lg[(size_t)(16 * t + 4 * r + g) * MT + 16 * tp + c];
  };
  T av[RING][4];
  const size_t slab = (size_t)MT * MT;
#pragma unroll
  for (int k = 0; k < RING - 1; ++k)
    if (k < NS)
#pragma unroll
      for (int r = 0; r < 4; ++r) av[k][r] = lrow(Lpad, k, r);

  double ex_re = 0.0, ex_im = 0.0, vb2_re = 0.0, vb2_im = 0.0, e1_re = 0.0, e1_im = 0.0;
  for (int gam = 0; gam <= G; ++gam) {
    const T* Lg = Lpad + (size_t)gam * slab;
    const T* Ln = Lpad + (size_t)min(gam + 1, G) * slab;
    // stage 1: Y^T tiles (tp, ct), one software pipeline over all steps; the
    // first RING - 1 steps of the next vector are issued at the end
    acc_t y1[S1MAX][NTC2];
#pragma unroll
    for (int q = 0; q < S1MAX; ++q)
#pragma unroll
      for (int ct = 0; ct < NTC2; ++ct) y1[q][ct] = MM::zero();
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      const int q = k / KT, t = k % KT;
      const int kn = k + RING - 1;
      if (kn < NS) {
#pragma unroll
        for (int r = 0; r < 4; ++r) av[kn % RING][r] = lrow(Lg, kn, r);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) av[kn % RING][r] = lrow(Ln, kn - NS, r);
      }
      if (active && wave + NWV * q < KT)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int ct = 0; ct < NTC2; ++ct)
            y1[q][ct] = MM::fma(av[k % RING][r], bT[ct][t][r], y1[q][ct]);
    }
    // the ring now holds the next vector's first steps at slots NS % RING ...;
    // rotate them to slots 0 .. RING - 2 (only when RING does not divide NS)
    if (NS % RING != 0) {
      T tmp[RING][4];
#pragma unroll
      for (int k = 0; k < RING; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) tmp[k][r] = av[(k + NS) % RING][r];
#pragma unroll
      for (int k = 0; k < RING; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) av[k][r] = tmp[k][r];
    }
    // the previous vector's stage-2 and transpose reads are done
    __syncthreads();
#pragma unroll
    for (int q = 0; q < S1MAX; ++q) {
      const int tp = wave + NWV * q;
      if (tp < KT)
#pragma unroll
        for (int ct = 0; ct < NTC2; ++ct)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            sY[(16 * tp + MM::row(g, r)) * NT2 + 16 * ct + c] = y1[q][ct][r];
    }
    __syncthreads();
    // stage 2: f^sp[it][jt] = sum_m Y^T[m][it cols] Theta^sp[m][jt cols]
    acc_t f[NTC2][2];
#pragma unroll
    for (int it = 0; it < NTC2; ++it) f[it][0] = f[it][1] = MM::zero();
    if (active) {
#pragma unroll
      for (int t = 0; t < KTMAX; ++t) {
        if (t < KT) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int m = 16 * t + 4 * r + g;
#pragma unroll
            for (int it = 0; it < NTC2; ++it) {
              const T a = sY[m * NT2 + 16 * it + c];
              f[it][0] = MM::fma(a, th[0][t][r], f[it][0]);
              f[it][1] = MM::fma(a, th[1][t][r], f[it][1]);
            }
          }
        }
      }
    }
    // f = Y_a Theta + i Y_b Theta
#pragma unroll
    for (int it = 0; it < NTC; ++it) {
      const acc_t fr = f[it][0] - f[it + NTC][1];
      const acc_t fi = f[it][1] + f[it + NTC][0];
      f[it][0] = fr;
      f[it][1] = fi;
    }
    // diagonal of f^sp in tile (jt, jt): element (row(g,r), c) with row == c
    double d_re = 0.0, d_im = 0.0;
#pragma unroll
    for (int it = 0; it < NTC; ++it)
      if (it == jt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (MM::row(g, r) == c) {
            d_re = (double)f[it][0][r];
            d_im = (double)f[it][1][r];
          }
    if (gam == G) {
      d_re = wave_sum(d_re);
      d_im = wave_sum(d_im);
      // one-body term: both spins' traces, gathered through LDS below
      if (lane == 0) {
        sD[(wave * 16) * 2] = d_re;
        sD[(wave * 16) * 2 + 1] = d_im;
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        for (int w = 0; w < NWV; ++w) {
          e1_re += sD[(w * 16) * 2];
          e1_im += sD[(w * 16) * 2 + 1];
        }
      }
      break;
    }
    // stage f^sp[:, jt] in LDS for the transpose, and the diagonal partials
    double* Fs = sF + (size_t)sp * NT * (NT + 1) * 2;
#pragma unroll
    for (int it = 0; it < NTC; ++it)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * it + MM::row(g, r), j = 16 * jt + c;
        Fs[(i * (NT + 1) + j) * 2] = (double)f[it][0][r];
        Fs[(i * (NT + 1) + j) * 2 + 1] = (double)f[it][1][r];
      }
    {
      double* d = sD + ((size_t)(gam & 15) * NWV * 16 + wave * 16 + c) * 2;
      if (MM::row(g, 0) == c || MM::row(g, 1) == c || MM::row(g, 2) == c || MM::row(g, 3) == c) {
        d[0] = d_re;
        d[1] = d_im;
      }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < NTC; ++it)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * it + MM::row(g, r), j = 16 * jt + c;
        const double tr_ = Fs[(j * (NT + 1) + i) * 2], ti_ = Fs[(j * (NT + 1) + i) * 2 + 1];
        const double ar = (double)f[it][0][r], ai = (double)f[it][1][r];
        ex_re += ar * tr_ - ai * ti_;
        ex_im += ar * ti_ + ai * tr_;
      }
    // every 16 vectors: wavefront 0 reduces the staged diagonals to vb_g
    if (((gam & 15) == 15 || gam == G - 1) && wave == 0) {
      const int cnt = (gam & 15) + 1, g0 = gam & ~15;
      const int gl = lane & 15, part = (lane >> 4) & 1;
      double v = 0.0;
      if (lane < 32 && gl < cnt)
        for (int q = 0; q < NWV * 16; ++q) v += sD[((size_t)gl * NWV * 16 + q) * 2 + part];
      const double vi = __shfl_down(v, 16, 64);
      if (lane < 16 && gl < cnt) {
        vb2_re += v * v - vi * vi;
        vb2_im += 2.0 * v * vi;
        double* o = vb + ((size_t)s * G + g0 + gl) * 2;
        o[0] = v;
        o[1] = vi;
      }
    }
  }
  // totals: ex from every lane of every wavefront, vb^2 from wavefront 0
  ex_re = wave_sum(ex_re);
  ex_im = wave_sum(ex_im);
  vb2_re = wave_sum(vb2_re);
  vb2_im = wave_sum(vb2_im);
  __syncthreads();
  if (lane == 0) {
    sD[wave * 4 + 0] = ex_re;
    sD[wave * 4 + 1] = ex_im;
    sD[wave * 4 + 2] = vb2_re;
    sD[wave * 4 + 3] = vb2_im;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double xr = 0.0, xi = 0.0;
    for (int w = 0; w < NWV; ++w) {
      xr += sD[w * 4 + 0];
      xi += sD[w * 4 + 1];
    }
    const double br = sD[2], bi = sD[3];
    double* o = ep + (size_t)s * 2;
    o[0] = active ? e1_re + 0.5 * br - 0.5 * xr : 0.0;
    o[1] = active ? e1_im + 0.5 * bi - 0.5 * xi : 0.0;
  }
  if (!active)
    for (int q = threadIdx.x; q < 2 * G; q += blockDim.x) vb[(size_t)s * G * 2 + q] = 0.0;
}

template <int KT, int NTC>
hipError_t launch_g(const afqmc_ctx_s* c, int nw, const double* phiT, const double* theta,
                    const double* logov, double* vb, double* ep) {
  const int n = nw * c->P, NT = 16 * NTC, NWV = 2 * NTC;
  const size_t lds = ((size_t)c->MT * 2 * NT * sizeof(float) + 7) / 8 * 8 +
                     ((size_t)2 * NT * (NT + 1) * 2 + (size_t)16 * NWV * 16 * 2) * sizeof(double);
  auto kern = k_contract_g<KT, NTC>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(n), dim3(128 * NTC), lds, c->stream, n, c->M, c->N, c->G, c->MT,
                     c->d_Lpad32, phiT, theta, logov, vb, ep);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_contract_g(const afqmc_ctx_s* c, int nw, const double* phiT, const double* theta,
                             const double* logov, double* vb, double* ep) {
  if (nw <= 0) return hipSuccess;
  const int KT = c->MT / 16, NTC = (c->N + 15) / 16;
  // KT * NTC <= 8 (register budget of the doubled B operands)
#define AFQMC_GC(KK, NC) \
  if (KT == KK && NTC == NC) return launch_g<KK, NC>(c, nw, phiT, theta, logov, vb, ep);
  AFQMC_GC(1, 1) AFQMC_GC(2, 1) AFQMC_GC(3, 1) AFQMC_GC(4, 1)
  AFQMC_GC(5, 1) AFQMC_GC(6, 1) AFQMC_GC(7, 1) AFQMC_GC(8, 1)
  AFQMC_GC(2, 2) AFQMC_GC(3, 2) AFQMC_GC(4, 2)
#undef AFQMC_GC
  return hipErrorInvalidValue;
}
