// Cholesky-vector contraction with FP32 matrix-core products and FP32
// accumulation (AFQMC_PREC_FP32, real trials).  Same quantities as k_contract
// (Sec. III.A, Eq. local-obs; Eq. shift1):
//   Y_g = Phi_T^T L_g,  f_g^s = Y_g Theta^s,  vb_g = sum_s tr f_g^s,
//   E_p = sum_s tr(Phi_T^T h1' Theta^s) + 1/2 sum_g [vb_g^2 - sum_s tr(f_g^s f_g^s)].
// Products: four v_mfma_f32_16x16x4f32 per 16-wide k block, the j-th on k = 16 t +
// 4 g + j (lane group g).  tr(f f): each lane sums, per vector, its products with
// rows 4 g .. 4 g + 3 and 16 + 4 g .. 16 + 4 g + 3 of one column in FP32; the sums
// over lanes and vectors and the diagonals' sums are FP64.
//
// What bounds it is the matrix cores.  One path and one vector at a time take
// ceil(N / 16) column tiles of Y_g = L_g Phi_T and as many row tiles of
// f = Y^T Theta.  Here the columns of two paths stand side by side in stage 1 and
// those of two vectors in stage 2, 8 T each, T = ceil(N / 8): T tiles for two,
// where an odd T would leave half of the last one empty each time.
//
// 2 T wavefronts share a pair of paths.  Stage 1: wavefront (vector v, tile ct)
// multiplies all row tiles of L_{2 grp + v}, read from global memory (L2) in operand
// order one row tile ahead, by its tile of the pair's packed Phi_T, held in
// registers, and leaves Y^T in LDS in stage 2's operand layout.  Stage 2:
// wavefront (path, tile) holds its tile of the two spins' packed Theta in
// registers and multiplies both vectors' rows.  Rows of f are packed in groups of
// four, 2 T a vector, so that a lane's rows of a vector are the ones it sums.  f
// goes through LDS for the transpose; Y and f have their own space, so that two
// vectors need two barriers.  Matrix cores and traces overlap: with N <= 24 a
// workgroup has two pairs, the second one barrier behind the first, so that one's
// stage 2 covers the other's trace and stage 1; for larger N (one pair, registers
// for two wavefronts a SIMD) the second path takes its trace after the next
// group's stage 1 instead of before.
//
// Measured, before (one path and vector at a time, L through LDS, three
// wavefronts a path) and now: M = 96, N = 24, 384 vectors, 8192 paths 30.8 -> 21.9 ms
// (90 -> 127 TFLOP/s of unpadded products; a large FP32 matrix product reaches 153);
// M = 64, 256 vectors, 4096 paths: N = 8 2.68 -> 0.99 ms, N = 16 2.56 -> 2.22, N = 24
// 6.03 -> 4.35; M = 128, N = 16, 2048 paths 4.68 -> 3.49; N = 32, 512 vectors, 4096
// paths 33.3 -> 33.3.  With few paths the vectors are split over workgroups: M = 70,
// N = 22, 240 vectors, 40 paths 1.79 -> 0.14 ms.
#include "afqmc_internal.h"
#include "contract_sum.h"
#include "dev_common.h"

namespace {

// Blocks of the sum over the vectors: at least four groups each (the sum at a block's end
// takes 0.3 us, a group of M = 24, N = 6 1.1), in a number that the likely ranges share evenly
__host__ __device__ constexpr int sum_blocks(int ngrp) {
  constexpr int n[] = {48, 24, 12, 8, 6, 4, 3, 2};
  for (int q : n)
    if (4 * q <= ngrp) return q;
  return 1;
}

template <int KT, int T>
struct Shape {
  static constexpr int NPR = T < 4 ? 2 : 1;        // pairs of paths
  static constexpr int S = 8 * T;                  // columns per path, spin or vector
  static constexpr int PW = 16 * T + 4;            // row length of the staged f (bank spread)
  static constexpr int NW = 2 * NPR * T;                 // wavefronts
  static constexpr int YP = 2 * 4 * KT * 16 * T;   // 4-row groups of one pair's Y^T (two vectors)
  static constexpr int FV = 2 * S * PW;            // floats of one vector's f (re, im)
  static constexpr size_t lds() {
    return (size_t)NPR * YP * 16 + (size_t)2 * NPR * 2 * FV * 4 + (size_t)NW * 16;
  }
};

template <int KT, int T>
__global__ void __launch_bounds__(T < 4 ? 256 * T : 128 * T)
k_contract_f32(int n_samples, int M, int N, int G, const fx4* Lop,
               const double* __restrict__ phiT, const double* __restrict__ theta,
               const double* __restrict__ logov, double* __restrict__ vb,
               double* __restrict__ epart) {
  typedef Shape<KT, T> Sh;
  constexpr int S = Sh::S, PW = Sh::PW, SLAB = KT * KT * 64;
  extern __shared__ double smem[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = lane >> 4, c = lane & 15;
  const int pair = wave / (2 * T), wq = wave % (2 * T);
  // stage 1: tile w1 of the pair's columns, vector v1; stage 2: path pp, tile w1 of the spins
  const int v1 = wq / T, w1 = wq % T, pp = v1;
  fx4* sY = reinterpret_cast<fx4*>(smem) + pair * Sh::YP;
  float* sF = reinterpret_cast<float*>(reinterpret_cast<fx4*>(smem) + Sh::NPR * Sh::YP) +
              (pair * 2 + pp) * 2 * Sh::FV;
  double* sT = smem + (Sh::NPR * Sh::YP * 16 + 2 * Sh::NPR * 2 * Sh::FV * 4) / 8;  // [wave][re, im]

  const int q = 16 * w1 + c, qh = q / S, qn = q % S;  // packed column: path or spin, electron
  const int s = (blockIdx.x * Sh::NPR + pair) * 2 + pp;       // this wavefront's path in stage 2
  const bool valid = s < n_samples;
  const int sc = valid ? s : n_samples - 1;
  const bool active = valid && !__builtin_isinf(logov[2 * sc]);

  fx4 bT[KT], th[2][KT];
  {
    const int sb = (blockIdx.x * Sh::NPR + pair) * 2 + qh, sbc = min(sb, n_samples - 1);
    const bool okb = sb < n_samples && !__builtin_isinf(logov[2 * sbc]) && qn < N;
    const bool okt = active && qn < N;
    const int nc = min(qn, N - 1);
#pragma unroll
    for (int t = 0; t < KT; ++t) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int m = 16 * t + 4 * g + j, mc = min(m, M - 1);
        bT[t][j] = (float)keep_if(phiT[((size_t)sbc * M + mc) * N + nc], okb && m < M);
        const double2 x = *reinterpret_cast<const double2*>(
            theta + ((((size_t)sc * 2 + qh) * M + mc) * N + nc) * 2);
        th[0][t][j] = (float)keep_if(x.x, okt && m < M);
        th[1][t][j] = (float)keep_if(x.y, okt && m < M);
      }
      // converted here: not all of the FP64 values at once in registers
      asm volatile("" : "+v"(bT[t]), "+v"(th[0][t]), "+v"(th[1][t])::"memory");
    }
  }
  // G vectors and h1' in groups of two; this workgroup's range of them
  const int ngrp = (G + 2) / 2;
  block_range rng(ngrp, blockIdx.y, gridDim.y, sum_blocks(ngrp));
  const int grp0 = rng.begin(), grp1 = rng.b.begin(rng.last);
  // operands of one row tile, read ahead: a[t] is reloaded right after its products
  fx4 a[KT];
  const fx4* Lw = Lop + (size_t)min(2 * grp0 + v1, G) * SLAB;
#pragma unroll
  for (int t = 0; t < KT; ++t) a[t] = Lw[t * 64 + lane];
  AFQMC_KEEP_AHEAD();
  fx4* yw = sY + (v1 * 4 * KT + g) * 16 * T + q;
  // stage 2's A operands: row 16 it + c of the packed rows is electron (16 it + c) % S of a vector
  const fx4* yr[T];
#pragma unroll
  for (int it = 0; it < T; ++it) {
    const int R = 16 * it + c;
    yr[it] = sY + ((R / S) * 4 * KT + g) * 16 * T + pp * S + R % S;
  }
  const bool late = Sh::NPR == 1 && pp == 1;  // (uniform in the wavefront)
  double e_re = 0.0, e_im = 0.0;  // this lane's share of E_p in the block of vectors
  if (Sh::NPR == 2 && pair == 1) __syncthreads();  // one barrier behind the first pair
  fx4 f[T][2];
  auto stage1 = [&](int grp) {
    const fx4* Ln = Lop + (size_t)min(2 * grp + 2 + v1, G) * SLAB;
    int ln = lane;
    asm volatile("" : "+v"(ln));  // offsets computed here, not kept over the loop
#pragma unroll
    for (int tp = 0; tp < KT; ++tp) {
      fx4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < KT; ++t) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          y = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t][j], bT[t][j], y, 0, 0, 0);
        a[t] = tp + 1 < KT ? Lw[((tp + 1) * KT + t) * 64 + ln] : Ln[t * 64 + ln];
        AFQMC_KEEP_AHEAD();
        __builtin_amdgcn_sched_barrier(0);  // the next row's products stay behind this row's
      }
      yw[4 * tp * 16 * T] = y;
    }
    Lw = Ln;
  };
  auto trace = [&](int grp) {
    // tr(f f): the partner of f^sp_{i n} is f^sp_{n i}, row n, packed column sp S + i; one
    // FP32 chain per vector over the lane's rows in order
    float x1r = 0.f, x1i = 0.f, x0r = 0.f, x0i = 0.f;  // running chain; the first vector's
#pragma unroll
    for (int it = 0; it < T; ++it) {
      const int R = 16 * it + 4 * g;
      if (T % 2 == 0 && it == T / 2) {  // the second vector begins
        x0r = x1r;
        x0i = x1i;
        x1r = 0.f;
        x1i = 0.f;
      } else if (T > 1 && T % 2 && it == T / 2) {  // lane groups 2, 3 have all of the first vector
        x0r = x1r;
        x0i = x1i;
        x1r = g < 2 ? x1r : 0.f;
        x1i = g < 2 ? x1i : 0.f;
      } else if (T % 2 && it == T / 2 + 1) {  // and 0, 1 now too
        x0r = g < 2 ? x1r : x0r;
        x0i = g < 2 ? x1i : x0i;
        x1r = g < 2 ? 0.f : x1r;
        x1i = g < 2 ? 0.f : x1i;
      }
      const float* p = sF + (R / S) * Sh::FV + qn * PW + qh * S + R % S;
      const fx4 pr = *reinterpret_cast<const fx4*>(p);
      const fx4 pi = *reinterpret_cast<const fx4*>(p + S * PW);
      AFQMC_KEEP_AHEAD();
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float ar = f[it][0][r], ai = f[it][1][r];
        x1r = fmaf(ar, pr[r], x1r);
        x1r = fmaf(-ai, pi[r], x1r);
        x1i = fmaf(ar, pi[r], x1i);
        x1i = fmaf(ai, pr[r], x1i);
      }
    }
    if (T == 1) {  // lane groups 0, 1 have the first vector, 2, 3 the second
      x0r = g < 2 ? x1r : 0.f;
      x0i = g < 2 ? x1i : 0.f;
      x1r = g < 2 ? 0.f : x1r;
      x1i = g < 2 ? 0.f : x1i;
    }
    if (2 * grp < G) {
      e_re -= 0.5 * (double)x0r;
      e_im -= 0.5 * (double)x0i;
    }
    if (2 * grp + 1 < G) {
      e_re -= 0.5 * (double)x1r;
      e_im -= 0.5 * (double)x1i;
    }
    // the diagonals' sums: 16 lanes per vector and part; the path's wavefronts take turns
    if (grp % T == w1) {
      const int v = lane >> 5, part = (lane >> 4) & 1;
      const float* p = sF + v * Sh::FV + part * S * PW;
      double x = 0.0;
#pragma unroll
      for (int e = 0; e < T; ++e) {
        const int k = c + 16 * e;  // packed column k: row k % S
        x += (double)p[(k % S) * PW + k];
      }
      x = row_sum(x);
      const double xi = __shfl_down(x, 16, 64);
      const int gam = 2 * grp + v;
      if ((lane & 31) == 0) {
        if (gam < G) {
          e_re += 0.5 * (x * x - xi * xi);
          e_im += x * xi;
          if (valid) *reinterpret_cast<double2*>(vb + ((size_t)s * G + gam) * 2) =
              active ? make_double2(x, xi) : make_double2(0.0, 0.0);
        } else if (gam == G) {
          e_re += x;
          e_im += xi;
        }
      }
    }
  };
  stage1(grp0);
  int bend = rng.end();
  for (int grp = grp0; grp < grp1; ++grp) {
    __syncthreads();
#pragma unroll
    for (int it = 0; it < T; ++it) f[it][0] = f[it][1] = fx4{0.f, 0.f, 0.f, 0.f};
    fx4 x[2];  // one operand read ahead
    x[0] = yr[0][0];
#pragma unroll
    for (int i = 0; i < KT * T; ++i) {
      const int t = i / T, it = i % T;
      if (i + 1 < KT * T) x[(i + 1) & 1] = yr[(i + 1) % T][4 * ((i + 1) / T) * 16 * T];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float xj = x[i & 1][j];
        f[it][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(xj, th[0][t][j], f[it][0], 0, 0, 0);
        f[it][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(xj, th[1][t][j], f[it][1], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int it = 0; it < T; ++it) {
      const int R = 16 * it + 4 * g;
      float* d = sF + (R / S) * Sh::FV + (R % S) * PW + q;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        d[r * PW] = f[it][0][r];
        d[S * PW + r * PW] = f[it][1][r];
      }
    }
    __syncthreads();
    if (!late) trace(grp);
    if (grp + 1 < grp1) stage1(grp + 1);
    if (late) trace(grp);
    if (grp + 1 == bend) {
      rng.add(e_re, e_im, epart, w1, T, n_samples, s, valid, active);
      e_re = e_im = 0.0;
      bend = rng.end();
    }
  }
  if (Sh::NPR == 2 && pair == 0) __syncthreads();
  const double2 e_wave = rng.total();  // with all lanes active
  if (lane == 0) *reinterpret_cast<double2*>(sT + wave * 2) = e_wave;
  __syncthreads();
  if (!rng.split && valid && w1 == 0 && lane == 0) {
    double re = 0.0, im = 0.0;
    for (int w = 0; w < T; ++w) {
      re += sT[(wave + w) * 2];
      im += sT[(wave + w) * 2 + 1];
    }
    *reinterpret_cast<double2*>(epart + (size_t)s * 2) =
        active ? make_double2(re, im) : make_double2(0.0, 0.0);
  }
}

template <int KT, int T>
hipError_t launch_f32(const afqmc_ctx_s* c, int n, int nsplit, const double* phiT,
                      const double* theta, const double* logov, double* vb, double* epart) {
  typedef Shape<KT, T> Sh;
  auto kern = k_contract_f32<KT, T>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)Sh::lds());
  if (e != hipSuccess) return e;
  constexpr int PP = 2 * Sh::NPR;  // paths per workgroup
  hipLaunchKernelGGL(kern, dim3((n + PP - 1) / PP, nsplit), dim3(64 * Sh::NW), Sh::lds(),
                     c->stream, n, c->M, c->N, c->G, reinterpret_cast<const fx4*>(c->d_Lpad32),
                     phiT, theta, logov, vb, epart);
  return hipGetLastError();
}

// L (double, row-major slabs) -> FP32 in A-operand order [slab][tp][t][g][c][j] =
// L[slab][16 tp + c][16 t + 4 g + j]; n = slabs x MT x MT.
__global__ void k_to_f32_op(size_t n, int MT, const double* __restrict__ src,
                            float* __restrict__ dst) {
  const size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= n) return;
  const int KT = MT / 16;
  const size_t slab = o / ((size_t)MT * MT);
  const int r = (int)(o % ((size_t)MT * MT));
  const int j = r & 3, cc = (r >> 2) & 15, gg = (r >> 6) & 3, t = (r >> 8) % KT, tp = (r >> 8) / KT;
  dst[o] = (float)src[slab * MT * MT + (size_t)(16 * tp + cc) * MT + 16 * t + 4 * gg + j];
}

}  // namespace

// 8-wide column tiles a path: with three past M = 96 a workgroup's two pairs of paths would need
// 162 KB of LDS and more, so that four, with one pair, take those sizes (the fourth is padding)
static int tiles(const afqmc_ctx_s* c) {
  const int T = (c->N + 7) / 8;
  return T == 3 && c->MT > 96 ? 4 : T;
}

// Ranges of g (slots: one workgroup a CU, or three of the small ones of N <= 8; at least
// eight groups of vectors to a range).  256 paths of M = 96, N = 24 (64 workgroups): 2.8 ms in
// one range, 0.72 in four.
contract_plan contract_f32_plan(const afqmc_ctx_s* c, int nw) {
  const int T = tiles(c), pp = T == 4 ? 2 : 4;
  const int ngrp = (c->G + 2) / 2;
  return plan_splits(((long)nw * c->P + pp - 1) / pp, T > 1 ? 256 : 768, ngrp, 8, T,
                     sum_blocks(ngrp));
}

hipError_t launch_contract_f32(const afqmc_ctx_s* c, int nw, int nsplit, const double* phiT,
                               const double* theta, const double* logov, double* vb,
                               double* epart) {
  if (nw <= 0) return hipSuccess;
  if (c->d_Lpad32 == nullptr) return hipErrorInvalidValue;
  const int n = nw * c->P, T = tiles(c);
#define AFQMC_CF(KK, TT)            \
  if (c->MT == 16 * KK && T == TT) \
    return launch_f32<KK, TT>(c, n, nsplit, phiT, theta, logov, vb, epart);
  AFQMC_CF(1, 1) AFQMC_CF(2, 1) AFQMC_CF(3, 1) AFQMC_CF(4, 1)
  AFQMC_CF(5, 1) AFQMC_CF(6, 1) AFQMC_CF(7, 1) AFQMC_CF(8, 1)
  AFQMC_CF(1, 2) AFQMC_CF(2, 2) AFQMC_CF(3, 2) AFQMC_CF(4, 2)
  AFQMC_CF(5, 2) AFQMC_CF(6, 2) AFQMC_CF(7, 2) AFQMC_CF(8, 2)
  AFQMC_CF(2, 3) AFQMC_CF(3, 3) AFQMC_CF(4, 3) AFQMC_CF(5, 3) AFQMC_CF(6, 3)
  AFQMC_CF(2, 4) AFQMC_CF(3, 4) AFQMC_CF(4, 4)
  AFQMC_CF(5, 4) AFQMC_CF(6, 4) AFQMC_CF(7, 4) AFQMC_CF(8, 4)
#undef AFQMC_CF
  return hipErrorInvalidValue;
}

hipError_t launch_to_f32_op(const afqmc_ctx_s* c, size_t n, const double* src, float* dst) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_to_f32_op, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, n,
                     c->MT, src, dst);
  return hipGetLastError();
}
