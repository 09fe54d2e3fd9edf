// Walker propagation in FP64 on the workgroup kernels (Sec. II.A, Eq. HS; Sec. II.B,
// Eq. walker_prop; the trial slices of Sec. II.C and the back-propagated bras of App. B):
// dst = El T_n(V) Er src for blocks of `spins` M x N complex matrices that share a V.
//
// Bound: the FP64 matrix cores.  The real and imaginary columns of all blocks of a V stand
// side by side, 16 to a wavefront, which keeps its columns of the Horner iterate in
// registers from start to end: an accumulator tile's entry is the next term's B operand
// (dev_common.h), and the columns of i Y that Im V multiplies are a lane exchange away.
// Only V is shared, through LDS, in double-buffered panels of 16 rows that come straight
// from global memory while the panel before multiplies.  X = Er src is read back from dst
// (or src) for every term rather than held.  So no product pads N to 16 (only the last of
// the 2 spins N / 16 column tiles is ragged) and the contraction index ends at M; the form
// with a wavefront per row tile (k_taylor_g) pads both and spends a barrier pair a term.
// M = 72, N = 18, 700 walkers: 701 -> 392 us (16 -> 28 TFLOP/s of the unpadded products);
// M = 142, N = 35, 300 walkers, the whole move 2.72 -> 2.16 ms; M = 80, N = 21, 50 walkers
// of 5 blocks, 20 terms of back-propagation, 5.48 -> 3.24 ms.
#include <algorithm>

#include "afqmc_internal.h"
#include "dev_common.h"

namespace {

typedef double dx2 __attribute__((ext_vector_type(2)));

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __attribute__((address_space(1))) void* gbl_ptr_t;

// LDS entries (complex) of one panel: 16 rows of V in whole 1 KB copies, and the
// columns past M that the last row's operands reach
__host__ __device__ constexpr int panel_size(int M) { return (16 * M + 63) / 64 * 64 + 16; }

template <int KT>
__global__ void __launch_bounds__(320, KT <= 5 ? 4 : KT <= 7 ? 3 : 2)
k_taylor_q(int n, int M, int N, int n_taylor, int spins, int nct, int parts,
           const double* __restrict__ vmat, const double* __restrict__ El,
           const double* __restrict__ Er, const double* src, int src_ws, double* dst) {
  extern __shared__ __attribute__((aligned(16))) double smem[];
  const int w = blockIdx.x / parts, part = blockIdx.x % parts;
  const int nwv = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = lane >> 4, c = lane & 15;
  const int ps = panel_size(M);
  const dx2* V = reinterpret_cast<const dx2*>(vmat) + (size_t)w * M * M;
  // this lane's real column: part ri of complex column q of the blocks side by side
  // column tiles of this workgroup; which wavefronts idle when they are fewer rotates, so
  // that the idle ones of a CU's workgroups fall on different SIMDs
  const int per = (nct + parts - 1) / parts, slot = (wave + (int)blockIdx.x) % nwv;
  const int ct = slot < per ? part * per + slot : nct;
  const int q = 8 * ct + (c >> 1), ri = c & 1;
  const bool okc = ct < nct && q < spins * N;
  const int sp = okc ? q / N : 0, nn = okc ? q % N : 0;
  const double* in = src + ((size_t)w * src_ws + sp) * M * N * 2 + 2 * nn + ri;
  double* out = dst + ((size_t)w * spins + sp) * M * N * 2 + 2 * nn + ri;

  // panel p (rows 16 p ..) of V to buffer b, straight from global memory
  auto copy_panel = [&](int p, int b) {
    int e = lane;
    asm volatile("" : "+v"(e));  // addresses computed here, not kept over the loop on the terms
    const dx2* src = V + p * 16 * M;
    const int chunks = ps / 64, last = M * M - 1 - p * 16 * M;
    for (int k = wave; k < chunks; k += nwv)
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)(src + min(k * 64 + e, last)),
                                       (lds_ptr_t)(smem + 2 * (b * ps + k * 64)), 16, 0, 0);
  };
  // orbitals past M: their rows of V are whatever the buffer holds, times zero
  for (int k = threadIdx.x; k < 4 * ps; k += blockDim.x) smem[k] = 0.0;
  double y[KT][4];
  auto row_ok = [&](int t, int r) { return t < KT - 1 || 16 * t + 4 * r + g < M; };
  // rows 16 t + 4 r + g of this lane's column at p, 0 outside M and the columns
  auto load_x = [&](const double* p, int t, double (&x)[4]) {
    int gg = g;
    asm volatile("" : "+v"(gg));
#pragma unroll
    for (int r = 0; r < 4; ++r)
      x[r] = keep_if(p[(unsigned)min(16 * t + 4 * r + gg, M - 1) * 2 * N], okc && row_ok(t, r));
  };
#pragma unroll
  for (int t = 0; t < KT; ++t) load_x(in, t, y[t]);
  dx4 acc[KT];
  auto apply = [&](const double* E) {  // acc = E y
#pragma unroll
    for (int q2 = 0; q2 < KT; ++q2) acc[q2] = dx4_zero();
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (t < KT - 1 || 16 * t + 4 * r < M) {
          int gg = g;
          asm volatile("" : "+v"(gg));
          const double* row = E + min(16 * t + 4 * r + gg, M - 1) * M;
          double e[KT];
#pragma unroll
          for (int q2 = 0; q2 < KT; ++q2) e[q2] = row[min(16 * q2 + c, M - 1)];
#pragma unroll
          for (int q2 = 0; q2 < KT; ++q2) acc[q2] = mfma_f64(e[q2], y[t][r], acc[q2]);
        }
  };
  const double* xp = in;  // X = Er src
  if (Er != nullptr) {
    apply(Er);
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool ok = okc && row_ok(t, r);
        y[t][r] = ok ? acc[t][r] : 0.0;
        if (ok) out[(size_t)(16 * t + 4 * r + g) * 2 * N] = y[t][r];
      }
    xp = out;
  }
  __syncthreads();
  copy_panel(0, 0);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  __syncthreads();
  int b = 0;
  for (int j = n_taylor; j >= 1; --j) {
#pragma unroll
    for (int q2 = 0; q2 < KT; ++q2) acc[q2] = dx4_zero();
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      // the next panel (of the next term after the last) while this one multiplies
      copy_panel(t + 1 < KT ? t + 1 : 0, b ^ 1);
      int ln = lane;
      asm volatile("" : "+v"(ln));
      const dx2* sv = reinterpret_cast<const dx2*>(smem) + b * ps + (ln >> 4) * M + (ln & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (t < KT - 1 || 16 * t + 4 * r < M) {
          // (re, im) columns of i Y: (-Im, Re)
          const double b1 = y[t][r], sw = dpp_f64<0xB1>(b1), b2 = ri ? sw : -sw;
#pragma unroll
          for (int q2 = 0; q2 < KT; ++q2) {
            const dx2 v = sv[4 * r * M + 16 * q2];
            acc[q2] = mfma_f64(v.x, b1, acc[q2]);
            acc[q2] = mfma_f64(v.y, b2, acc[q2]);
          }
        }
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the next panel is in LDS
      __syncthreads();
      b ^= 1;
    }
    const double invj = 1.0 / (double)j;
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      double x[4];
      load_x(xp, t, x);
#pragma unroll
      for (int r = 0; r < 4; ++r) y[t][r] = row_ok(t, r) ? fma(acc[t][r], invj, x[r]) : 0.0;
    }
  }
  apply(El);
#pragma unroll
  for (int t = 0; t < KT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (okc && row_ok(t, r)) out[(size_t)(16 * t + 4 * r + g) * 2 * N] = acc[t][r];
}

// Workgroups and their wavefronts for n V of `spins` blocks: up to five column tiles in one
// workgroup, more in fours (3 or 4 wavefronts active)
struct q_shape {
  int nct, nwv, parts, active;
  q_shape(int N, int spins)
      : nct((spins * N + 7) / 8),
        nwv(nct <= 5 ? nct : 4),
        parts((nct + nwv - 1) / nwv),
        active((nct + parts - 1) / parts) {}
};

template <int KT>
hipError_t launch_q(const afqmc_ctx_s* c, int n, int spins, int n_taylor, const double* vmat,
                    const double* El, const double* Er, const double* src, int src_ws,
                    double* dst) {
  const q_shape q(c->N, spins);
  const size_t lds = (size_t)2 * panel_size(c->M) * 16;
  auto kern = k_taylor_q<KT>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(n * q.parts), dim3(64 * q.nwv), lds, c->stream, n, c->M, c->N,
                     n_taylor, spins, q.nct, q.parts, vmat, El, Er, src, src_ws, dst);
  return hipGetLastError();
}

}  // namespace

namespace {
// The time of `groups` workgroups of w wavefronts on the chip's 256 CUs, `fit` of them at a
// time on one, in passes of one wavefront: each batch takes as long as its busiest SIMD.
// Workgroups that share a CU overlap a little; a lone wavefront on a SIMD waits more.
double passes(long groups, int fit, int w) {
  auto batch = [&](int r) {
    const double b = std::max((double)((w * r + 3) / 4), 0.85 * r * ((w + 3) / 4));
    return r == 0 ? 0.0 : std::max(b, 1.25);
  };
  const int r = (int)((groups + 255) / 256);
  return (r / fit) * batch(fit) + batch(r % fit);
}
}  // namespace

// Against k_taylor_g, whose workgroup is one block's row tiles: the time of each from its
// products a wavefront (the padding of N to 16 and of the contraction index is its loss) and
// the passes that its workgroups take.  This one has fewer and longer wavefronts, so that it
// is for calls that fill the chip: M = 72, N = 18, walker moves, k_taylor_g and here, 100
// walkers 154 and 182 us, 140 271 and 189, 500 518 and 294; M = 128, N = 20, 100 walkers 243
// and 428, 300 626 and 824; M = 142, N = 35, 20 walkers 545 and 373, 300 1684 and 1150.  Over
// 220 sizes the choice is 0.2 % behind the better one in the mean (the products alone, for calls
// of 256 wavefronts or more: 5 %).  Both give the same bits, so that a walker does not depend on
// how many others share the call.
bool taylor_q_better(const afqmc_ctx_s* c, int n, int spins) {
  const int KT = c->MT / 16, KS = (c->M + 3) / 4, ntc = (c->N + 15) / 16;
  const q_shape q(c->N, spins);
  const int waves = KT <= 5 ? 16 : KT <= 7 ? 12 : 8;  // by registers, of this kernel on a CU
  const int fit = std::max(1, std::min(waves / q.nwv, (160 * 1024) / (2 * panel_size(c->M) * 16)));
  const double here = 2.0 * KT * KS * passes((long)n * q.parts, fit, q.active);
  const double there = 16.0 * ntc * KT * passes((long)n * spins, KT <= 4 ? 2 : 1, KT);
  return there >= 1.1 * here;
}

hipError_t launch_taylor_q(const afqmc_ctx_s* c, int n, int spins, int n_taylor,
                           const double* vmat, const double* El, const double* Er,
                           const double* src, int src_ws, double* dst) {
  if (n <= 0) return hipSuccess;
  switch (c->MT / 16) {
#define AFQMC_T(KK) \
  case KK: return launch_q<KK>(c, n, spins, n_taylor, vmat, El, Er, src, src_ws, dst);
    AFQMC_T(1) AFQMC_T(2) AFQMC_T(3) AFQMC_T(4) AFQMC_T(5)
    AFQMC_T(6) AFQMC_T(7) AFQMC_T(8) AFQMC_T(9) AFQMC_T(10)
#undef AFQMC_T
    default: return hipErrorInvalidValue;
  }
}
