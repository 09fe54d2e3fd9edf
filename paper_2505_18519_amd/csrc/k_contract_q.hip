// FP64 Cholesky contraction, any M <= 160 and N <= 40: force bias and local energy
//  of every path (Sec. III.A, Eq. local-obs; Eq. shift1).  Per
// path p and vector g (both spins s):
//   Y_g = Phi_T^T L_g,  f_g^s = Y_g Theta^s,  vb_g = sum_s tr f_g^s,
//   E_p = sum_s tr(Phi_T^T h1' Theta^s) + 1/2 sum_g [vb_g^2 - sum_s tr(f_g^s f_g^s)].
// h1' rides along as slab g = n_chol of the padded L array.
//
// Bound: the FP64 matrix cores (72 TFLOP/s in a large product on this card).  Both
// stages are laid out so that they multiply no padding beyond N rounded up to 4, which
// the 4x4x4 FP64 product makes possible: it runs at the rate of the 16x16x4 one (76.7
// against 76.9 TFLOP/s measured).
//  * Four vectors g at a time.  Stage 1 gives a vector to each wavefront (two to a
//    vector with eight): Y_g^T = L_g Phi_T with rows of L_g from global memory as A
//    operands, Phi_T in 16-wide column tiles and, for the N mod 16 rest, 4-wide ones.
//  * Stage 2 is one product of a path's Theta (4 N rows: orbital, spin, real and
//    imaginary part) with the stacked Y of the four vectors (4 N columns), both whole
//    multiples of 16; a wavefront keeps its tiles of f in registers over the loop on
//    the orbitals, which runs in chunks of rows of Y^T that fit LDS.
//  * tr(f f) pairs the tiles (a, b) and (b, a), so half of f goes through LDS.
// CT, the complex trial determinants of multi-slice trials: stage 1 runs on the planes
// Re Phi_T and Im Phi_T, which share each L operand, and stage 2 sums Y_re Theta and Y_im
// (i Theta), the second from Theta's parts exchanged and signed.
// PP = 2 paths share a workgroup where L_g's L2 traffic would bound (N <= 20): each L
// operand then feeds both paths.  A few paths (or a last round of workgroups that fills
// little of the chip) are split further over ranges of g (contract_q_plan).
//
// Measured on 2048 paths (M > 128: 1024), before (operands in registers, or for N > 32
// streamed, N padded to 16) and now, TFLOP/s of the unpadded products:
// M = 24, N = 6: 7.7 -> 18.7; 45, 11: 18 -> 36; 72, 18: 15 -> 46; 96, 24: 34 -> 58;
// 128, 16: 42 -> 61; 112, 28: 45 -> 56; 142, 35: 18 -> 55; 160, 40: 31 -> 58; 128, 32:
// 60 -> 60.
#include "afqmc_internal.h"
#include "contract_sum.h"
#include "dev_common.h"

namespace {

// D(4x4, four blocks b) += A_b(4x4) B_b(4x4).  Lane l = 16 g + 4 b + i supplies
// A_b[i][g] and B_b[g][i] and holds D_b[g][i].
__device__ __forceinline__ double mfma_f64_4(double a, double b, double acc) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, acc, 0, 0, 0);
}

constexpr int GV = 4;  // vectors of a group

template <int NG, int KC, int NW, int PP, bool CT>
struct qshape {
  static_assert(!CT || PP == 1, "complex trials: one path a workgroup");
  static constexpr int PL = CT ? 2 : PP;  // planes of Phi_T and Y: paths, or real and imaginary
  static constexpr int NF = NG / 4, NR = NG % 4;  // 16- and 4-wide column tiles of Phi_T
  static constexpr int NF1 = NF > 0 ? NF : 1, NR1 = NR > 0 ? NR : 1;
  static constexpr int HV = NW / GV;           // wavefronts that share a vector in stage 1
  static constexpr int MC = 16 * KC * HV;      // rows of Y^T of one chunk
  static constexpr int SYS = MC * 16 + 4;      // stride of the row groups of Y in LDS
  static constexpr int NWP = NW / PP;             // wavefronts of a path in stage 2
  static constexpr int NWA = NG < NWP ? NG : NWP;  // of them with tiles of f
  // a wavefront's tiles (jg, ig) of f: NC whole columns jg, and of the NL tiles of the
  // columns left over at most NE, in NX columns
  static constexpr int NC = NG / NWA, NL = (NG - NC * NWA) * NG, NE = (NL + NWA - 1) / NWA;
  static constexpr int extra_columns() {
    int m = 0;
    for (int w = 0; w < NWA; ++w) {
      const int e0 = w * NL / NWA, e1 = (w + 1) * NL / NWA;
      if (e1 > e0 && (e1 - 1) / NG - e0 / NG + 1 > m) m = (e1 - 1) / NG - e0 / NG + 1;
    }
    return m;
  }
  static constexpr int NX = extra_columns();
  static_assert(NX <= 2, "leftover tiles of a wavefront span at most two columns");
  static constexpr int NB = NC + NX;  // tile columns touched
  static constexpr int NPAIR = NG * (NG - 1) / 2;
  // doubles of the shared buffer: Y of a chunk, then one tile of f per pair
  static constexpr int SBUF = PL * NG * SYS > PP * NPAIR * 256 ? PL * NG * SYS : PP * NPAIR * 256;
};

template <int NG, int KC, int NW, int PP, bool CT>
__global__ void __launch_bounds__(64 * NW, 2)
k_contract_q(int n_samples, int M, int N, int G, int KT, const double* __restrict__ Lpad,
             const double* __restrict__ phiT, const double* __restrict__ theta,
             const double* __restrict__ logov, double* __restrict__ vb, double* __restrict__ epart) {
  typedef qshape<NG, KC, NW, PP, CT> Q;
  constexpr int PL = Q::PL, NF = Q::NF, NR = Q::NR, NF1 = Q::NF1, NR1 = Q::NR1, HV = Q::HV, MC = Q::MC,
                SYS = Q::SYS, NWP = Q::NWP, NWA = Q::NWA, NC = Q::NC, NL = Q::NL, NE = Q::NE,
                NB = Q::NB, NX = Q::NX, NE1 = NE > 0 ? NE : 1;
  extern __shared__ __attribute__((aligned(16))) double smem[];
  const int MT = 16 * KT;
  double* sY = smem;  // [PL][NG][SYS], then f [PP][pair][spin][lane][2]
  // Phi_T by steps of 4 orbitals: per plane NF operands [4][16], then NR operands [4][4]
  double* sP = sY + Q::SBUF;
  double* sD = sP + 4 * KT * PL * 16 * NG;  // [2][NW][16][2] diagonal sums
  double* sE = sD + 2 * NW * 32;          // [NW][2]

  const int s0 = blockIdx.x * PP;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int g = lane >> 4, c = lane & 15;
  // path of this wavefront in stage 2 and its place among that path's wavefronts
  const int pw = wave / NWP, wi = wave % NWP;
  // groups of this workgroup's range; vectors 0 .. G (h1') in all
  block_range rng((G + GV) / GV, blockIdx.y, gridDim.y);
  const int grp0 = rng.begin(), grp1 = rng.b.begin(rng.last);
  bool active[PP];  // singular paths contribute zero
  bool any = false;
#pragma unroll
  for (int p = 0; p < PP; ++p) {
    active[p] = s0 + p < n_samples && !__builtin_isinf(logov[2 * (size_t)min(s0 + p, n_samples - 1)]);
    any |= active[p];
    if (s0 + p < n_samples && !active[p]) {
      for (int q = tid + 64 * NW * blockIdx.y; q < 2 * G; q += 64 * NW * gridDim.y)
        vb[(size_t)(s0 + p) * G * 2 + q] = 0.0;
      if (rng.split) {
        if (wave < NWP) zero_blocks(rng, epart, wave, NWP, n_samples, s0 + p, lane);
      } else if (tid < 2) {
        epart[2 * (size_t)(s0 + p) + tid] = 0.0;
      }
    }
  }
  if (!any) return;
  // Phi_T to LDS, zero outside M x N
#pragma unroll
  for (int p = 0; p < PL; ++p) {
    const int pp = CT ? 0 : p;
    const double* src = phiT + (size_t)min(s0 + pp, n_samples - 1) * M * N * (CT ? 2 : 1);
    for (int q = tid; q < MT * 4 * NG; q += 64 * NW) {
      const int m = q / (4 * NG), n = q % (4 * NG);
      const size_t e = (size_t)min(m, M - 1) * N + min(n, N - 1);
      const double x = keep_if(CT ? src[2 * e + p] : src[e], active[pp] && m < M && n < N);
      double* d = sP + ((m >> 2) * PL + p) * 16 * NG;
      if (n < 16 * NF) d[(n >> 4) * 64 + (m & 3) * 16 + (n & 15)] = x;
      else d[NF * 64 + ((n >> 2) - 4 * NF) * 16 + (m & 3) * 4 + (n & 3)] = x;
    }
  }
  const int v = wave & 3, h = wave >> 2;
  const size_t slab = (size_t)MT * MT;
  // the last 16-wide tile of the contraction index holds more than 8 of the M rows
  const bool whole = M > 16 * KT - 8;
  const int KH = (M + 7) / 8;

  double e_re = 0.0, e_im = 0.0;  // this lane's share of E_p in the block of vectors

  const unsigned lofs = g * MT + c;  // this lane's entry of a 4 x 16 operand of L
  auto load_l = [&](const double* Lg, int tb, int t, double (&o)[4][KC]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double* p = Lg + (size_t)(16 * t + 4 * r) * MT;
#pragma unroll
      for (int q = 0; q < KC; ++q) o[r][q] = p[lofs + 16 * min(tb + q, KT - 1)];
    }
  };
  // stage 1 for the first n of KC row tiles from tb: Y_g^T = L_g Phi_T, A[c][g] =
  // L[4 k + g][16 tp + c] (L symmetric); L operands one 16-wide k tile ahead (the last
  // trip loads the next chunk's first), Phi_T operands one step ahead
  dx4 y[PL][KC][NF1];
  double yr[PL][KC][NR1];
  double ac[4][KC];
  auto stage1 = [&](auto QN, const double* Lg, int tb, const double* Ln, int tbn) {
    constexpr int n = decltype(QN)::value;
    int ln = lane;
    asm volatile("" : "+v"(ln));  // addresses computed here, not kept over the loop over g
    const double *pf = sP + ln, *pr = sP + NF * 64 + (ln >> 4) * 4 + (ln & 3);
    auto load_p = [&](int k, double (&bf)[PL][NF1], double (&br)[PL][NR1]) {  // step k from pf
#pragma unroll
      for (int p = 0; p < PL; ++p) {
#pragma unroll
        for (int ct = 0; ct < NF; ++ct) bf[p][ct] = pf[(k * PL + p) * 16 * NG + ct * 64];
#pragma unroll
        for (int ct = 0; ct < NR; ++ct) br[p][ct] = pr[(k * PL + p) * 16 * NG + ct * 16];
      }
    };
    double an[4][KC];
    double bf[2][PL][NF1], br[2][PL][NR1];
    load_p(0, bf[0], br[0]);
    auto step = [&](int r, const double (&a)[KC], double (&b0)[PL][NF1], double (&b1)[PL][NR1]) {
#pragma unroll
      for (int q = 0; q < n; ++q)
#pragma unroll
        for (int p = 0; p < PL; ++p) {
#pragma unroll
          for (int ct = 0; ct < NF; ++ct) y[p][q][ct] = mfma_f64(a[q], b0[p][ct], y[p][q][ct]);
#pragma unroll
          for (int ct = 0; ct < NR; ++ct) yr[p][q][ct] = mfma_f64_4(a[q], b1[p][ct], yr[p][q][ct]);
        }
    };
    for (int t = 0; t < KT - 1; ++t) {
      load_l(Lg, tb, t + 1, an);
      AFQMC_KEEP_AHEAD();
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        load_p(r + 1, bf[(r + 1) & 1], br[(r + 1) & 1]);
        step(r, ac[r], bf[r & 1], br[r & 1]);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = 0; q < KC; ++q) ac[r][q] = an[r][q];
      pf += 4 * PL * 16 * NG;
      pr += 4 * PL * 16 * NG;
    }
    load_l(Ln, tbn, 0, an);
    AFQMC_KEEP_AHEAD();
    load_p(1, bf[1], br[1]);
    step(0, ac[0], bf[0], br[0]);
    if (whole) load_p(2, bf[0], br[0]);
    step(1, ac[1], bf[1], br[1]);
    if (whole) {
      load_p(3, bf[1], br[1]);
      step(2, ac[2], bf[0], br[0]);
      step(3, ac[3], bf[1], br[1]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int q = 0; q < KC; ++q) ac[r][q] = an[r][q];
  };

  // stage 2: tile (jg, ig) of f holds, at lane 16 j + 4 v + i and element 2 s + part,
  // f_v^s[4 ig + i][4 jg + j]: A = Theta (rows 4 q + j), B = Y (columns 4 v + i).
  // Wavefront wi of a path has the columns jg = wi NC + b and the leftover tiles
  // e0 .. e0 + ne - 1, tile e being (NC NWA + e / NG, e % NG).
  const int e0 = wi * NL / NWA, ne = (wi + 1) * NL / NWA - e0;
  const int ie = NL > 0 ? e0 % NG : 0, je = NC * NWA + (NL > 0 ? e0 / NG : 0);
  const bool tiles = wi < NWA;
  dx4 f[NC][NG], fe[NE1];
  constexpr int TP = CT ? 2 : 1;  // Theta operands of a tile column: Theta, i Theta
  double bc[2][TP][NB];
  const double* th = theta + (size_t)min(s0 + pw, n_samples - 1) * 4 * M * N;
  double* sYp = sY + (CT ? 0 : pw) * NG * SYS;
  auto load_t = [&](int t, double (&o)[2][TP][NB]) {  // Theta operands of steps 2 t, 2 t + 1
    int cc = c;
    asm volatile("" : "+v"(cc));  // offsets computed here, not kept over the loop over g
    unsigned co[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int jg = b < NC ? wi * NC + b : je + b - NC;
      co[b] = (cc >> 3) * 2 * M * N + 2 * min(4 * jg + (cc & 3), N - 1) + ((cc >> 2) & 1);
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const unsigned m = min(8 * t + 4 * r + g, M - 1);
#pragma unroll
      for (int b = 0; b < NB; ++b) o[r][0][b] = th[co[b] + m * 2 * N];
      if constexpr (CT) {  // i Theta: -Im, Re
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const double x = th[(co[b] ^ 1) + m * 2 * N];
          o[r][TP - 1][b] = (cc & 4) ? x : -x;
        }
      }
    }
  };
  auto stage2 = [&](int ch0) {
    const int kt = min(MC / 8, KH - 2 * ch0);  // pairs of steps of this chunk
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const double* py = sYp + ln;
    const double* pe = py + ie * SYS;
    const int wrap = NG - ie;  // leftover tiles from this one on are in the second column
    // Y operands of step k from py, plane p
    auto load_y = [&](int k, double (&a)[TP][NG], double (&e)[TP][NE1]) {
#pragma unroll
      for (int p = 0; p < TP; ++p) {
#pragma unroll
        for (int ig = 0; ig < NG; ++ig) a[p][ig] = py[(p * NG + ig) * SYS + k * 64];
#pragma unroll
        for (int q = 0; q < NE; ++q)
          if (q + 1 < NE || NL % NWA == 0 || q < ne)
            e[p][q] = pe[(p * NG + (NX == 2 && q >= wrap ? q - NG : q)) * SYS + k * 64];
      }
    };
    double a[2][TP][NG], e[2][TP][NE1], bn[2][TP][NB];
    load_y(0, a[0], e[0]);
    auto step = [&](int r) {
#pragma unroll
      for (int p = 0; p < TP; ++p) {
        unrolled<NC * NG>([&](auto I) {
          constexpr int b = decltype(I)::value / NG, ig = decltype(I)::value % NG;
          f[b][ig] = mfma_f64(bc[r][p][b], a[r][p][ig], f[b][ig]);
        });
        unrolled<NE>([&](auto I) {
          constexpr int q = decltype(I)::value;
          if (q + 1 < NE || NL % NWA == 0 || q < ne)
            fe[q] = mfma_f64(NX == 2 && q < wrap ? bc[r][p][NB - 2] : bc[r][p][NB - 1], e[r][p][q],
                             fe[q]);
        });
      }
    };
    for (int t = 0; t < kt - 1; ++t) {
      load_t(2 * ch0 + t + 1, bn);
      AFQMC_KEEP_AHEAD();
      load_y(1, a[1], e[1]);
      step(0);
      load_y(2, a[0], e[0]);
      step(1);
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int p = 0; p < TP; ++p)
#pragma unroll
          for (int b = 0; b < NB; ++b) bc[r][p][b] = bn[r][p][b];
      py += 128;
      pe += 128;
    }
    load_y(1, a[1], e[1]);
    step(0);
    step(1);
  };
  // every tile of this wavefront: fn(tile, ig, jg)
  auto each = [&](auto fn) {
    unrolled<NC * NG>([&](auto I) {
      constexpr int b = decltype(I)::value / NG, ig = decltype(I)::value % NG;
      fn(f[b][ig], ig, wi * NC + b);
    });
    unrolled<NE>([&](auto I) {
      constexpr int q = decltype(I)::value;
      if (q < ne) fn(fe[q], ie + q < NG ? ie + q : ie + q - NG, ie + q < NG ? je : je + 1);
    });
  };
  // tr(f f): of the tiles (a, b) and (b, a), a < b, one wavefront's goes through LDS and
  // the other reads it transposed (which one alternates, for balance); a diagonal tile is
  // transposed by lane permutes.  Entry l = 16 x + y of a staged tile sits at 16 x + (y + x)
  // mod 16, so that both the rows written and the columns read spread over the banks.
  double* sFp = sY + pw * Q::NPAIR * 256;
  auto staged = [](int ig, int jg) { return ((ig + jg) & 1) == (jg > ig ? 1 : 0); };
  auto slot = [](int ig, int jg) {
    const int hi = max(ig, jg), lo = min(ig, jg);
    return (hi * (hi - 1) / 2 + lo) * 256;
  };
  auto put_f = [&]() {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    double* dl = sFp + ((ln & 48) | ((ln + (ln >> 4)) & 15)) * 2;
    each([&](const dx4& x, int ig, int jg) {
      if (ig != jg && staged(ig, jg)) {
        double* d = dl + slot(ig, jg);
        *reinterpret_cast<double2*>(d) = make_double2(x[0], x[1]);
        *reinterpret_cast<double2*>(d + 128) = make_double2(x[2], x[3]);
      }
    });
  };
  auto get_f = [&](bool ok_v) {
    double o_re = 0.0, o_im = 0.0, d_re = 0.0, d_im = 0.0;
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int lg = ln >> 4, lj = ln & 3, lv = ln & 12;
    const double* sl = sFp + (16 * lj + ((lv + lg + lj) & 15)) * 2;
    each([&](const dx4& x0, int ig, int jg) {
      if (ig != jg && staged(ig, jg)) return;
      dx4 x = x0;
      if (max(ig, jg) == NG - 1) {  // outside N x N
        const bool ok = 4 * ig + lj < N && 4 * jg + lg < N;
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = ok ? x[r] : 0.0;
      }
      if (ig != jg) {
        const double* p = sl + slot(ig, jg);
        const double2 z0 = *reinterpret_cast<const double2*>(p);
        const double2 z1 = *reinterpret_cast<const double2*>(p + 128);
        o_re = fma(x[0], z0.x, o_re);
        o_im = fma(x[0], z0.y, o_im);
        o_re = fma(-x[1], z0.y, o_re);
        o_im = fma(x[1], z0.x, o_im);
        o_re = fma(x[2], z1.x, o_re);
        o_im = fma(x[2], z1.y, o_im);
        o_re = fma(-x[3], z1.y, o_re);
        o_im = fma(x[3], z1.x, o_im);
      } else {
        const int src = 16 * lj + lv + lg;
        dx4 z;
#pragma unroll
        for (int r = 0; r < 4; ++r) z[r] = __shfl(x[r], src, 64);
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
          d_re = fma(x[r], z[r], d_re);
          d_im = fma(x[r], z[r + 1], d_im);
          d_re = fma(-x[r + 1], z[r + 1], d_re);
          d_im = fma(x[r + 1], z[r], d_im);
        }
      }
    });
    const double t_re = fma(2.0, o_re, d_re), t_im = fma(2.0, o_im, d_im);
    e_re -= ok_v ? 0.5 * t_re : 0.0;
    e_im -= ok_v ? 0.5 * t_im : 0.0;
  };
  // the diagonal elements f_v[i][i] of both spins, summed over this wavefront's tiles
  auto put_d = [&](double* d) {
    double x = 0.0, z = 0.0;
    each([&](const dx4& t, int ig, int jg) {
      if (ig == jg) {
        const bool ok = 4 * ig + g < N;
        x += ok ? t[0] + t[2] : 0.0;
        z += ok ? t[1] + t[3] : 0.0;
      }
    });
    if ((c & 3) == g) *reinterpret_cast<double2*>(d + (wave * 16 + c) * 2) = make_double2(x, z);
  };

  const double* Lv = Lpad + (size_t)min(GV * grp0 + v, G) * slab;  // this wavefront's vector
  load_l(Lv, h * KC, 0, ac);
  __syncthreads();
  int bend = rng.end();
  for (int grp = grp0; grp < grp1; ++grp) {
    const double* Lnext = Lpad + (size_t)min(GV * (grp + 1) + v, G) * slab;
    unrolled<NC * NG>(
        [&](auto I) { f[decltype(I)::value / NG][decltype(I)::value % NG] = dx4_zero(); });
    unrolled<NE>([&](auto I) { fe[decltype(I)::value] = dx4_zero(); });
    for (int ch0 = 0; ch0 < KT; ch0 += KC * HV) {
      const int tb = ch0 + h * KC;
      const bool lastc = ch0 + KC * HV >= KT;
      const double* Ln = lastc ? Lnext : Lv;
      const int tbn = lastc ? h * KC : tb + KC * HV;
#pragma unroll
      for (int p = 0; p < PL; ++p)
#pragma unroll
        for (int q = 0; q < KC; ++q) {
#pragma unroll
          for (int ct = 0; ct < NF; ++ct) y[p][q][ct] = dx4_zero();
#pragma unroll
          for (int ct = 0; ct < NR; ++ct) yr[p][q][ct] = 0.0;
        }
      const int rows = KT - tb;  // a half chunk past the last row tile has none
      if (rows >= KC) stage1(std::integral_constant<int, KC>{}, Lv, tb, Ln, tbn);
      else if (rows > 0) {
        if constexpr (KC > 1)
          if (rows == 1) stage1(std::integral_constant<int, 1>{}, Lv, tb, Ln, tbn);
        if constexpr (KC > 2)
          if (rows == 2) stage1(std::integral_constant<int, 2>{}, Lv, tb, Ln, tbn);
        if constexpr (KC > 3)
          if (rows == 3) stage1(std::integral_constant<int, 3>{}, Lv, tb, Ln, tbn);
        if constexpr (KC > 4)
          if (rows == 4) stage1(std::integral_constant<int, 4>{}, Lv, tb, Ln, tbn);
      } else {
        load_l(Ln, tbn, 0, ac);
      }
      if (tiles) load_t(2 * ch0, bc);
      AFQMC_KEEP_AHEAD();
      __syncthreads();  // the shared buffer's last readers are done
      int ln = lane;
      asm volatile("" : "+v"(ln));
      double* dy = sY + 4 * v + (ln & 3) + (ln >> 4) * 16 + h * KC * 256;
      const int wf = ((ln >> 2) & 3) * SYS, wr = (ln & 12) * 16;
#pragma unroll
      for (int p = 0; p < PL; ++p)
#pragma unroll
        for (int q = 0; q < KC; ++q)
          if (tb + q < KT) {
            const int m0 = 16 * q;
            double* d = dy + p * NG * SYS;
#pragma unroll
            for (int ct = 0; ct < NF; ++ct)
#pragma unroll
              for (int r = 0; r < 4; ++r)
                d[wf + 4 * ct * SYS + (m0 + 4 * r) * 16] = y[p][q][ct][r];
#pragma unroll
            for (int ct = 0; ct < NR; ++ct)
              d[wr + (4 * NF + ct) * SYS + m0 * 16] = yr[p][q][ct];
          }
      __syncthreads();
      if (tiles) stage2(ch0);
    }
    Lv = Lnext;
    double* d = sD + (grp & 1) * NW * 32;
    if (tiles) put_d(d);
    if constexpr (NG > 1) __syncthreads();  // every Y of the last chunk is read
    if (tiles) put_f();
    __syncthreads();
    if (tiles) get_f(GV * grp + (c >> 2) < G);
    if (wi == 0) {  // lane 4 v + i < 16: vb of vector v
      double x = 0.0, z = 0.0;
#pragma unroll
      for (int q = 0; q < NWA; ++q) {
        const double2 e = *reinterpret_cast<const double2*>(d + ((wave + q) * 16 + c) * 2);
        x += e.x;
        z += e.y;
      }
      x += dpp_f64<0xB1>(x);
      z += dpp_f64<0xB1>(z);
      x += dpp_f64<0x4E>(x);
      z += dpp_f64<0x4E>(z);
      const int vec = GV * grp + (c >> 2);
      if (lane < 16 && (c & 3) == 0 && active[PP > 1 ? pw : 0]) {
        if (vec < G) {
          *reinterpret_cast<double2*>(vb + ((size_t)(s0 + pw) * G + vec) * 2) = make_double2(x, z);
          e_re += 0.5 * (x * x - z * z);
          e_im += x * z;
        } else if (vec == G) {
          e_re += x;
          e_im += z;
        }
      }
    }
    if (grp + 1 == bend) {
      rng.add(e_re, e_im, epart, wi, NWP, n_samples, s0 + pw, active[PP > 1 ? pw : 0], true);
      e_re = e_im = 0.0;
      bend = rng.end();
    }
  }
  const double2 e_wave = rng.total();  // with all lanes active
  if (lane == 0) *reinterpret_cast<double2*>(sE + wave * 2) = e_wave;
  __syncthreads();
  if (!rng.split && wi == 0 && lane == 0 && active[PP > 1 ? pw : 0]) {
    double xr = 0.0, xi = 0.0;
    for (int q = 0; q < NWP; ++q) {
      xr += sE[(wave + q) * 2];
      xi += sE[(wave + q) * 2 + 1];
    }
    epart[2 * (size_t)(s0 + pw)] = xr;
    epart[2 * (size_t)(s0 + pw) + 1] = xi;
  }
}

template <int NG, int KC, int NW, int PP, bool CT = false>
hipError_t launch_q(const afqmc_ctx_s* c, int n, int nsplit, const double* phiT,
                    const double* theta, const double* logov, double* vb, double* epart) {
  typedef qshape<NG, KC, NW, PP, CT> Q;
  const size_t lds = sizeof(double) * ((size_t)Q::SBUF + (size_t)Q::PL * c->MT * 4 * NG +
                                       2 * NW * 32 + NW * 2);
  auto kern = k_contract_q<NG, KC, NW, PP, CT>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((n + PP - 1) / PP, nsplit), dim3(64 * NW), lds, c->stream, n, c->M,
                     c->N, c->G, c->MT / 16, c->d_Lpad, phiT, theta, logov, vb, epart);
  return hipGetLastError();
}

}  // namespace

// Two paths per workgroup: for N <= 16, and for N <= 20 while two such workgroups fit a
// CU's LDS (M <= 112).  M = 72, N = 18: 4.04 ms with one path, 3.73 with two; M = 150,
// N = 20: 16.0 and 16.4.
static int paths_per_group(int NG, int KT) { return NG <= 4 || (NG == 5 && KT <= 7) ? 2 : 1; }

// Ranges of g that the paths' workgroups are split into (slots: what the CUs hold at once, by
// registers 4 a CU up to N = 12, 2 up to N = 28, 1 of eight wavefronts past that; at least
// four groups of vectors to a range).  600 paths of M = 142, N = 35 fill 2.3 rounds of 256:
// 24.7 ms in one range, 17.9 in several.
contract_plan contract_q_plan(const afqmc_ctx_s* c, int nw) {
  const int NG = (c->N + 3) / 4, pp = c->ctrial ? 1 : paths_per_group(NG, c->MT / 16);
  // wavefronts a path, as dispatched below: eight a workgroup past N = 28 (complex N = 24)
  const int nwp = (NG > (c->ctrial ? 6 : 7) ? 8 : 4) / pp;
  return plan_splits(((long)nw * c->P + pp - 1) / pp, NG <= 3 ? 1024 : NG <= 7 ? 512 : 256,
                     (c->G + GV) / GV, 4, nwp);
}

hipError_t launch_contract_q(const afqmc_ctx_s* c, int nw, int nsplit, const double* phiT,
                             const double* theta, const double* logov, double* vb, double* epart) {
  if (nw <= 0) return hipSuccess;
  const int n = nw * c->P, KT = c->MT / 16;
  // rows of Y^T per wavefront and chunk, wavefronts, paths: the fastest spill-free choice of
  // KC = 1 .. 5, NW = 4, 8, PP = 1, 2 at the sizes above (next best 1 to 8 % slower)
#define AFQMC_Q(KK, WW, PP) \
  return launch_q<NG, KK, WW, PP>(c, n, nsplit, phiT, theta, logov, vb, epart)
#define AFQMC_QN(NN) case NN: { constexpr int NG = NN;
  if (c->ctrial) {
#define AFQMC_QC(NN, KK, WW) \
  case NN: return launch_q<NN, KK, WW, 1, true>(c, n, nsplit, phiT, theta, logov, vb, epart);
    switch ((c->N + 3) / 4) {
      AFQMC_QC(1, 2, 4) AFQMC_QC(2, 2, 4) AFQMC_QC(3, 2, 4) AFQMC_QC(4, 2, 4)
      AFQMC_QC(5, 2, 4) AFQMC_QC(6, 2, 4) AFQMC_QC(7, 1, 8) AFQMC_QC(8, 1, 8)
#undef AFQMC_QC
      default: return hipErrorInvalidValue;
    }
  }
  switch ((c->N + 3) / 4) {
    AFQMC_QN(1) AFQMC_Q(2, 4, 2); }
    AFQMC_QN(2) AFQMC_Q(2, 4, 2); }
    AFQMC_QN(3) AFQMC_Q(2, 4, 2); }
    AFQMC_QN(4) AFQMC_Q(2, 4, 2); }
    AFQMC_QN(5) if (paths_per_group(NG, KT) == 2) AFQMC_Q(2, 4, 2); AFQMC_Q(3, 4, 1); }
    AFQMC_QN(6) AFQMC_Q(3, 4, 1); }
    AFQMC_QN(7) AFQMC_Q(2, 4, 1); }
    AFQMC_QN(8) AFQMC_Q(2, 8, 1); }
    AFQMC_QN(9) AFQMC_Q(3, 8, 1); }
    AFQMC_QN(10) AFQMC_Q(2, 8, 1); }
    default: return hipErrorInvalidValue;
  }
#undef AFQMC_QN
#undef AFQMC_Q
}
