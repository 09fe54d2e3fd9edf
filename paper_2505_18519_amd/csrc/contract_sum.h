// The order in which the contraction kernels sum E_p over the Cholesky vectors.  The
// vectors fall into blocks whose bounds depend on their number alone.  In each of the
// wavefronts that share a path, each row of 16 lanes adds a block over its lanes, then the
// blocks in order; the rows and the wavefronts are added last.  A call may therefore give
// whole blocks to any number of workgroups (ranges of blocks, gridDim.y of them) and E_p
// keeps its bits: which number is fastest depends on how many paths the call has, and a
// path's results must not.
#pragma once

#include <algorithm>

#include "dev_common.h"

// Blocks: up to 48, which 1, 2, 3, 4, 6, 8, 12 and 16 workgroups share evenly (by the count of
// granules, 16 blocks leave one call in four 5 % or more behind an even split, 48 one in
// twenty).  The sums at their ends cost whole-chip calls up to 1 % at M >= 64, up to 3 % at
// M = 24.
constexpr int kSumBlocks = 48;
constexpr int kMaxWaves = 8;  // wavefronts that share a path, at most

// granules: the vectors in the steps that a kernel takes them in
struct vec_blocks {
  int granules, n, most;
  __host__ __device__ vec_blocks(int g, int m) : granules(g), n(g < m ? g : m), most(m) {}
  __host__ __device__ int begin(int b) const { return granules < most ? b : b * granules / most; }
};

// How a call splits: nsplit workgroups along the vectors.  More than one leave each
// wavefront's block sums in memory for k_combine, [blocks][waves][paths][rows] complex.
struct contract_plan {
  int nsplit = 1, blocks = 1, waves = 1;
  size_t part_bytes(size_t paths) const { return (size_t)blocks * waves * paths * 64; }
};

// The fewest workgroups along the vectors (up to 16, each at least `least` granules) within
// 4 % of the shortest time: rounds of the `slots` workgroups that the chip holds times the
// longest range (the mean range where the blocks are so many that ranges differ little).
inline contract_plan plan_splits(long units, long slots, int granules, int least, int waves,
                                 int most = kSumBlocks) {
  const vec_blocks b(granules, most);
  contract_plan p;
  p.blocks = b.n;
  p.waves = waves;
  double best = 1e300;
  for (int k = 1; k <= 16 && k <= b.n && (k == 1 || k * least <= granules); ++k) {
    double len = (double)granules / k;
    if (b.n < kSumBlocks)
      for (int i = 0; i < k; ++i)
        len = std::max(len, (double)(b.begin((i + 1) * b.n / k) - b.begin(i * b.n / k)));
    const double t = (double)((units * k + slots - 1) / slots) * len;
    if (t < 0.96 * best) {
      best = t;
      p.nsplit = k;
    }
  }
  return p;
}

// The blocks of range y of ny, taken one after another; each row of 16 lanes keeps a running
// total of its sums, real part in lane 0 and imaginary part in lane 1.
struct block_range {
  vec_blocks b;
  int cur, last;  // the block in progress; the range's end
  bool split;     // more than one range
  double tot = 0.0;
  __device__ block_range(int granules, int y, int ny, int most = kSumBlocks)
      : b(granules, most), cur(y * b.n / ny), last((y + 1) * b.n / ny), split(ny > 1) {}
  __device__ int begin() const { return b.begin(cur); }  // granules of the block in progress
  __device__ int end() const { return b.begin(cur + 1); }
  // its lanes' sums (all 64 lanes active), to the totals or to the block sums in memory (write:
  // the path is there; zeros for one that is not live)
  __device__ __forceinline__ void add(double re, double im, double* part, int wave, int waves,
                                      int paths, int path, bool write, bool live) {
    const int lane = threadIdx.x & 63;
    const bool odd = lane & 1;
    double x = odd ? im : re;  // even lanes take the real parts of both, odd the imaginary
    x += dpp_f64<0xB1>(odd ? re : im);
    x += dpp_f64<0x4E>(x);
    x += dpp_f64<0x124>(x);  // rotated by 4 and by 8 within the row
    x += dpp_f64<0x128>(x);
    if (!split)
      tot += x;
    else if (write && (lane & 15) < 2)
      part[((((size_t)cur * waves + wave) * paths + path) * 4 + (lane >> 4)) * 2 + (lane & 1)] =
          live ? x : 0.0;
    ++cur;
  }
  // the totals of the four rows, added (all 64 lanes active)
  __device__ double2 total() const {
    return make_double2((readlane_f64(tot, 0) + readlane_f64(tot, 16)) +
                            (readlane_f64(tot, 32) + readlane_f64(tot, 48)),
                        (readlane_f64(tot, 1) + readlane_f64(tot, 17)) +
                            (readlane_f64(tot, 33) + readlane_f64(tot, 49)));
  }
};

// zeros in place of the block sums of a path without overlap
__device__ __forceinline__ void zero_blocks(const block_range& r, double* part, int wave, int waves,
                                            int paths, int path, int lane) {
  for (int q = 4 * r.cur + lane; q < 4 * r.last; q += 64)
    *reinterpret_cast<double2*>(
        part + ((((size_t)(q >> 2) * waves + wave) * paths + path) * 4 + (q & 3)) * 2) =
        make_double2(0.0, 0.0);
}
