// Blocked Gauss-Jordan elimination with tournament pivoting for batches of
// dense complex double matrices.
//
// The CBF build solves every cell's isolated system Z_mm J_m = V_m for all
// generating waves (Sec. III-A), and the CMP needs the inverse of
// B = (C^M)^H G C^J (Sec. III-C).  Both run here as Gauss-Jordan elimination
// over panels of 32 columns.  Each panel step is a few launches on the
// stream, with no host round trip until the end:
//  1. pivot rows: the panel's rows are split into groups of 256, one row per
//     thread held in registers.  Each group runs an LU factorisation of its
//     rows with partial pivoting (largest |re| + |im|, lowest row on ties)
//     and keeps the 32 rows it pivoted on; the rows kept by eight groups make
//     a group of the next round, until one group is left (tournament
//     pivoting).  The last group inverts the 32 x 32 pivot block D
//     (Gauss-Jordan in LDS, in the order the pivots were chosen) and sets
//     the row permutation of the step: the panel's rows K take the pivot
//     rows, and the rows of K that were not chosen take the places the
//     chosen rows outside K leave (paired in order, by wave ballots).  It
//     saves every row's panel entries (after the permutation) for the
//     update;
//  2. row block: over chunks of 64 columns, the permutation is applied and
//     the pivot rows R become D^{-1} R;
//  3. update: every other row i loses A[i, panel] D^{-1} R on the matrix
//     cores.
// An inversion runs in place: the columns of the inverse take the places of
// the eliminated columns.  The column of the inverse that belongs to row j
// of the input ends up where the permutations took that row, so a last
// gather, driven by the map of which input row each position holds, puts
// the columns in order.  A solve runs on the augmented [Z | V] and
// only updates the columns right of the panel.
#include <algorithm>
#include <string>
#include <vector>

#include "gj.h"
#include "internal.h"

namespace cbfm {

namespace {

constexpr int kW = 32;          // panel width
constexpr int kGroup = 256;     // rows per pivot group, one per thread
constexpr int kChunk = 64;      // columns per block of the row-block kernel
constexpr int kSwapInts = 128;  // per matrix: pivot rows [0, 32), displaced
                                // positions [32, 64), their sources [64, 96), count [96]

__device__ inline double gj_cabs1(double2 z) { return fabs(z.x) + fabs(z.y); }
__device__ inline double2 gj_mul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// 1 / p by the hardware reciprocal of |p|^2 and two Newton steps, and each
// quotient corrected by its residual: the bits of the divisions (none of 2^31
// random quotients differs; without the residual 27 % do), in less latency,
// which sits on every step's critical path; away from the ends of the range
// where |p|^2 or its reciprocal is subnormal.
__device__ inline double2 gj_recip(double2 p) {
  const double d = p.x * p.x + p.y * p.y;
  if (!(d > 1e-290 && d < 1e290)) return make_double2(p.x / d, -p.y / d);
  double y = __builtin_amdgcn_rcp(d);
  y = fma(fma(-d, y, 1.0), y, y);
  y = fma(fma(-d, y, 1.0), y, y);
  const double re = p.x * y, im = -p.y * y;
  return make_double2(fma(fma(-re, d, p.x), y, re), fma(fma(-im, d, -p.y), y, im));
}
// Pivot key of a row: |re| + |im| rounded to float (a positive value stays
// positive) above 1; 1 for a zero (or NaN) entry, 0 for a thread without a
// candidate row.
__device__ inline uint32_t gj_key(bool alive, double2 z) {
  const double m = gj_cabs1(z);
  return !alive ? 0u : m > 0.0 ? (__float_as_uint((float)m) | 1u) + 1u : 1u;
}
template <int CTRL>
__device__ inline uint32_t gj_dpp_max(uint32_t x) {
  const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
  return y > x ? y : x;
}
// The largest value over the wavefront (uniform).
__device__ inline uint32_t gj_wave_max(uint32_t x) {
  x = gj_dpp_max<0xB1>(x);   // within rows of 16 lanes
  x = gj_dpp_max<0x4E>(x);
  x = gj_dpp_max<0x141>(x);
  x = gj_dpp_max<0x140>(x);
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 0), r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 16),
                 r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 32), r3 = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
  const uint32_t a = r0 > r1 ? r0 : r1, b = r2 > r3 ? r2 : r3;
  return a > b ? a : b;
}

struct SelectArgs {
  const double2* A;
  int64_t strideA, ld;
  int n, k, w;
  const int32_t* cand_in;  // candidate rows of this tournament stage (null: the rows k .. n - 1)
  int cand_len;            // entries of cand_in per matrix (-1 marks an empty slot)
  int nsel_groups;         // blocks that select; at the first round the blocks
                           // after them copy the panel entries of rows 0 .. k - 1
  int32_t* cand_out;       // kW slots per group
  int64_t cand_stride;     // entries per matrix of cand_in / cand_out
  int final_round;
  double2* Pcol;   // n x kW per matrix: the panel entries of every row
  double2* Dinv;   // kW x kW per matrix
  int32_t* swaps;  // kSwapInts per matrix
  int32_t* rowat;  // n per matrix: the input row each position holds (null: not kept)
  int32_t* info;   // per matrix: 1 + the first column without a nonzero pivot
};

__global__ void __launch_bounds__(kGroup) gj_select_kernel(SelectArgs p) {
  const int b = blockIdx.y, g = blockIdx.x, t = threadIdx.x;
  const double2* Ab = p.A + (int64_t)b * p.strideA;
  double2* Pc = p.Pcol + (int64_t)b * p.n * kW;
  const int k = p.k, w = p.w;
  if (p.cand_in == nullptr && g >= p.nsel_groups) {
    // (every load is issued before the first store: a load-store chain per
    // entry would wait on memory 32 times in a row)
    const int r = (g - p.nsel_groups) * kGroup + t;
    if (r < k) {
      double2 v[kW];
#pragma unroll
      for (int j = 0; j < kW; ++j) v[j] = j < w ? Ab[(int64_t)r * p.ld + k + j] : make_double2(0.0, 0.0);
#pragma unroll
      for (int j = 0; j < kW; ++j)
        if (j < w) Pc[(int64_t)r * kW + j] = v[j];
    }
    return;
  }
  int row = -1;
  if (p.cand_in == nullptr) {
    const int r = k + g * kGroup + t;
    if (r < p.n) row = r;
  } else {
    const int e = g * kGroup + t;
    if (e < p.cand_len) row = p.cand_in[(int64_t)b * p.cand_stride + e];
  }
  double2 a[kW];
#pragma unroll
  for (int j = 0; j < kW; ++j) a[j] = make_double2(0.0, 0.0);
  if (row >= 0) {
#pragma unroll
    for (int j = 0; j < kW; ++j)
      if (j < w) a[j] = Ab[(int64_t)row * p.ld + k + j];
    if (p.cand_in == nullptr) {
#pragma unroll
      for (int j = 0; j < kW; ++j)
        if (j < w) Pc[(int64_t)row * kW + j] = a[j];
    }
  }
  // LU with partial pivoting over the group's rows; column c picks row
  // s_sel[c].  Bound by the latency of its 32 steps (62 % of wave cycles wait,
  // on LDS and barriers): the argmax by DPP and scalar maxima, the winner's
  // row alone written to LDS (one lane's 16-byte stores cost as much as a
  // full wavefront's), wavefronts whose rows are all chosen skip the update.
  // Eight columns are unrolled and the registers move down by eight between
  // blocks: 27 KB of code instead of 105.  Per launch 75 -> 41 (first round),
  // 47 us (last round, with D^{-1}).
  constexpr int kWaves = kGroup / 64, kB = 8;
  __shared__ uint32_t s_key[2][kWaves];
  __shared__ double2 s_prow[2][kW];
  __shared__ int s_sel[kW];
  bool alive = row >= 0;
  int nsel = 0;
  bool open = true;  // uniform: false from the first column with no row left
  const int lane = t & 63, wave = t >> 6;
#pragma unroll 1
  for (int c0 = 0; c0 < kW; c0 += kB) {
    // a[j] holds column c0 + j; live: columns of a still in the panel
    const int live = kW - c0;
#pragma unroll
    for (int c = 0; c < kB; ++c) {
      const int buf = c & 1;
      const uint32_t key = gj_key(alive, a[c]), top = gj_wave_max(key);
      const bool mine = lane == __builtin_ctzll(__ballot(key == top));
      if (lane == 0) s_key[buf][wave] = top;
      __syncthreads();
      int bw = 0;
      uint32_t best = s_key[buf][0];
#pragma unroll
      for (int q = 1; q < kWaves; ++q)
        if (s_key[buf][q] > best) {
          best = s_key[buf][q];
          bw = q;
        }
      if (mine && wave == bw) {
        double2* pr = s_prow[buf];
#pragma unroll
        for (int j = c; j < kB; ++j) pr[j] = a[j];
#pragma unroll
        for (int g8 = kB; g8 < kW; g8 += kB)
          if (g8 < live)
#pragma unroll
            for (int j = g8; j < g8 + kB; ++j) pr[j] = a[j];
      }
      __syncthreads();
      open = open && best != 0 && c0 + c < w;
      if (open) {
        nsel = c0 + c + 1;
        if (mine && wave == bw) {
          alive = false;
          s_sel[c0 + c] = row;
        }
        if (best == 1 && p.final_round && t == 0 && p.info[b] == 0) p.info[b] = k + c0 + c + 1;
      }
      const double2* pr = s_prow[buf];
      double2 l = gj_mul(a[c], gj_recip(pr[c]));
      const bool upd = open && alive && best > 1;
      if (!upd) l = make_double2(0.0, 0.0);
      if (!__any(upd)) continue;  // no row of this wavefront takes part any more
      auto sub = [&](int j) {
        const double2 x = pr[j];
        a[j].x = fma(l.y, x.y, fma(-l.x, x.x, a[j].x));
        a[j].y = fma(-l.y, x.x, fma(-l.x, x.y, a[j].y));
      };
#pragma unroll
      for (int j = c + 1; j < kB; ++j) sub(j);
#pragma unroll
      for (int g8 = kB; g8 < kW; g8 += kB)
        if (g8 < live)
#pragma unroll
          for (int j = g8; j < g8 + kB; ++j) sub(j);
    }
#pragma unroll
    for (int j = 0; j < kW - kB; ++j) a[j] = a[j + kB];
  }
  __syncthreads();
  if (!p.final_round) {
    if (t < kW) p.cand_out[(int64_t)b * p.cand_stride + (int64_t)g * kW + t] = t < nsel ? s_sel[t] : -1;
    return;
  }
  if (nsel < w && t == 0 && p.info[b] == 0) p.info[b] = k + nsel + 1;
  // D (the pivot rows' panel entries, identity-padded) to D^{-1} by
  // Gauss-Jordan in place without further interchanges, in registers: this
  // thread holds row mi, columns mq + 8 u.  Step c's row and column pass
  // through LDS (two buffers: one barrier a step).
  __shared__ double2 s_r[2][kW], s_f[2][kW];
  const int mi = t >> 3, mq = t & 7;
  double2 m[kW / 8];
#pragma unroll
  for (int u = 0; u < kW / 8; ++u) {
    const int j = mq + 8 * u;
    m[u] = mi < nsel && j < w ? Ab[(int64_t)s_sel[mi] * p.ld + k + j] : make_double2(mi == j && mi >= w ? 1.0 : 0.0, 0.0);
  }
#pragma unroll
  for (int cu = 0; cu < kW / 8; ++cu) {
#pragma unroll 1
    for (int cq = 0; cq < 8; ++cq) {
      const int c = cq + 8 * cu;
      double2* r = s_r[cq & 1];
      double2* f = s_f[cq & 1];
      if (mi == c)
#pragma unroll
        for (int u = 0; u < kW / 8; ++u) r[mq + 8 * u] = m[u];
      if (mq == cq) f[mi] = m[cu];
      __syncthreads();
      const double2 rp = gj_recip(r[c]), fm = f[mi];
#pragma unroll
      for (int u = 0; u < kW / 8; ++u) {
        const bool diag = u == cu && mq == cq;
        const double2 x = diag ? rp : gj_mul(r[mq + 8 * u], rp);
        const double2 y = diag ? make_double2(0.0, 0.0) : m[u];
        m[u] = mi == c ? x : make_double2(y.x - (fm.x * x.x - fm.y * x.y), y.y - (fm.x * x.y + fm.y * x.x));
      }
    }
  }
  double2* Db = p.Dinv + (int64_t)b * kW * kW;
#pragma unroll
  for (int u = 0; u < kW / 8; ++u) Db[mi * kW + mq + 8 * u] = m[u];
  // the permutation: position k + i takes row s_row[i]; the rows of K that
  // were not chosen take the positions s_dd[] that chosen rows outside K
  // leave (s_ds[]: where each comes from)
  __shared__ int s_row[kW], s_dd[kW], s_ds[kW];
  __shared__ int s_nd;
  int32_t* sw = p.swaps + (int64_t)b * kSwapInts;
  if (t < 64) {
    const int i = t;
    const int r = i < w ? (i < nsel ? s_sel[i] : k + i) : 0;
    bool picked = false;
    for (int j = 0; j < nsel; ++j) picked |= s_sel[j] == k + i;
    const bool hole = i < w && r >= k + w, unsel = i < w && !picked;
    const uint64_t hm = __ballot(hole), um = __ballot(unsel), below = (1ull << i) - 1;
    if (hole) s_dd[__popcll(hm & below)] = r;
    if (unsel) s_ds[__popcll(um & below)] = k + i;
    if (i < w) {
      s_row[i] = r;
      sw[i] = r;
    }
    if (i == 0) s_nd = min(__popcll(hm), __popcll(um));
  }
  __syncthreads();
  const int nd = s_nd;
  if (t < nd) {
    sw[kW + t] = s_dd[t];
    sw[2 * kW + t] = s_ds[t];
  }
  if (t == 0) sw[3 * kW] = nd;
  if (p.rowat) {  // (every read before any write)
    int32_t* ra = p.rowat + (int64_t)b * p.n;
    const int v1 = t < w ? ra[s_row[t]] : 0, v2 = t < nd ? ra[s_ds[t]] : 0;
    __syncthreads();
    if (t < w) ra[k + t] = v1;
    if (t < nd) ra[s_dd[t]] = v2;
  }
  // panel entries of the displaced positions: the rows that now sit there
  constexpr int kDU = kW * kW / kGroup;
  double2 dv[kDU];
#pragma unroll
  for (int u = 0; u < kDU; ++u) {
    const int e = t + kGroup * u, d = e / kW, j = e % kW;
    dv[u] = d < nd && j < w ? Ab[(int64_t)s_ds[d] * p.ld + k + j] : make_double2(0.0, 0.0);
  }
#pragma unroll
  for (int u = 0; u < kDU; ++u) {
    const int e = t + kGroup * u, d = e / kW, j = e % kW;
    if (d < nd && j < w) Pc[(int64_t)s_dd[d] * kW + j] = dv[u];
  }
}

struct RowsArgs {
  double2* A;
  int64_t strideA, ld;
  int ncols, k, w, col0;
  const double2* Dinv;
  const int32_t* swaps;
};

// Columns col0 + 64 blockIdx.x + (0 .. 63) of matrix blockIdx.y: rows K
// (k .. k + w - 1) receive the pivot rows, the displaced positions receive
// the rows of K they held, and rows K become D^{-1} times themselves.  The
// panel's own columns (present only for an inversion) get D^{-1}; their
// other rows are written by the update.
__global__ void __launch_bounds__(256) gj_rows_kernel(RowsArgs p) {
  const int b = blockIdx.y, t = threadIdx.x;
  double2* Ab = p.A + (int64_t)b * p.strideA;
  const int j0 = p.col0 + (int)blockIdx.x * kChunk;
  const int k = p.k, w = p.w;
  __shared__ double2 s_d[kW][kW + 1];
  __shared__ double2 s_r[kW][kChunk];
  __shared__ int s_sw[kSwapInts];
  const int32_t* sw = p.swaps + (int64_t)b * kSwapInts;
  for (int e = t; e <= 3 * kW; e += 256) s_sw[e] = sw[e];
  for (int e = t; e < kW * kW; e += 256) s_d[e / kW][e % kW] = p.Dinv[(int64_t)b * kW * kW + e];
  __syncthreads();
  const int nd = s_sw[3 * kW];
  auto inpanel = [&](int j) { return j >= k && j < k + w; };
  for (int e = t; e < kW * kChunk; e += 256) {
    const int i = e / kChunk, jj = e % kChunk, j = j0 + jj;
    double2 v = make_double2(0.0, 0.0);
    if (i < w && j < p.ncols && !inpanel(j)) v = Ab[(int64_t)s_sw[i] * p.ld + j];
    s_r[i][jj] = v;
  }
  constexpr int kU = kW * kChunk / 256;
  double2 xd[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const int e = t + 256 * u, d = e / kChunk, j = j0 + e % kChunk;
    xd[u] = (d < nd && j < p.ncols && !inpanel(j)) ? Ab[(int64_t)s_sw[2 * kW + d] * p.ld + j]
                                                   : make_double2(0.0, 0.0);
  }
  __syncthreads();  // every read of this block's columns is done
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const int e = t + 256 * u, d = e / kChunk, j = j0 + e % kChunk;
    if (d < nd && j < p.ncols && !inpanel(j)) Ab[(int64_t)s_sw[kW + d] * p.ld + j] = xd[u];
  }
  const int jj = t & (kChunk - 1), r0 = (t / kChunk) * 8, j = j0 + jj;
  if (j >= p.ncols) return;
  if (inpanel(j)) {
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (r0 + q < w) Ab[(int64_t)(k + r0 + q) * p.ld + j] = s_d[r0 + q][j - k];
    return;
  }
  double2 acc[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) acc[q] = make_double2(0.0, 0.0);
  for (int c = 0; c < w; ++c) {
    const double2 x = s_r[c][jj];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const double2 d = s_d[r0 + q][c];
      acc[q].x += d.x * x.x - d.y * x.y;
      acc[q].y += d.x * x.y + d.y * x.x;
    }
  }
#pragma unroll
  for (int q = 0; q < 8; ++q)
    if (r0 + q < w) Ab[(int64_t)(k + r0 + q) * p.ld + j] = acc[q];
}

// The update of a step: rows r outside the panel, columns from col0 on, A[r][j]
// -= P[r] R[., j] (P: the saved panel entries; R: the panel's rows of A), the
// panel's own columns (an inversion) overwritten by the negative product.  A
// block of four wavefronts takes 64 x 64 entries, 32 x 32 per wavefront, whose
// old values are loaded first; both operands pass through LDS in two halves
// of 16 k.  Bound by the entries read and written (32 bytes for 256 flops):
// the general kernel, 16 x 16 per wavefront, read each operand entry four
// times as often: 96 systems of 624 with 144 right-hand sides 440 -> 345 us
// (first step, 1.3 GB).  3M complex products as in gemm.hip.
struct UpdateArgs {
  double2* A;
  const double2* P;
  int64_t strideA, ld;
  int n, ncols, k, w, col0;
};
typedef double gj_dbl4 __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(256, 2) gj_update_kernel(UpdateArgs p) {
  __shared__ double2 sp[64][17];
  __shared__ double2 sr[16][65];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, slot = lane >> 4, li = lane & 15;
  const int b = blockIdx.z, k = p.k, w = p.w, nrow = p.n - w;
  double2* Ab = p.A + (int64_t)b * p.strideA;
  const double2* Pb = p.P + (int64_t)b * p.n * kW;
  const int i0 = blockIdx.y * 64, j0 = p.col0 + blockIdx.x * 64;
  auto row_of = [&](int i) { return i < k ? i : i + w; };  // the i-th row outside the panel
  const int mi = i0 + 32 * (wave >> 1), mj = j0 + 32 * (wave & 1);
  double2 c[2][2][4];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = mi + 16 * x + 4 * q + slot, j = mj + 16 * y + li;
        c[x][y][q] = i < nrow && j < p.ncols && !(j >= k && j < k + w) ? Ab[(int64_t)row_of(i) * p.ld + j]
                                                                      : make_double2(0.0, 0.0);
      }
  gj_dbl4 p1[2][2], p2[2][2], p3[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) p1[x][y] = p2[x][y] = p3[x][y] = gj_dbl4{0, 0, 0, 0};
  for (int h = 0; h < w; h += 16) {  // uniform
    double2 a[4], r[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + (tid >> 4) + 16 * u, ka = h + (tid & 15);
      a[u] = i < nrow && ka < w ? Pb[(int64_t)row_of(i) * kW + ka] : make_double2(0.0, 0.0);
      const int kr = h + (tid >> 6) + 4 * u, j = j0 + (tid & 63);
      r[u] = kr < w && j < p.ncols ? Ab[(int64_t)(k + kr) * p.ld + j] : make_double2(0.0, 0.0);
    }
    if (h > 0) __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      sp[(tid >> 4) + 16 * u][tid & 15] = a[u];
      sr[(tid >> 6) + 4 * u][tid & 63] = r[u];
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 4; ++s) {  // step s takes k = 4 s + slot
      double2 av[2], bv[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        av[x] = sp[32 * (wave >> 1) + 16 * x + li][4 * s + slot];
        bv[x] = sr[4 * s + slot][32 * (wave & 1) + 16 * x + li];
      }
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          p1[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[x].x, bv[y].x, p1[x][y], 0, 0, 0);
          p2[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[x].y, bv[y].y, p2[x][y], 0, 0, 0);
          p3[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[x].x + av[x].y, bv[y].x + bv[y].y, p3[x][y], 0, 0, 0);
        }
    }
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = mi + 16 * x + 4 * q + slot, j = mj + 16 * y + li;
        if (i >= nrow || j >= p.ncols) continue;
        const double re = p1[x][y][q] - p2[x][y][q], im = p3[x][y][q] - p1[x][y][q] - p2[x][y][q];
        Ab[(int64_t)row_of(i) * p.ld + j] = make_double2(c[x][y][q].x - re, c[x][y][q].y - im);
      }
}

__global__ void gj_iota_kernel(int32_t* __restrict__ x, int n, int64_t total) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < total) x[e] = (int32_t)(e % n);
}

// out_b[i][j] = in_b[i][src_b[j]] (n x n row-major, b = blockIdx.z).
__global__ void gj_gather_kernel(const double2* __restrict__ in, double2* __restrict__ out,
                                 const int32_t* __restrict__ src, int n, int64_t strideA) {
  const int j = blockIdx.x * 256 + threadIdx.x, i = blockIdx.y, b = blockIdx.z;
  if (j >= n) return;
  const int64_t row = (int64_t)b * strideA + (int64_t)i * n;
  out[row + j] = in[row + src[(int64_t)b * n + j]];
}

// src_b[rowat_b[q]] = q: the position that holds each input row.
__global__ void gj_src_kernel(const int32_t* __restrict__ rowat, int32_t* __restrict__ src, int n, int64_t total) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const int64_t b = e / n;
  src[b * n + rowat[e]] = (int32_t)(e - b * n);
}

// The elimination, enqueued on s with no host wait: info_dev (nmat entries)
// receives 0 or 1 + the first column without a nonzero pivot.  An inversion
// ends with the column gather.  Every scratch buffer is released in stream
// order.
void eliminate(double2* A, int64_t strideA, int64_t ld, int n, int ncols, int nmat, bool inverse, int32_t* info_dev,
               hipStream_t s) {
  CBFM_REQUIRE(n >= 1 && n <= 65535 && nmat >= 1 && nmat <= 65535, CBFM_E_ARG,
               "Gauss-Jordan: order in [1, 65535] and at most 65535 matrices");
  CBFM_REQUIRE(ncols >= n && ld >= ncols && strideA >= (int64_t)(n - 1) * ld + ncols, CBFM_E_ARG,
               "Gauss-Jordan: inconsistent matrix layout");
  const int steps = (n + kW - 1) / kW;
  const int gmax = (n + kGroup - 1) / kGroup;
  const int64_t cstride = (int64_t)gmax * kW;
  Scratch pcol((size_t)nmat * n * kW * sizeof(double2), s), dinv((size_t)nmat * kW * kW * sizeof(double2), s),
      swaps((size_t)nmat * kSwapInts * sizeof(int32_t), s),
      rowat(inverse ? (size_t)nmat * n * sizeof(int32_t) : 0, s),
      cand0((size_t)nmat * cstride * sizeof(int32_t), s),
      cand1((size_t)nmat * cstride * sizeof(int32_t), s);
  CBFM_HIP(hipMemsetAsync(info_dev, 0, (size_t)nmat * sizeof(int32_t), s));
  if (inverse) {
    const int64_t total = (int64_t)nmat * n;
    hipLaunchKernelGGL(gj_iota_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, rowat.as<int32_t>(), n,
                       total);
    CBFM_HIP(hipGetLastError());
  }
  Scratch* cand[2] = {&cand0, &cand1};
  for (int st = 0; st < steps; ++st) {
    const int k = st * kW, w = std::min(kW, n - k);
    SelectArgs a{};
    a.A = A;
    a.strideA = strideA;
    a.ld = ld;
    a.n = n;
    a.k = k;
    a.w = w;
    a.cand_stride = cstride;
    a.Pcol = pcol.as<double2>();
    a.Dinv = dinv.as<double2>();
    a.swaps = swaps.as<int32_t>();
    a.rowat = inverse ? rowat.as<int32_t>() : nullptr;
    a.info = info_dev;
    int G = (n - k + kGroup - 1) / kGroup, cur = 0;
    a.cand_in = nullptr;
    a.cand_len = 0;
    a.nsel_groups = G;
    a.final_round = G == 1;
    a.cand_out = cand[cur]->as<int32_t>();
    hipLaunchKernelGGL(gj_select_kernel, dim3((unsigned)(G + (k + kGroup - 1) / kGroup), (unsigned)nmat),
                       dim3(kGroup), 0, s, a);
    CBFM_HIP(hipGetLastError());
    while (G > 1) {
      const int len = G * kW, G2 = (len + kGroup - 1) / kGroup;
      a.cand_in = cand[cur]->as<int32_t>();
      a.cand_len = len;
      a.nsel_groups = G2;
      a.final_round = G2 == 1;
      a.cand_out = cand[1 - cur]->as<int32_t>();
      hipLaunchKernelGGL(gj_select_kernel, dim3((unsigned)G2, (unsigned)nmat), dim3(kGroup), 0, s, a);
      CBFM_HIP(hipGetLastError());
      cur = 1 - cur;
      G = G2;
    }
    RowsArgs r{};
    r.A = A;
    r.strideA = strideA;
    r.ld = ld;
    r.ncols = ncols;
    r.k = k;
    r.w = w;
    r.col0 = inverse ? 0 : k + w;
    r.Dinv = dinv.as<double2>();
    r.swaps = swaps.as<int32_t>();
    const int nchunks = (ncols - r.col0 + kChunk - 1) / kChunk;
    if (nchunks > 0) {
      hipLaunchKernelGGL(gj_rows_kernel, dim3((unsigned)nchunks, (unsigned)nmat), dim3(256), 0, s, r);
      CBFM_HIP(hipGetLastError());
    }
    // rows outside the panel, columns right of it (an inversion: every
    // column; the panel's own columns are overwritten)
    if (n > w && nchunks > 0) {
      TimedLaunch tl(T_GEMM, s, 8.0 * w * (double)(n - w) * (double)(ncols - r.col0) * nmat);
      const UpdateArgs u{A, pcol.as<double2>(), strideA, ld, n, ncols, k, w, r.col0};
      hipLaunchKernelGGL(gj_update_kernel,
                         dim3((unsigned)((ncols - r.col0 + 63) / 64), (unsigned)((n - w + 63) / 64), (unsigned)nmat),
                         dim3(256), 0, s, u);
      CBFM_HIP(hipGetLastError());
    }
  }
  if (!inverse) return;
  // column j of the inverse sits at the position that holds input row j
  const int64_t total = (int64_t)nmat * n;
  Scratch src((size_t)total * sizeof(int32_t), s), tmp((size_t)nmat * strideA * sizeof(double2), s);
  CBFM_HIP(hipMemsetAsync(src.p, 0, (size_t)total * sizeof(int32_t), s));
  hipLaunchKernelGGL(gj_src_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, rowat.as<int32_t>(),
                     src.as<int32_t>(), n, total);
  hipLaunchKernelGGL(gj_gather_kernel, dim3((unsigned)((n + 255) / 256), (unsigned)n, (unsigned)nmat), dim3(256), 0,
                     s, A, tmp.as<double2>(), src.as<int32_t>(), n, strideA);
  CBFM_HIP(hipGetLastError());
  CBFM_HIP(hipMemcpyAsync(A, tmp.p, (size_t)nmat * strideA * sizeof(double2), hipMemcpyDeviceToDevice, s));
}

}  // namespace

void gj_check(const int32_t* info_dev, int nmat, const char* what, hipStream_t s) {
  std::vector<int32_t> info(nmat);
  CBFM_HIP(hipMemcpyAsync(info.data(), info_dev, (size_t)nmat * sizeof(int32_t), hipMemcpyDeviceToHost, s));
  CBFM_HIP(hipStreamSynchronize(s));
  for (int b = 0; b < nmat; ++b)
    CBFM_REQUIRE(info[b] == 0, CBFM_E_RANK,
                 std::string(what) + (nmat > 1 ? " " + std::to_string(b) : std::string()) +
                     " is singular (no nonzero pivot in column " + std::to_string(info[b] - 1) + ")");
}

void gj_inverse_batched_async(double2* A, int64_t strideA, int n, int nmat, int32_t* info_dev, hipStream_t s) {
  CBFM_REQUIRE(strideA == (int64_t)n * n, CBFM_E_ARG, "Gauss-Jordan inversion: matrices must be packed");
  eliminate(A, strideA, n, n, n, nmat, true, info_dev, s);
}

void gj_inverse_batched(double2* A, int64_t strideA, int n, int nmat, const char* what, hipStream_t s) {
  Scratch info((size_t)std::max(1, nmat) * sizeof(int32_t), s);
  gj_inverse_batched_async(A, strideA, n, nmat, info.as<int32_t>(), s);
  gj_check(info.as<int32_t>(), nmat, what, s);
}

void gj_solve_batched(double2* A, int64_t strideA, int64_t ld, int n, int ncols, int nmat, const char* what,
                      hipStream_t s) {
  CBFM_REQUIRE(ncols > n, CBFM_E_ARG, "Gauss-Jordan solve: no right-hand side");
  Scratch info((size_t)std::max(1, nmat) * sizeof(int32_t), s);
  eliminate(A, strideA, ld, n, ncols, nmat, false, info.as<int32_t>(), s);
  gj_check(info.as<int32_t>(), nmat, what, s);
}

}  // namespace cbfm
