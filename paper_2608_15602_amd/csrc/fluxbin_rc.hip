// FluxBin weight decomposition on the GPU (fp64): RC_Decomp and StructuralSearch.
//
// RC_Decomp (App. algorithm "FluxBin Sub-routines"; Def. RC decomposition, Props. 3.2 and 3.3) approximates X * mask,
// block by block of g columns, by K binary bases W^(k) = (alpha_r^(k) alpha_c^(k)^T) * B^(k) with one row scale per
// (row, block) and one column scale per column:
//   greedy initialization: for k = 1..K: B^(k) = sign of the residual on the mask (sign(0) = +1), alpha_c^(k) = 1, one
//   row-scale and one column-scale least-squares update (Prop. 3.2), the residual loses the base's contribution;
//   T rounds of: for each base the row then the column scales by least squares against the target X * mask minus the
//   other bases' contributions; then every element's signs by exhaustive search over the 2^K combinations (Prop. 3.3),
//   first minimum in the order c = 0..2^K-1 (bit k of c set: b_k = +1); signs are 0 off the mask.
// StructuralSearch (Def. Hessian-based Column Saliency, with a diagonal inverse Hessian): S_j = sum_i W_ij^2 / h_j^2,
// and per block of g columns the s columns of largest saliency (equal scores: smaller column index first).
//
// Blocks of at most 128 columns (with eps > 0, and rows enough that the workspace holds the partial sums) run as fused
// passes, one launch per base and round (below). Otherwise every step is a data-parallel kernel over the whole matrix (all
// blocks at once). Launches are in sequence on the stream.
// Sums use fixed reduction trees (no atomics), so results are deterministic. Arithmetic is fp64, the precision in which
// the integer sign decisions are taken.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fluxbin_internal.h"

namespace fluxbin {

namespace {

struct RcArgs {
  const float* X;         // [M][N]
  const uint8_t* mask;    // [N] or nullptr (all columns)
  const uint32_t* pB;     // prior bases subtracted from X (canonical bit planes [Kp][M][ceil(N/32)]), or nullptr
  const double* par;      // [Kp][M][pG]
  const double* pac;      // [Kp][N]
  int32_t Kp;
  int64_t pg, pG, pW;
  int8_t* B;              // [K][M][N]
  double* ar;             // [K][M][G]
  double* ac;             // [K][N]
  int64_t M, N, g, G;
  int32_t K;
  double eps;
};

__device__ __forceinline__ bool rc_in(const RcArgs& a, int64_t j) { return a.mask == nullptr || a.mask[j] != 0; }

// The matrix being decomposed at (i, j), before the mask: X, or X minus the prior bases' approximation (the residual of
// an earlier decomposition, FluxBin-Hybrid step 3), the prior contributions summed first in base order.
__device__ __forceinline__ double rc_x(const RcArgs& a, int64_t i, int64_t j) {
  const double x = double(a.X[i * a.N + j]);
  if (a.pB == nullptr) return x;
  double s = 0.0;
  for (int p = 0; p < a.Kp; ++p) {
    const double m = a.par[(p * a.M + i) * a.pG + j / a.pg] * a.pac[p * a.N + j];
    const bool plus = (a.pB[(p * a.M + i) * a.pW + (j >> 5)] >> (j & 31)) & 1u;
    s += plus ? m : -m;
  }
  return x - s;
}

__device__ __forceinline__ double rc_contrib(const RcArgs& a, int kk, int64_t i, int64_t j) {
  const double m = a.ar[(kk * a.M + i) * a.G + j / a.g] * a.ac[kk * a.N + j];
  return m * double(a.B[(kk * a.M + i) * a.N + j]);
}

// Target of base k at (i, j). Initialization (init != 0): the residual after bases 0..k-1, subtracted one by one.
// Rounds: X * mask minus the sum of the other bases' contributions (summed first, in base order).
__device__ __forceinline__ double rc_target(const RcArgs& a, int k, int init, int64_t i, int64_t j) {
  const double x = rc_in(a, j) ? rc_x(a, i, j) : 0.0;
  if (init) {
    double r = x;
    for (int kk = 0; kk < k; ++kk) r -= rc_contrib(a, kk, i, j);
    return r;
  }
  double s = 0.0;
  for (int kk = 0; kk < a.K; ++kk)
    if (kk != k) s += rc_contrib(a, kk, i, j);
  return x - s;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__global__ void k_rc_fill(double* p, int64_t n, double v) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Greedy initialization of base k's signs: sign of the residual after bases 0..k-1 on the mask, 0 off it.
__global__ void k_rc_init_sign(RcArgs a, int k) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= a.M * a.N) return;
  const int64_t i = e / a.N, j = e - i * a.N;
  int8_t b = 0;
  if (rc_in(a, j)) b = rc_target(a, k, 1, i, j) >= 0.0 ? int8_t(1) : int8_t(-1);
  a.B[(int64_t(k) * a.M + i) * a.N + j] = b;
}

// Row scales of base k (Prop. 3.2): one wavefront per (row, block), lanes over the block's columns.
__global__ void __launch_bounds__(256) k_rc_row(RcArgs a, int k, int init) {
  const int64_t wid = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (wid >= a.M * a.G) return;   // whole wavefronts leave together
  const int64_t i = wid / a.G, blk = wid - i * a.G;
  const int64_t c0 = blk * a.g, c1 = c0 + a.g < a.N ? c0 + a.g : a.N;
  double num = 0.0, den = 0.0;
  for (int64_t j = c0 + lane; j < c1; j += 64) {
    const double cb = a.ac[int64_t(k) * a.N + j] * double(a.B[(int64_t(k) * a.M + i) * a.N + j]);
    num += cb * rc_target(a, k, init, i, j);
    den += cb * cb;
  }
  num = wave_sum(num);
  den = wave_sum(den);
  if (lane == 0) a.ar[(int64_t(k) * a.M + i) * a.G + blk] = num / (den + a.eps);
}

// Column scales of base k (Prop. 3.2), first stage: workgroup (tile of 64 columns, row slice r of RS) sums its rows
// in four interleaved sub-slices combined in a fixed order, into part[r][2][N] (numerator, denominator).
__global__ void __launch_bounds__(256) k_rc_col(RcArgs a, int k, int init, int64_t rows_per_slice, double* part) {
  __shared__ double s_num[4][64], s_den[4][64];
  const int c = threadIdx.x & 63, sub = threadIdx.x >> 6;
  const int64_t j = int64_t(blockIdx.x) * 64 + c;
  const int64_t r = blockIdx.y;
  const int64_t i0 = r * rows_per_slice, i1 = i0 + rows_per_slice < a.M ? i0 + rows_per_slice : a.M;
  double num = 0.0, den = 0.0;
  if (j < a.N) {
    const int64_t blk = j / a.g;
    for (int64_t i = i0 + sub; i < i1; i += 4) {
      const double rb = a.ar[(int64_t(k) * a.M + i) * a.G + blk] * double(a.B[(int64_t(k) * a.M + i) * a.N + j]);
      num += rb * rc_target(a, k, init, i, j);
      den += rb * rb;
    }
  }
  s_num[sub][c] = num;
  s_den[sub][c] = den;
  __syncthreads();
  if (sub == 0 && j < a.N) {
    part[(r * 2 + 0) * a.N + j] = ((s_num[0][c] + s_num[1][c]) + s_num[2][c]) + s_num[3][c];
    part[(r * 2 + 1) * a.N + j] = ((s_den[0][c] + s_den[1][c]) + s_den[2][c]) + s_den[3][c];
  }
}

// Second stage: the slices' sums added in slice order, then the least-squares quotient.
__global__ void k_rc_col_fin(RcArgs a, int k, int64_t slices, const double* part) {
  const int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (j >= a.N) return;
  double n = 0.0, d = 0.0;
  for (int64_t r = 0; r < slices; ++r) {
    n += part[(r * 2 + 0) * a.N + j];
    d += part[(r * 2 + 1) * a.N + j];
  }
  a.ac[int64_t(k) * a.N + j] = n / (d + a.eps);
}

// Joint sign search (Prop. 3.3) for every element: the first of the 2^K combinations with the smallest |x - approx|.
template <int K>
__global__ void k_rc_sign(RcArgs a) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= a.M * a.N) return;
  const int64_t i = e / a.N, j = e - i * a.N;
  const bool in = rc_in(a, j);
  const double x = in ? rc_x(a, i, j) : 0.0;
  const int64_t blk = j / a.g;
  double m[K];
#pragma unroll
  for (int k = 0; k < K; ++k) m[k] = a.ar[(int64_t(k) * a.M + i) * a.G + blk] * a.ac[int64_t(k) * a.N + j];
  double best = 0.0;
  int best_c = -1;
#pragma unroll
  for (int c = 0; c < (1 << K); ++c) {
    double approx = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) approx += ((c >> k) & 1) ? m[k] : -m[k];
    const double err = fabs(x - approx);
    if (best_c < 0 || err < best) {
      best = err;
      best_c = c;
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k)
    a.B[(int64_t(k) * a.M + i) * a.N + j] = in ? (((best_c >> k) & 1) ? int8_t(1) : int8_t(-1)) : int8_t(0);
}

// Signs to canonical planes [K][M][ceil(N/32)]: bit t of word w is B[k][i][32w + t] == +1.
__global__ void k_rc_bits(RcArgs a, uint32_t* out) {
  const int64_t W = (a.N + 31) / 32;
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= int64_t(a.K) * a.M * W) return;
  const int64_t row = e / W, w = e - row * W;   // row = k * M + i
  uint32_t bits = 0u;
  for (int t = 0; t < 32; ++t) {
    const int64_t j = w * 32 + t;
    if (j < a.N && a.B[row * a.N + j] == 1) bits |= 1u << t;
  }
  out[e] = bits;
}

// Column saliency S_j = sum_i W_ij^2 / h_j^2: a workgroup per C columns, SL row slices combined in a fixed order. 16
// columns (64-byte row segments) and 64 slices rather than 64 columns and 4 slices: 4096 columns are then a workgroup per
// CU instead of 64 workgroups (4096 x 4096: 255 -> 22 us; a read of the matrix at 5 TB/s is 13 us). Where 64-column
// workgroups fill the CUs as well (64 columns per CU and more), they are the faster form, with 4 slices for few rows
// (whole search in a graph, 16 columns -> 64: 64 x 65536 23.8 -> 12.8 us, 1024 x 65536 94.6 -> 50.6, 4096 x 16384 90.9 ->
// 49.8).
template <int C, int SL>
__global__ void __launch_bounds__(C * SL) k_saliency(const float* W, const double* h, int64_t M, int64_t N, double* S) {
  __shared__ double s_sum[SL][C + 1];
  const int c = int(threadIdx.x) % C, slice = int(threadIdx.x) / C;
  const int64_t j = int64_t(blockIdx.x) * C + c;
  double acc = 0.0;
  if (j < N) {
    int64_t i = slice;
    for (; i + 7 * SL < M; i += 8 * SL) {   // eight loads in flight
      float w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) w[u] = W[(i + SL * u) * N + j];
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += double(w[u]) * double(w[u]);
    }
    for (; i < M; i += SL) {
      const double w = double(W[i * N + j]);
      acc += w * w;
    }
  }
  s_sum[slice][c] = acc;
  __syncthreads();
  for (int half = SL / 2; half >= 1; half >>= 1) {
    if (slice < half) s_sum[slice][c] += s_sum[slice + half][c];
    __syncthreads();
  }
  if (slice == 0 && j < N) S[j] = s_sum[0][c] / (h[j] * h[j]);
}

// Per block of g columns (a workgroup each, g <= 1024): column j is selected when fewer than s columns of the block
// rank before it (larger score, or equal score and smaller index); the selected columns are written in increasing
// index order after the min(s, g) columns of every earlier block.
__global__ void __launch_bounds__(1024) k_topk(const double* S, int64_t N, int64_t g, int64_t s, int32_t* idx,
                                               uint8_t* mask) {
  __shared__ double sc[1024];
  __shared__ int sel[1024];
  const int64_t c0 = int64_t(blockIdx.x) * g;
  const int n = int(c0 + g < N ? g : N - c0);
  const int t = threadIdx.x;
  if (t < n) sc[t] = S[c0 + t];
  __syncthreads();
  int chosen = 0;
  if (t < n) {
    int rank = 0;
    for (int u = 0; u < n; ++u) rank += (sc[u] > sc[t] || (sc[u] == sc[t] && u < t)) ? 1 : 0;
    chosen = rank < s ? 1 : 0;
  }
  sel[t] = chosen;
  if (mask != nullptr && t < n) mask[c0 + t] = uint8_t(chosen);
  __syncthreads();
  if (t < n && chosen) {
    int before = 0;
    for (int u = 0; u < t; ++u) before += sel[u];
    idx[int64_t(blockIdx.x) * s + before] = int32_t(c0 + t);
  }
}

unsigned grid_for(int64_t n, int per) { return unsigned((n + per - 1) / per); }

// Row slices of the column-scale sums: at least 256 rows each, at most 64 slices.
int64_t col_slices(int64_t M) {
  const int64_t s = M / 256;
  return s < 1 ? 1 : (s > 64 ? 64 : s);
}

// ---------------------------------------------------------------------------------------------------------------------
// Fused passes (blocks of at most 128 columns). One launch per base and round instead of five: a wavefront takes whole
// rows of a block, so the joint sign search of the round before, base k's row scale and the row's terms of base k's
// column sums follow one another on values in registers, and the matrix is read once per base and round. The column
// scales need every row: a launch leaves one sum per row slice and column, and the next one's workgroups add the slices
// of their block first. Signs are bits (one 64-bit word per row, block and 64 columns).
//
// With a mask (the salient columns of FluxBin-Hybrid: 8 or 16 of 128) only its columns are carried along: a wavefront's lanes
// are the masked columns of several rows, and x (minus the prior bases) is computed once, into an fp64 copy of those columns.
//
// 4096 x 4096, 2 + 2 bases, 8 salient columns per block, 10 rounds, both decompositions and the saliency search:
// 9880 -> 899 us. Of the 23 launches over the full matrix a round pass takes 22 us (64 MB of X: 13 us at the copy rate)
// and one with the sign search 34 (fp64 issue; 42 with every combination's error as its own sum and a select per sign);
// a launch over the masked columns 9 to 12 us (latency). About 7 us of each pass are its start: the slices' sums, added by
// four threads per column (one thread: 1 to 1.5 us more), and the quotients; two waves of smaller workgroups pay it twice
// (768 or 1024 workgroups 1.2 to 1.3 times as long). Sign words and row scales through scalar loads: 25.8 and 39 us.
// ---------------------------------------------------------------------------------------------------------------------

constexpr int kRcWaves = 8;        // wavefronts of a workgroup
constexpr int kRcMaxG = 128;       // block columns: two per lane
constexpr int kRcParts = 64 * kRcWaves / kRcMaxG;   // threads per column where the slices' sums are added

struct RcPass {
  RcArgs a;
  uint64_t* bits;          // [K][G][M][2] signs of a block's listed columns 0..63, 64..127 (set: +1)
  const int32_t* nm;       // [G] listed columns of a block, or nullptr (all)
  const uint16_t* cols;    // [G][g] their offsets in the block, increasing
  const double* xc;        // x of the listed columns of blocks with nm <= cap: [M][nm] at blk * M * cap
  int32_t cap;
  int32_t kprev;           // base whose column sums num_in and den_in hold (-1: none)
  int64_t rows_per_slice, slices;
  const double* num_in;    // [slices][N], [slices][G]
  const double* den_in;
  double* num_out;
  double* den_out;
};

// What a pass does with its rows, for base KB.
enum RcMode {
  kRcInit,       // greedy initialization: signs of the residual, then row scales and column sums
  kRcRound,      // row scales and column sums with the signs as they are
  kRcSignRound,  // the joint sign search first
  kRcSign,       // the joint sign search only
  kRcScales,     // no rows: only the column scales of the pass before
};

template <int CTRL>
__device__ __forceinline__ double rc_dpp(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const int lo = __builtin_amdgcn_mov_dpp(int(uint32_t(u)), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(int(uint32_t(u >> 32)), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t(uint32_t(hi)) << 32) | uint32_t(lo));
}

__device__ __forceinline__ double rc_readlane(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(u)), lane));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(u >> 32)), lane));
  return __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo);
}

// v + v of lane ^ D, D = 16 or 32: the two registers of a swap hold the lane's and its partner's.
template <int D>
__device__ __forceinline__ double rc_add_swapped(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = uint32_t(u), hi = uint32_t(u >> 32);
  uint64_t x, y;
  if constexpr (D == 16) {
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    x = (uint64_t(h[0]) << 32) | l[0];
    y = (uint64_t(h[1]) << 32) | l[1];
  } else {
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    x = (uint64_t(h[0]) << 32) | l[0];
    y = (uint64_t(h[1]) << 32) | l[1];
  }
  return __builtin_bit_cast(double, x) + __builtin_bit_cast(double, y);
}

// Sums of four values over the wavefront, value lane & 3 in each lane: two exchange steps that halve the values carried,
// then four that add over the lanes (3 + 4 additions instead of 24).
__device__ __forceinline__ double rc_sum4(const double (&v)[4], int lane) {
  const bool o1 = (lane & 1) != 0, o2 = (lane & 2) != 0;
  const double a = (o1 ? v[1] : v[0]) + rc_dpp<0xB1>(o1 ? v[0] : v[1]);   // quad_perm 1,0,3,2
  const double b = (o1 ? v[3] : v[2]) + rc_dpp<0xB1>(o1 ? v[2] : v[3]);
  double s = (o2 ? b : a) + rc_dpp<0x4E>(o2 ? a : b);                       // quad_perm 2,3,0,1
  s += rc_dpp<0x124>(s);                                                    // row_ror 4
  s += rc_dpp<0x128>(s);                                                    // row_ror 8
  return rc_add_swapped<32>(rc_add_swapped<16>(s));
}

// -b v for a sign b = +-1 given as a mask (b = +1: plus) or as a word with its top bit set for +1 (two instructions
// either way; with the top bit, the shift that brings it there included).
__device__ __forceinline__ double rc_minus(double v, bool plus) { return plus ? -v : v; }
__device__ __forceinline__ double rc_minus(double v, uint32_t top) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  return __builtin_bit_cast(double, (uint64_t(uint32_t(u >> 32) ^ (top & 0x80000000u)) << 32) | uint32_t(u));
}

// Joint sign search (Prop. 3.3) for one element: whether b_k = +1. The first of the 2^K combinations, bit k of c being
// b_k = +1, with the least |x - sum b_k m_k|. Combinations c and ~c are each other's negatives exactly (rounding is
// symmetric), and the choice is kept as wavefront masks: 12 vector instructions per element for K = 2.
template <int K>
__device__ __forceinline__ void rc_search(double x, const double (&m)[K], bool (&plus)[K]) {
  constexpr int H = 1 << (K - 1);
  double sum[H];   // combinations with b_{K-1} = -1
#pragma unroll
  for (int c = 0; c < H; ++c) {
    double v = K > 1 && (c & 1) ? m[0] : -m[0];
#pragma unroll
    for (int k = 1; k < K; ++k) v += ((c >> k) & 1) ? m[k] : -m[k];
    sum[c] = v;
  }
  double best = fabs(x - sum[0]);
#pragma unroll
  for (int k = 0; k < K; ++k) plus[k] = false;
#pragma unroll
  for (int c = 1; c < 2 * H; ++c) {
    const double err = fabs(c < H ? x - sum[c] : x + sum[2 * H - 1 - c]);
    const bool less = err < best;
    best = fmin(best, err);
#pragma unroll
    for (int k = 0; k < K; ++k) plus[k] = ((c >> k) & 1) ? plus[k] | less : plus[k] & !less;
  }
}

// Column scales of the lane's columns: base kprev's from the slices' sums (slice order), the others' as stored; base
// k's are 1 in its initialization. col[c]: the lane's columns in the matrix, or -1.
template <int K, int KB, RcMode MODE>
__device__ __forceinline__ void rc_scales(const RcPass& p, int64_t blk, int64_t c0, int nc, const int64_t (&col)[2],
                                          double* s_ac, double (*s_part)[2][kRcMaxG], double (&ac)[K][2]) {
  const RcArgs& a = p.a;
  double stored[K][2];   // requested before the sums
#pragma unroll
  for (int kk = 0; kk < K; ++kk)
#pragma unroll
    for (int c = 0; c < 2; ++c)
      stored[kk][c] = MODE != kRcScales && (MODE != kRcInit || kk < KB) && col[c] >= 0 && kk != p.kprev
                          ? a.ac[int64_t(kk) * a.N + col[c]]
                          : 0.0;
  if (p.kprev >= 0) {   // a quarter of the slices per thread, then the quarters in order
    const int t = int(threadIdx.x) & (kRcMaxG - 1), part = int(threadIdx.x) / kRcMaxG;
    const int64_t q = (p.slices + kRcParts - 1) / kRcParts, r1 = q * part + q < p.slices ? q * part + q : p.slices;
    if (t < nc) {
      double n = 0.0, d = 0.0;
      for (int64_t r0 = q * part; r0 < r1; r0 += 4) {
        double u[4], w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {   // unconditional: the loads are in flight together
          const int64_t rr = r0 + r < r1 ? r0 + r : r1 - 1;
          u[r] = p.num_in[rr * a.N + c0 + t];
          w[r] = p.den_in[rr * a.G + blk];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          n += r0 + r < r1 ? u[r] : 0.0;
          d += r0 + r < r1 ? w[r] : 0.0;
        }
      }
      s_part[part][0][t] = n;
      s_part[part][1][t] = d;
    }
    __syncthreads();
    if (part == 0 && t < nc) {
      double n = 0.0, d = 0.0;
#pragma unroll
      for (int k = 0; k < kRcParts; ++k) {
        n += s_part[k][0][t];
        d += s_part[k][1][t];
      }
      const bool in = p.nm == nullptr || rc_in(a, c0 + t);
      const double v = in ? n / (d + a.eps) : 0.0;
      s_ac[t] = v;
      if (blockIdx.y == 0) a.ac[int64_t(p.kprev) * a.N + c0 + t] = v;
    }
    __syncthreads();
  }
#pragma unroll
  for (int kk = 0; kk < K; ++kk)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      double v = 0.0;
      if (col[c] >= 0) {
        if (MODE == kRcInit && kk == KB)
          v = 1.0;
        else if (kk == p.kprev)
          v = s_ac[col[c] - c0];
        else if (MODE != kRcInit || kk < KB)
          v = stored[kk][c];
      }
      ac[kk][c] = v;
    }
}

// Target of base k for one element with the contributions m[kk] * b_kk of the other bases (order as rc_target).
template <int K, int KB, RcMode MODE, class Sign>
__device__ __forceinline__ double rc_residual(double x, const double (&m)[K], const Sign (&b)[K]) {
  if constexpr (MODE == kRcInit) {
#pragma unroll
    for (int kk = 0; kk < KB; ++kk) x += rc_minus(m[kk], b[kk]);
    return x;
  }
  if constexpr (K == 1) return x;
  double s = 0.0;   // minus their sum
#pragma unroll
  for (int kk = 0; kk < K; ++kk)
    if (kk != KB) s = kk == (KB == 0 ? 1 : 0) ? rc_minus(m[kk], b[kk]) : s + rc_minus(m[kk], b[kk]);
  return x + s;
}

// Whether a pass reads base kk's row scales / signs.
template <int KB, RcMode MODE>
__device__ __forceinline__ constexpr bool rc_reads_ar(int kk) {
  return MODE == kRcInit ? kk < KB : MODE == kRcRound ? kk != KB : true;
}
template <int KB, RcMode MODE>
__device__ __forceinline__ constexpr bool rc_reads_signs(int kk) {
  return MODE == kRcInit ? kk < KB : MODE == kRcRound;
}

// The workgroup's column sums: the wavefronts' (and, with several rows per wavefront, the row groups') in a fixed order.
// ALL: off covers every column of the block.
template <bool ALL>
__device__ __forceinline__ void rc_store_sums(const RcPass& p, int64_t blk, int64_t c0, int nc, const int (&off)[2],
                                              const double (&cn)[2], double cd, double (&s_sum)[kRcWaves][kRcMaxG],
                                              double (&s_den)[kRcWaves]) {
  const int wave = int(threadIdx.x) >> 6, lane = int(threadIdx.x) & 63;
  if constexpr (!ALL) {
    for (int t = lane; t < nc; t += 64) s_sum[wave][t] = 0.0;
    __syncthreads();
  }
#pragma unroll
  for (int c = 0; c < 2; ++c)
    if (off[c] >= 0) s_sum[wave][off[c]] = cn[c];
  if (lane == 0) s_den[wave] = cd;
  __syncthreads();
  const int t = int(threadIdx.x);
  if (t < nc) {
    double n = 0.0;
    for (int w = 0; w < kRcWaves; ++w) n += s_sum[w][t];
    p.num_out[int64_t(blockIdx.y) * p.a.N + c0 + t] = n;
  }
  if (t == 0) {
    double d = 0.0;
    for (int w = 0; w < kRcWaves; ++w) d += s_den[w];
    p.den_out[int64_t(blockIdx.y) * p.a.G + blk] = d;
  }
}

// Four rows of a block as a wavefront loads them.
template <int K>
struct RcRows {
  float x[4][2];
  double ar[K][4];
  uint32_t w[K][4][2];
};

// Every column of the block, X as given: lane l has columns l and l + 64, a wavefront four rows at a time, the next four
// requested before them.
template <int K, int KB, RcMode MODE>
__global__ void __launch_bounds__(64 * kRcWaves) k_rc_pass(RcPass p) {
  __shared__ double s_ac[kRcMaxG], s_den[kRcWaves];
  __shared__ union {
    double sum[kRcWaves][kRcMaxG], part[kRcParts][2][kRcMaxG];
  } sh;
  constexpr bool kUpdate = MODE != kRcSign, kSearch = MODE == kRcSign || MODE == kRcSignRound;
  const RcArgs& a = p.a;
  const int lane = int(threadIdx.x) & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int64_t blk = blockIdx.x, c0 = blk * a.g;
  const int nc = int(c0 + a.g < a.N ? a.g : a.N - c0);
  const int off[2] = {lane < nc ? lane : -1, lane + 64 < nc ? lane + 64 : -1};
  const int64_t col[2] = {off[0] >= 0 ? c0 + off[0] : -1, off[1] >= 0 ? c0 + off[1] : -1};
  const int64_t i0 = int64_t(blockIdx.y) * p.rows_per_slice;
  const int64_t i1 = i0 + p.rows_per_slice < a.M ? i0 + p.rows_per_slice : a.M;
  const float* xp = a.X + c0;
  // columns past the block read its first one; their scales are zero and their x is replaced by zero
  const int offc[2] = {off[0] >= 0 ? off[0] : 0, off[1] >= 0 ? off[1] : 0};
  auto load = [&](int64_t i, RcRows<K>& r) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t row = i + u < i1 ? i + u : i1 - 1;
#pragma unroll
      for (int c = 0; c < 2; ++c) r.x[u][c] = xp[row * a.N + offc[c]];
#pragma unroll
      for (int kk = 0; kk < K; ++kk) {
        if (rc_reads_ar<KB, MODE>(kk)) r.ar[kk][u] = a.ar[(int64_t(kk) * a.M + row) * a.G + blk];
        if (rc_reads_signs<KB, MODE>(kk)) {
          const uint32_t* q = reinterpret_cast<const uint32_t*>(p.bits + ((int64_t(kk) * a.G + blk) * a.M + row) * 2);
          r.w[kk][u][0] = q[lane >> 5];
          r.w[kk][u][1] = q[2 + (lane >> 5)];
        }
      }
    }
  };
  int64_t i = i0 + 4 * wave;
  RcRows<K> next;
  if (i < i1) load(i, next);   // while the column scales are put together
  double ac[K][2];
  rc_scales<K, KB, MODE>(p, blk, c0, nc, col, s_ac, sh.part, ac);
  const double den = kUpdate ? wave_sum(ac[KB][0] * ac[KB][0] + ac[KB][1] * ac[KB][1]) + a.eps : 0.0;

  double cn[2] = {0.0, 0.0}, cd = 0.0;
  for (; i < i1; i += 4 * kRcWaves) {
    const RcRows<K> r = next;
    if (i + 4 * kRcWaves < i1) load(i + 4 * kRcWaves, next);
    asm volatile("" ::: "memory");   // requested here
    double num[4], tgt[4][2];   // both times -1: minus the targets times base KB's signs
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      num[u] = 0.0;
      uint64_t ball[K][2];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const double x = off[c] >= 0 ? double(r.x[u][c]) : 0.0;
        double m[K];
        std::conditional_t<kSearch, bool, uint32_t> sign[K];
#pragma unroll
        for (int kk = 0; kk < K; ++kk) {
          m[kk] = rc_reads_ar<KB, MODE>(kk) ? r.ar[kk][u] * ac[kk][c] : 0.0;
          sign[kk] = rc_reads_signs<KB, MODE>(kk) ? r.w[kk][u][c] << (31 - (lane & 31)) : 0u;
        }
        if constexpr (kSearch) {
          rc_search<K>(x, m, sign);
#pragma unroll
          for (int kk = 0; kk < K; ++kk) ball[kk][c] = __builtin_amdgcn_ballot_w64(off[c] >= 0 && sign[kk]);
        }
        if constexpr (kUpdate) {
          const double t = rc_residual<K, KB, MODE>(x, m, sign);
          if constexpr (MODE == kRcInit) {
            sign[KB] = t >= 0.0 ? 0x80000000u : 0u;
            ball[KB][c] = __builtin_amdgcn_ballot_w64(off[c] >= 0 && t >= 0.0);
          }
          tgt[u][c] = rc_minus(t, sign[KB]);
          num[u] += ac[KB][c] * tgt[u][c];
        }
      }
      if ((kSearch || MODE == kRcInit) && i + u < i1 && lane < 2) {
#pragma unroll
        for (int kk = 0; kk < K; ++kk)
          if (kSearch || kk == KB)
            p.bits[((int64_t(kk) * a.G + blk) * a.M + i + u) * 2 + lane] = lane == 0 ? ball[kk][0] : ball[kk][1];
      }
    }
    if constexpr (kUpdate) {
      const double v = rc_sum4(num, lane) / den;
      if (lane < 4 && i + lane < i1) a.ar[(int64_t(KB) * a.M + i + lane) * a.G + blk] = -v;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (i + u >= i1) continue;
        const double vu = rc_readlane(v, u);
#pragma unroll
        for (int c = 0; c < 2; ++c) cn[c] += vu * tgt[u][c];
        cd += vu * vu;
      }
    }
  }
  if constexpr (kUpdate) rc_store_sums<true>(p, blk, c0, nc, off, cn, cd, sh.sum, s_den);
}

// Listed columns only (and prior bases): U groups of 64 / P rows at a time, P = 8, 16, 32 or 64 lanes per row, C = 2
// columns per lane where a block lists more than 64. Bound by latency (loads, exchanges, a quotient per row), so the
// groups' loads are requested together.
template <int K, int KB, RcMode MODE, int U, int C>
__device__ __forceinline__ void rc_list_rows(const RcPass& p, int64_t blk, int nm, int P, const int (&off)[2],
                                             const int64_t (&col)[2], const double (&ac)[K][2], double den,
                                             double (&cn)[2], double& cd) {
  constexpr bool kUpdate = MODE != kRcSign, kSearch = MODE == kRcSign || MODE == kRcSignRound;
  const RcArgs& a = p.a;
  const int lane = int(threadIdx.x) & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int RW = 64 / P, pos = lane & (P - 1), sub = lane / P;
  const int64_t i0 = int64_t(blockIdx.y) * p.rows_per_slice;
  const int64_t i1 = i0 + p.rows_per_slice < a.M ? i0 + p.rows_per_slice : a.M;
  const bool copied = p.xc != nullptr && nm <= p.cap;
  const int64_t base_words = a.G * a.M * 2;
  for (int64_t ib = i0 + U * RW * wave; ib < i1; ib += U * RW * kRcWaves) {
    double x[U][C], ar[K][U];
    uint64_t w[K][U][C];
    int64_t row[U];
    bool in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = ib + RW * u + sub;
      in[u] = i < i1;
      row[u] = in[u] ? i : i1 - 1;
#pragma unroll
      for (int c = 0; c < C; ++c) {
        x[u][c] = 0.0;
        if (off[c] >= 0)
          x[u][c] = copied ? p.xc[blk * a.M * p.cap + row[u] * nm + pos + 64 * c] : rc_x(a, row[u], col[c]);
      }
#pragma unroll
      for (int kk = 0; kk < K; ++kk) {
        if (rc_reads_ar<KB, MODE>(kk)) ar[kk][u] = a.ar[(int64_t(kk) * a.M + row[u]) * a.G + blk];
#pragma unroll
        for (int c = 0; c < C; ++c)
          if (rc_reads_signs<KB, MODE>(kk)) w[kk][u][c] = p.bits[kk * base_words + (blk * a.M + row[u]) * 2 + c];
      }
    }
    double num[U], tgt[U][C];   // both times -1: minus the targets times base KB's signs
#pragma unroll
    for (int u = 0; u < U; ++u) {
      num[u] = 0.0;
      uint64_t* word = p.bits + (blk * a.M + row[u]) * 2;
      auto store = [&](int kk, int c, bool plus) __attribute__((always_inline)) {
        const uint64_t ball = __builtin_amdgcn_ballot_w64(off[c] >= 0 && plus);
        if (in[u] && pos == 0)
          word[kk * base_words + c] = P == 64 ? ball : (ball >> (sub * P)) & ((uint64_t(1) << P) - 1);
      };
#pragma unroll
      for (int c = 0; c < C; ++c) {
        double m[K];
        std::conditional_t<kSearch, bool, uint32_t> sign[K];
#pragma unroll
        for (int kk = 0; kk < K; ++kk) {
          m[kk] = rc_reads_ar<KB, MODE>(kk) ? ar[kk][u] * ac[kk][c] : 0.0;
          sign[kk] = rc_reads_signs<KB, MODE>(kk) ? uint32_t(w[kk][u][c] >> pos) << 31 : 0u;
        }
        if constexpr (kSearch) {
          rc_search<K>(x[u][c], m, sign);
#pragma unroll
          for (int kk = 0; kk < K; ++kk) store(kk, c, sign[kk]);
        }
        if constexpr (kUpdate) {
          const double t = rc_residual<K, KB, MODE>(x[u][c], m, sign);
          if constexpr (MODE == kRcInit) {
            sign[KB] = t >= 0.0 ? 0x80000000u : 0u;
            store(KB, c, t >= 0.0);
          }
          tgt[u][c] = rc_minus(t, sign[KB]);
          num[u] += ac[KB][c] * tgt[u][c];
        }
      }
    }
    if constexpr (kUpdate) {
      for (int s = 1; s < P; s <<= 1)
#pragma unroll
        for (int u = 0; u < U; ++u) num[u] += __shfl_xor(num[u], s, 64);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const double r = num[u] / den;
        if (!in[u]) continue;
        if (pos == 0) a.ar[(int64_t(KB) * a.M + row[u]) * a.G + blk] = -r;
#pragma unroll
        for (int c = 0; c < C; ++c) cn[c] += r * tgt[u][c];
        cd += r * r;
      }
    }
  }
}

template <int K, int KB, RcMode MODE>
__global__ void __launch_bounds__(64 * kRcWaves) k_rc_pass_list(RcPass p) {
  __shared__ double s_ac[kRcMaxG], s_den[kRcWaves];
  __shared__ union {
    double sum[kRcWaves][kRcMaxG], part[kRcParts][2][kRcMaxG];
  } sh;
  constexpr bool kUpdate = MODE != kRcSign;
  const RcArgs& a = p.a;
  const int lane = int(threadIdx.x) & 63;
  const int64_t blk = blockIdx.x, c0 = blk * a.g;
  const int nc = int(c0 + a.g < a.N ? a.g : a.N - c0);
  const int nm = p.nm != nullptr ? p.nm[blk] : nc;
  const int P = nm > 32 ? 64 : nm > 16 ? 32 : nm > 8 ? 16 : 8;
  const int pos = lane & (P - 1);
  int off[2];
  int64_t col[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int e = pos + 64 * c;
    off[c] = (c == 0 || P == 64) && e < nm ? (p.nm != nullptr ? int(p.cols[blk * a.g + e]) : e) : -1;
    col[c] = off[c] >= 0 ? c0 + off[c] : -1;
  }
  double ac[K][2];
  rc_scales<K, KB, MODE>(p, blk, c0, nc, col, s_ac, sh.part, ac);
  double den = ac[KB][0] * ac[KB][0] + ac[KB][1] * ac[KB][1];
  for (int s = 1; s < P; s <<= 1) den += __shfl_xor(den, s, 64);
  den += a.eps;

  double cn[2] = {0.0, 0.0}, cd = 0.0;
  if (nm > 64)
    rc_list_rows<K, KB, MODE, 1, 2>(p, blk, nm, P, off, col, ac, den, cn, cd);
  else
    rc_list_rows<K, KB, MODE, 4, 1>(p, blk, nm, P, off, col, ac, den, cn, cd);
  if constexpr (kUpdate) {
    for (int s = P; s < 64; s <<= 1) {   // the wavefront's row groups
      cn[0] += __shfl_xor(cn[0], s, 64);
      cd += __shfl_xor(cd, s, 64);
    }
    if (lane >= P) off[0] = off[1] = -1;
    rc_store_sums<false>(p, blk, c0, nc, off, cn, cd, sh.sum, s_den);
  }
}

// Only the column scales of the pass before.
template <int K>
__global__ void __launch_bounds__(64 * kRcWaves) k_rc_last_scales(RcPass p) {
  __shared__ double s_ac[kRcMaxG], s_part[kRcParts][2][kRcMaxG];
  const int64_t blk = blockIdx.x, c0 = blk * p.a.g, none[2] = {-1, -1};
  double ac[K][2];
  rc_scales<K, 0, kRcScales>(p, blk, c0, int(c0 + p.a.g < p.a.N ? p.a.g : p.a.N - c0), none, s_ac, s_part, ac);
}

// The masked columns of every block (a workgroup each): their offsets, their number, and zero column scales off the mask.
__global__ void __launch_bounds__(kRcMaxG) k_rc_list(RcArgs a, int32_t* nm, uint16_t* cols, uint16_t* pos) {
  __shared__ int in[kRcMaxG];
  const int t = int(threadIdx.x);
  const int64_t c0 = int64_t(blockIdx.x) * a.g;
  const int nc = int(c0 + a.g < a.N ? a.g : a.N - c0);
  in[t] = t < nc && rc_in(a, c0 + t) ? 1 : 0;
  __syncthreads();
  int before = 0;
  for (int u = 0; u < t; ++u) before += in[u];
  if (t < nc) {
    pos[c0 + t] = in[t] != 0 ? uint16_t(before) : uint16_t(0xFFFFu);
    if (in[t] != 0)
      cols[int64_t(blockIdx.x) * a.g + before] = uint16_t(t);
    else
      for (int k = 0; k < a.K; ++k) a.ac[int64_t(k) * a.N + c0 + t] = 0.0;
  }
  if (t == kRcMaxG - 1) nm[blockIdx.x] = before + in[t];
}

// x of the listed columns [M][nm] of the blocks that list at most cap.
__global__ void __launch_bounds__(256) k_rc_copy(RcArgs a, const int32_t* nm, const uint16_t* cols, int cap, double* xc) {
  const int64_t blk = blockIdx.y;
  const int n = nm[blk];
  if (n > cap) return;
  for (int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x; e < a.M * n; e += int64_t(gridDim.x) * 256) {
    const int64_t i = e / n;
    xc[blk * a.M * cap + e] = rc_x(a, i, blk * a.g + cols[blk * a.g + (e - i * n)]);
  }
}

// The blocks' sign words to canonical planes [K][M][ceil(N/32)], blocks of whole words: one thread per (base, block, row).
__global__ void __launch_bounds__(256) k_rc_planes_blocks(RcArgs a, const uint64_t* bits, const int32_t* nm,
                                                          const uint16_t* cols, uint32_t* out) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x, blk = blockIdx.y, k = blockIdx.z;
  if (i >= a.M) return;
  const int64_t W = (a.N + 31) / 32, w0 = blk * (a.g / 32);
  uint64_t v[2] = {bits[((k * a.G + blk) * a.M + i) * 2], bits[((k * a.G + blk) * a.M + i) * 2 + 1]};
  if (nm != nullptr) {   // listed columns to their places
    uint64_t to[2] = {0, 0};
    const int n = nm[blk];
    for (int e = 0; e < n; ++e) {
      const int t = cols[blk * a.g + e];
      const uint64_t bit = ((e < 64 ? v[0] : v[1]) >> (e & 63)) & 1u;
      to[0] |= t < 64 ? bit << t : 0;
      to[1] |= t >= 64 ? bit << (t & 63) : 0;
    }
    v[0] = to[0];
    v[1] = to[1];
  }
  uint32_t* dst = out + (k * a.M + i) * W + w0;
  for (int w = 0; w < a.g / 32 && w0 + w < W; ++w) dst[w] = uint32_t(v[w >> 1] >> (32 * (w & 1)));
}

// The same for any block width: one thread per word.
__global__ void __launch_bounds__(256) k_rc_planes(RcArgs a, const uint64_t* bits, const uint16_t* pos, uint32_t* out) {
  const int64_t W = (a.N + 31) / 32;
  const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (e >= int64_t(a.K) * a.M * W) return;
  const int64_t row = e / W, w = e - row * W, k = row / a.M, i = row - k * a.M;
  uint32_t v = 0u;
  for (int t = 0; t < 32; ++t) {
    const int64_t j = w * 32 + t;
    if (j >= a.N) break;
    const int64_t blk = j / a.g;
    const int q = pos != nullptr ? int(pos[j]) : int(j - blk * a.g);
    if (q == 0xFFFF) continue;
    v |= uint32_t((bits[((k * a.G + blk) * a.M + i) * 2 + (q >> 6)] >> (q & 63)) & 1u) << t;
  }
  out[e] = v;
}

// Workspace of the fused passes within `bytes`; false if they do not fit (few rows) or do not take the call.
struct RcPlan {
  size_t bits, num[2], den[2], nm, cols, pos, xc;
  int64_t slices, rows_per_slice;
  int32_t cap;
};

bool rc_plan(const RcArgs& a, size_t bytes, RcPlan* q) {
  // eps = 0: the quotients off the mask are 0 / 0 in the general kernels
  if (a.g > kRcMaxG || !(a.eps > 0.0) || a.M >= (int64_t(1) << 31) || a.G > 65535) return false;
  // about two workgroups per CU, at least 64 rows each (two rounds of the wavefronts)
  int64_t s = (512 + a.G - 1) / a.G;
  const int64_t most = (a.M + 63) / 64;
  s = s < 1 ? 1 : s > 64 ? 64 : s;
  s = s > most ? most : s;
  q->rows_per_slice = ((a.M + s - 1) / s + 31) / 32 * 32;
  q->slices = (a.M + q->rows_per_slice - 1) / q->rows_per_slice;
  size_t off = 0;
  auto take = [&](size_t n) {
    const size_t at = off;
    off = (off + n + 255) & ~size_t(255);
    return at;
  };
  q->bits = take(size_t(a.K) * size_t(a.G) * size_t(a.M) * 16);
  for (int i = 0; i < 2; ++i) {
    q->num[i] = take(size_t(q->slices) * size_t(a.N) * 8);
    q->den[i] = take(size_t(q->slices) * size_t(a.G) * 8);
  }
  q->nm = q->cols = q->pos = q->xc = 0;
  q->cap = 0;
  if (a.mask != nullptr) {
    q->nm = take(size_t(a.G) * 4);
    q->cols = take(size_t(a.G) * size_t(a.g) * 2);
    q->pos = take(size_t(a.N) * 2);
    if (off < bytes) {   // the rest: fp64 copies of up to cap columns of every block
      const size_t per = size_t(a.G) * size_t(a.M) * 8;
      const size_t c = (bytes - off) / per;
      q->cap = int32_t(c > 64 ? 64 : c);
      q->xc = off;
    }
  }
  return off <= bytes;
}

template <int K, int KB, RcMode MODE>
void rc_launch(const RcPass& p, bool list, hipStream_t stream) {
  const dim3 grid(unsigned(p.a.G), unsigned(p.slices)), block(64 * kRcWaves);
  if (list)
    hipLaunchKernelGGL((k_rc_pass_list<K, KB, MODE>), grid, block, 0, stream, p);
  else
    hipLaunchKernelGGL((k_rc_pass<K, KB, MODE>), grid, block, 0, stream, p);
}

template <int K>
void rc_fused(const RcArgs& a, const RcPlan& q, int T, uint8_t* ws, uint32_t* d_signs, hipStream_t stream) {
  RcPass p{};
  p.a = a;
  p.bits = reinterpret_cast<uint64_t*>(ws + q.bits);
  p.rows_per_slice = q.rows_per_slice;
  p.slices = q.slices;
  const bool masked = a.mask != nullptr, list = masked || a.pB != nullptr;
  int32_t* nm = reinterpret_cast<int32_t*>(ws + q.nm);
  uint16_t* cols = reinterpret_cast<uint16_t*>(ws + q.cols);
  uint16_t* pos = reinterpret_cast<uint16_t*>(ws + q.pos);
  if (masked) {
    p.nm = nm;
    p.cols = cols;
    hipLaunchKernelGGL(k_rc_list, dim3(unsigned(a.G)), dim3(kRcMaxG), 0, stream, a, nm, cols, pos);
    if (q.cap > 0) {
      double* xc = reinterpret_cast<double*>(ws + q.xc);
      p.xc = xc;
      p.cap = q.cap;
      hipLaunchKernelGGL(k_rc_copy, dim3(grid_for(a.M * 8, 256), unsigned(a.G)), dim3(256), 0, stream, a, nm, cols, q.cap,
                         xc);
    }
  }
  int turn = 0;
  auto buffers = [&](int kprev) {
    p.kprev = kprev;
    p.num_in = reinterpret_cast<double*>(ws + q.num[turn]);
    p.den_in = reinterpret_cast<double*>(ws + q.den[turn]);
    turn ^= 1;
    p.num_out = reinterpret_cast<double*>(ws + q.num[turn]);
    p.den_out = reinterpret_cast<double*>(ws + q.den[turn]);
  };
  auto init = [&](auto kb) {
    constexpr int KB = decltype(kb)::value;
    if constexpr (KB < K) {
      buffers(KB - 1);
      rc_launch<K, KB, kRcInit>(p, list, stream);
    }
  };
  auto round = [&](auto kb) {
    constexpr int KB = decltype(kb)::value;
    if constexpr (KB < K) {
      buffers(KB == 0 ? K - 1 : KB - 1);
      rc_launch<K, KB, kRcRound>(p, list, stream);
    }
  };
  using std::integral_constant;
  init(integral_constant<int, 0>());
  init(integral_constant<int, 1>());
  init(integral_constant<int, 2>());
  init(integral_constant<int, 3>());
  for (int t = 0; t < T; ++t) {
    if (t == 0) {
      round(integral_constant<int, 0>());
    } else {
      buffers(K - 1);
      rc_launch<K, 0, kRcSignRound>(p, list, stream);
    }
    round(integral_constant<int, 1>());
    round(integral_constant<int, 2>());
    round(integral_constant<int, 3>());
  }
  buffers(K - 1);   // the last column scales, and the last round's signs
  if (T > 0)
    rc_launch<K, 0, kRcSign>(p, list, stream);
  else
    hipLaunchKernelGGL(k_rc_last_scales<K>, dim3(unsigned(a.G)), dim3(64 * kRcWaves), 0, stream, p);
  if (a.g % 32 == 0)
    hipLaunchKernelGGL(k_rc_planes_blocks, dim3(grid_for(a.M, 256), unsigned(a.G), unsigned(K)), dim3(256), 0, stream, a,
                       p.bits, p.nm, p.cols, d_signs);
  else
    hipLaunchKernelGGL(k_rc_planes, dim3(grid_for(int64_t(K) * a.M * ((a.N + 31) / 32), 256)), dim3(256), 0, stream, a,
                       p.bits, masked ? pos : nullptr, d_signs);
}

}  // namespace

}  // namespace fluxbin

using namespace fluxbin;

extern "C" {

fluxbin_status fluxbin_rc_workspace_query(int64_t M, int64_t N, int32_t K, size_t* bytes) {
  clear_error();
  if (!bytes) return fail(FLUXBIN_ERR_INVALID_ARG, "bytes is NULL");
  if (M < 1 || N < 1 || K < 1 || K > 4) return fail(FLUXBIN_ERR_INVALID_ARG, "M, N >= 1 and K in 1..4 required");
  // int8 signs [K][M][N], then (256-byte aligned) the column-scale partial sums [slices][2][N] fp64
  *bytes = ((size_t(K) * size_t(M) * size_t(N) + 255) & ~size_t(255)) + size_t(col_slices(M)) * 2 * size_t(N) * 8;
  return FLUXBIN_OK;
}

fluxbin_status fluxbin_rc_decompose(const float* d_X, const uint8_t* d_mask, const uint32_t* d_prior_signs,
                                    const double* d_prior_alpha_r, const double* d_prior_alpha_c, int32_t Kp,
                                    int64_t gp, int64_t M, int64_t N, int32_t K, int32_t T, int64_t g, double eps,
                                    uint32_t* d_signs, double* d_alpha_r, double* d_alpha_c, void* d_ws,
                                    size_t ws_bytes, hipStream_t stream) {
  size_t need = 0;
  fluxbin_status st = fluxbin_rc_workspace_query(M, N, K, &need);
  if (st != FLUXBIN_OK) return st;
  if (!d_X || !d_signs || !d_alpha_r || !d_alpha_c || !d_ws)
    return fail(FLUXBIN_ERR_INVALID_ARG, "a required pointer is NULL");
  if (T < 0 || g < 1 || !(eps >= 0.0)) return fail(FLUXBIN_ERR_INVALID_ARG, "T >= 0, g >= 1 and eps >= 0 required");
  if (d_prior_signs && (!d_prior_alpha_r || !d_prior_alpha_c || Kp < 1 || Kp > 4 || gp < 1))
    return fail(FLUXBIN_ERR_INVALID_ARG, "prior bases need their scales, Kp in 1..4 and gp >= 1");
  if (M * N > (int64_t(1) << 36)) return fail(FLUXBIN_ERR_UNSUPPORTED, "matrix of %lld elements too large",
                                              (long long)(M * N));
  if (ws_bytes < need)
    return fail(FLUXBIN_ERR_BUFFER_TOO_SMALL, "workspace has %zu bytes, needs %zu", ws_bytes, need);
  RcArgs a{};
  a.X = d_X;
  a.mask = d_mask;
  a.B = static_cast<int8_t*>(d_ws);
  a.ar = d_alpha_r;
  a.ac = d_alpha_c;
  a.M = M;
  a.N = N;
  a.g = g;
  a.G = (N + g - 1) / g;
  a.K = K;
  a.eps = eps;
  a.pB = d_prior_signs;
  a.par = d_prior_alpha_r;
  a.pac = d_prior_alpha_c;
  a.Kp = d_prior_signs ? Kp : 0;
  a.pg = d_prior_signs ? gp : 1;
  a.pG = (N + a.pg - 1) / a.pg;
  a.pW = (N + 31) / 32;
  RcPlan plan;
  if (rc_plan(a, need, &plan)) {   // by the queried size: the same kernels for any larger workspace
    uint8_t* ws = static_cast<uint8_t*>(d_ws);
    switch (K) {
      case 1: rc_fused<1>(a, plan, T, ws, d_signs, stream); break;
      case 2: rc_fused<2>(a, plan, T, ws, d_signs, stream); break;
      case 3: rc_fused<3>(a, plan, T, ws, d_signs, stream); break;
      default: rc_fused<4>(a, plan, T, ws, d_signs, stream); break;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "launching the decomposition kernels");
    return FLUXBIN_OK;
  }
  const int64_t elems = M * N;
  const int64_t slices = col_slices(M);
  const int64_t rows_per_slice = (M + slices - 1) / slices;
  double* part = reinterpret_cast<double*>(static_cast<char*>(d_ws) +
                                           ((size_t(K) * size_t(M) * size_t(N) + 255) & ~size_t(255)));
  const dim3 col_grid(grid_for(N, 64), unsigned(slices));
  for (int k = 0; k < K; ++k) {
    hipLaunchKernelGGL(k_rc_fill, dim3(grid_for(N, 256)), dim3(256), 0, stream, d_alpha_c + int64_t(k) * N, N, 1.0);
    hipLaunchKernelGGL(k_rc_init_sign, dim3(grid_for(elems, 256)), dim3(256), 0, stream, a, k);
    hipLaunchKernelGGL(k_rc_row, dim3(grid_for(M * a.G, 4)), dim3(256), 0, stream, a, k, 1);
    hipLaunchKernelGGL(k_rc_col, col_grid, dim3(256), 0, stream, a, k, 1, rows_per_slice, part);
    hipLaunchKernelGGL(k_rc_col_fin, dim3(grid_for(N, 256)), dim3(256), 0, stream, a, k, slices, part);
  }
  for (int t = 0; t < T; ++t) {
    for (int k = 0; k < K; ++k) {
      hipLaunchKernelGGL(k_rc_row, dim3(grid_for(M * a.G, 4)), dim3(256), 0, stream, a, k, 0);
      hipLaunchKernelGGL(k_rc_col, col_grid, dim3(256), 0, stream, a, k, 0, rows_per_slice, part);
      hipLaunchKernelGGL(k_rc_col_fin, dim3(grid_for(N, 256)), dim3(256), 0, stream, a, k, slices, part);
    }
    switch (K) {
      case 1: hipLaunchKernelGGL(k_rc_sign<1>, dim3(grid_for(elems, 256)), dim3(256), 0, stream, a); break;
      case 2: hipLaunchKernelGGL(k_rc_sign<2>, dim3(grid_for(elems, 256)), dim3(256), 0, stream, a); break;
      case 3: hipLaunchKernelGGL(k_rc_sign<3>, dim3(grid_for(elems, 256)), dim3(256), 0, stream, a); break;
      default: hipLaunchKernelGGL(k_rc_sign<4>, dim3(grid_for(elems, 256)), dim3(256), 0, stream, a); break;
    }
  }
  const int64_t words = int64_t(K) * M * ((N + 31) / 32);
  hipLaunchKernelGGL(k_rc_bits, dim3(grid_for(words, 256)), dim3(256), 0, stream, a, d_signs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "launching the decomposition kernels");
  return FLUXBIN_OK;
}

fluxbin_status fluxbin_structural_search(const float* d_W, const double* d_hinv_diag, int64_t M, int64_t N,
                                         int64_t g, int64_t s, double* d_scores, int32_t* d_sal_idx,
                                         uint8_t* d_mask, hipStream_t stream) {
  clear_error();
  if (!d_W || !d_hinv_diag || !d_scores || !d_sal_idx) return fail(FLUXBIN_ERR_INVALID_ARG, "a pointer is NULL");
  if (M < 1 || N < 1 || g < 1 || s < 1) return fail(FLUXBIN_ERR_INVALID_ARG, "M, N, g, s >= 1 required");
  if (g > 1024) return fail(FLUXBIN_ERR_UNSUPPORTED, "group of %lld columns > 1024", (long long)g);
  if (s > g) return fail(FLUXBIN_ERR_INVALID_ARG, "s = %lld > g = %lld", (long long)s, (long long)g);
  if (M * N > (int64_t(1) << 36)) return fail(FLUXBIN_ERR_UNSUPPORTED, "matrix too large");
  const auto saliency = [&](auto kernel, int c, int slices) {
    hipLaunchKernelGGL(kernel, dim3(grid_for(N, c)), dim3(unsigned(c * slices)), 0, stream, d_W, d_hinv_diag, M, N, d_scores);
  };
  if (N < 64 * int64_t(device_cu_count()))
    saliency(k_saliency<16, 64>, 16, 64);
  else if (M > 256)
    saliency(k_saliency<64, 16>, 64, 16);
  else
    saliency(k_saliency<64, 4>, 64, 4);
  hipLaunchKernelGGL(k_topk, dim3(unsigned((N + g - 1) / g)), dim3(1024), 0, stream, d_scores, N, g, s, d_sal_idx,
                     d_mask);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "launching the saliency kernels");
  return FLUXBIN_OK;
}

}  // extern "C"
