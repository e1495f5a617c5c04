// Small-batch (B = 2..16) product of libfluxbin on the block-scaled matrix instructions of gfx950.
//
// What is computed is the other kernels' product (Eqs. 10-11 and 15), for every batch row b < B:
//   y[b, i] = sum_c rscale[plane(c)][i] * sum_{v in chunk c} s(i, v) * p[b, v],   p[b, v] = colscale[v] * x[b, xidx[v]].
// A chunk's inner sum is a (rows x 128) block of +-1 times a (128 x B) block of fp32 products. Both operands of
// v_mfma_scale_f32_16x16x128_f8f6f4 can be narrow: the signs are fp4 values (+-1.0, eight per register), and each
// product p is written as a sum of base-32 digits held in fp6 (e2m3), every 32-column block of a digit with its own
// power-of-two scale (the instruction's E8M0 block scale). One instruction then covers a whole chunk of 16 rows for 16
// (digit, batch row) columns.
//
// Why: decoding the signs bounded the fp16 form of this product (fluxbin_gemm_mfma.hip): two sign bits per operand
// register, 1.5 vector instructions each. fp4 takes eight sign bits per register, a shift and one bit operation
// (v_bitop3_b32): 7 instructions per lane for 16 rows x 128 columns instead of 24. Measured instruction rates (gfx950,
// one SIMD, cycles at 2.4 GHz): 16x16x128 fp4 x fp6 with scales 19, 16x16x32 f16 16.9 (a quarter of the columns).
//
// Precision. p is exact in fp32 (two 11-bit significands). Digit d of a 32-column block is p's remainder rounded to
// fp6 at scale 2^(E - 1 - 5 d), E the exponent of the block's largest |p|: magnitudes up to 4, rounded to 2^-3 of the
// scale at most. After six digits the remainder is at most 2^-29 of the block's largest |p|, after the five of 9 to 16
// batch rows on layers with one row scale per chunk (five instructions instead of six) 2^-24 (an fp32 sum rounds at 2^-24
// of its running value). Digit products +-q are exact, and they are summed in the matrix core's fp32 accumulation; row
// scale and chunk order are as in the other kernels. Error against 64 bits, relative to that of the kernel it takes over
// from, on normal, outlier, widely spread, lognormal, positive and sparse activations and on blocks with one product
// thousands of times the others: five digits 0.56 to 0.93 of the fp16 form's, six 0.48 to 0.97; on layers with fine salient
// groups 0.54 to 0.80 of the generic kernel's and 0.62 to 0.92 of the batch-1 launches'. Blocks with an infinity or NaN (in
// x or in a column scale) get zero digits and a mark, and are added by scalar fp32 code after the matrix instructions.
//
// Work decomposition. A wavefront owns RB 16-row blocks and takes every W-th chunk of its workgroup's part of the
// chunks: one 16-byte load per lane brings 64 rows' entries, four 16 x 128 sign tiles. Un-rotating an entry
// is a 128-bit rotation by a per-lane amount (four funnel shifts, eight selects), and a 4 x 4 transpose between the
// registers and the 16-lane groups (four v_permlane swaps) leaves each tile in matrix operand order: no LDS. The
// digits of a chunk are read from an image that a first kernel (k_mx_image) writes once per call to the workspace.
// A wavefront's loads of them (1.6 KB per instruction and chunk, from the XCD's L2) are shared by its RB tiles only, so
// RB = 8; 4 on layers with fine salient groups, whose chunks' sums need the registers. Wavefronts run independently,
// without barriers; at the end their sums are added through LDS in wavefront order, and with parts > 1 workgroups per row
// tile their sums by a second kernel in part order: deterministic.
#include "fluxbin_device.h"
#include "fluxbin_signs.h"

namespace fluxbin {

namespace {

typedef int mx_i32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t mx_u32x2 __attribute__((ext_vector_type(2)));
typedef sign_u32x4 mx_u32x4;
typedef uint32_t mx_u32x6 __attribute__((ext_vector_type(6)));
typedef float mx_f32x4 __attribute__((ext_vector_type(4)));
typedef float mx_f32x16 __attribute__((ext_vector_type(16)));
typedef float mx_f32x32 __attribute__((ext_vector_type(32)));

constexpr int kDigits = mx_digits(1, true);   // of the fine groups' results (any number of batch rows)
constexpr uint32_t kMxOdd = 0x80000000u;   // in a lane's last scale word, whose top byte no instruction uses

// Digits per instruction and instructions per chunk with nbp padded batch rows (2, 4, 8 or 16): operand row m of
// instruction t holds digit t * (16 / nbp) + m / nbp of batch row m mod nbp.
template <int NBP, bool FINE>
constexpr int mx_t() { return mx_instr(NBP, FINE); }

// ---------------------------------------------------------------------------------------------------------------------
// Image: per chunk T digit operands (64 lanes x 16 bytes, then 64 lanes x 8 bytes each) and the lanes' block scales.
// ---------------------------------------------------------------------------------------------------------------------

// 32 fp32 values to fp6 (e2m3) divided by `scale` (a power of two), rounded to nearest even; value 2i from lo[i],
// 2i + 1 from hi[i]. Written as an instruction: its destination must not overlap its sources (it is written before all
// of them are read), which the compiler's own form does not ensure.
__device__ __forceinline__ mx_u32x6 mx_to_fp6(const mx_f32x16& lo, const mx_f32x16& hi, float scale) {
  mx_u32x6 r;
  asm("v_cvt_scalef32_2xpk16_fp6_f32 %0, %1, %2, %3" : "=&v"(r) : "v"(lo), "v"(hi), "v"(scale));
  return r;
}

// One thread per (chunk, 32-column block g, padded batch row): all digits of its 32 products. Batch rows past B, columns
// without a source and digits past the last are zero. Bound by latency: column scales and activations in one round trip
// (salient chunks: the indices in another before it), then about 400 instructions.
template <int NBP, bool FINE>
__global__ void __launch_bounds__(64) k_mx_image(GemmArgs a, int x_aligned) {
  constexpr int ND = mx_digits(NBP, FINE), T = mx_t<NBP, FINE>(), DP = 16 / NBP;
  const int tid = int(blockIdx.x) * 64 + int(threadIdx.x);
  const int b = tid & (NBP - 1), g = (tid / NBP) & 3, c = tid / (4 * NBP);
  if (c >= a.NCP) return;
  const mx_u32x4* cc = reinterpret_cast<const mx_u32x4*>(a.colscale + c * kChunk + 32 * g);
  const uint16_t* x = a.x + int64_t(b < a.B ? b : 0) * a.ldx;
  mx_u32x4 cw[4], xw[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) cw[k] = cc[k];
  uint32_t none = 0;   // columns without a source
  const int j0 = (c % a.ncg) * kChunk + 32 * g;
  if (c < a.ngc && x_aligned != 0 && j0 + 32 <= a.N) {   // 16-byte aligned rows, a block inside the row: wide loads
#pragma unroll
    for (int k = 0; k < 4; ++k) xw[k] = reinterpret_cast<const mx_u32x4*>(x + j0)[k];
  } else {
    uint32_t xi[32];
    if (c < a.ngc) {
#pragma unroll
      for (int col = 0; col < 32; ++col) xi[col] = j0 + col < a.N ? uint32_t(j0 + col) : 0xFFFFu;
    } else {
      const mx_u32x4* ci = reinterpret_cast<const mx_u32x4*>(a.xidx + c * kChunk + 32 * g);
      mx_u32x4 iw[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) iw[k] = ci[k];
#pragma unroll
      for (int col = 0; col < 32; ++col) xi[col] = (iw[col >> 3][(col >> 1) & 3] >> (16 * (col & 1))) & 0xFFFFu;
    }
    uint16_t xv[32];
#pragma unroll
    for (int col = 0; col < 32; ++col) {   // unconditional: the loads are in flight together
      xv[col] = x[xi[col] == 0xFFFFu ? 0 : xi[col]];
      none |= xi[col] == 0xFFFFu ? 1u << col : 0u;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) xw[k >> 2][k & 3] = uint32_t(xv[2 * k]) | (uint32_t(xv[2 * k + 1]) << 16);
  }
  if (b >= a.B) none = ~0u;
  // element e of the operand is the block's column 4 (e mod 8) + e / 8: the order in which a word's sign bits come out
  // of the decode's four shifts
  mx_f32x16 lo, hi;
  uint32_t top = 0;
#pragma unroll
  for (int col = 0; col < 32; ++col) {
    const int sh = 16 * (col & 1);
    float p = h2f(uint16_t(cw[col >> 3][(col >> 1) & 3] >> sh)) * h2f(uint16_t(xw[col >> 3][(col >> 1) & 3] >> sh));
    p = (none >> col) & 1u ? 0.f : p;
    const uint32_t mag = __builtin_bit_cast(uint32_t, p) & 0x7FFFFFFFu;
    top = mag > top ? mag : top;
    const int e = 8 * (col & 3) + (col >> 2);
    if (e & 1)
      hi[e >> 1] = p;
    else
      lo[e >> 1] = p;
  }
  const bool odd = top >= 0x7F800000u;   // an infinity or a NaN: left to mx_add_odd
  if (odd) {
#pragma unroll
    for (int i = 0; i < 16; ++i) lo[i] = hi[i] = 0.f;
  }
  // exponent of digit 0's scale: the largest |p| is in [2, 4) of it (all zero: any)
  const uint32_t e0 = top < 0x10000000u || odd ? 100u : (top >> 23) - 1u;
  uint8_t* img = reinterpret_cast<uint8_t*>(a.img) + int64_t(c) * mx_chunk_bytes(T);
#pragma unroll
  for (int d = 0; d < T * DP; ++d) {
    const int t = d / DP, lane = b + NBP * (d % DP) + 16 * g;
    mx_u32x6 q = {0, 0, 0, 0, 0, 0};
    if (d < ND) {
      const float sc = __builtin_bit_cast(float, (e0 - 5u * uint32_t(d)) << 23);
      q = mx_to_fp6(lo, hi, sc);
      if (d + 1 < ND) {
        const mx_f32x32 back = __builtin_amdgcn_cvt_scalef32_pk32_f32_fp6(q, sc);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          lo[i] -= back[2 * i];
          hi[i] -= back[2 * i + 1];
        }
      }
    }
    *reinterpret_cast<mx_u32x4*>(img + t * 1024 + lane * 16) = mx_u32x4{q[0], q[1], q[2], q[3]};
    *reinterpret_cast<mx_u32x2*>(img + T * 1024 + t * 512 + lane * 8) = mx_u32x2{q[4], q[5]};
  }
  // the lanes' scale bytes, one per instruction, and in the top byte the mark of an odd block
#pragma unroll
  for (int dd = 0; dd < DP; ++dd) {
    uint32_t w[2] = {0, 0};
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int d = t * DP + dd;
      w[t >> 2] |= (e0 - 5u * uint32_t(d < ND ? d : 0)) << (8 * (t & 3));
    }
    if (odd && dd == 0) w[T > 4 ? 1 : 0] |= kMxOdd;
    uint32_t* dst = reinterpret_cast<uint32_t*>(img + T * 1536) + (b + NBP * dd + 16 * g) * (T > 4 ? 2 : 1);
    dst[0] = w[0];
    if constexpr (T > 4) dst[1] = w[1];
  }
}

// ---------------------------------------------------------------------------------------------------------------------
// Product
// ---------------------------------------------------------------------------------------------------------------------

template <int T>
struct MxOperand {
  mx_i32x8 q[T];   // six registers used
  uint32_t sc[T > 4 ? 2 : 1];
};

template <int T>
__device__ __forceinline__ void mx_load_operand(const GemmArgs& a, int c, int lane, MxOperand<T>& o) {
  const uint8_t* img = reinterpret_cast<const uint8_t*>(a.img) + int64_t(c) * mx_chunk_bytes(T);
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const mx_u32x4 lo = *reinterpret_cast<const mx_u32x4*>(img + t * 1024 + lane * 16);
    const mx_u32x2 hi = *reinterpret_cast<const mx_u32x2*>(img + T * 1024 + t * 512 + lane * 8);
    o.q[t] = mx_i32x8{int(lo[0]), int(lo[1]), int(lo[2]), int(lo[3]), int(hi[0]), int(hi[1]), 0, 0};
  }
  const uint32_t* sc = reinterpret_cast<const uint32_t*>(img + T * 1536);
  if constexpr (T > 4) {
    const mx_u32x2 v = *reinterpret_cast<const mx_u32x2*>(sc + 2 * lane);
    o.sc[0] = v[0];
    o.sc[1] = v[1];
  } else {
    o.sc[0] = sc[lane];
  }
}

// The sign words of two tiles -> their fp4 operands: +1.0 (0x2) for a set bit, -1.0 (0xA) for a clear one; register j,
// nibble n holds bit 4 n + j (the bits a 64-bit shift pushes from one word into the other land below bit 3).
__device__ __forceinline__ void mx_signs(uint32_t w0, uint32_t w1, mx_i32x8& s0, mx_i32x8& s1) {
  const uint64_t w = (uint64_t(w1) << 32) | w0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint64_t v = j < 3 ? sign_shl64(w, 3 - j) : w;
    s0[j] = int((~uint32_t(v) & 0x88888888u) | 0x22222222u);
    s1[j] = int((~uint32_t(v >> 32) & 0x88888888u) | 0x22222222u);
  }
}

// One tile's (16 rows x 128 columns) inner sums: lane (row n, g) gets operand rows 4 g .. 4 g + 3. The instruction's two
// scale operands are a byte of a register each: the digits' block scales and 1.0 (127).
template <int T>
__device__ __forceinline__ mx_f32x4 mx_mul(const MxOperand<T>& o, int t, const mx_i32x8& s, const mx_f32x4& d) {
  const int sc = int(o.sc[t >> 2]);
  switch (t & 3) {
    case 0: return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(o.q[t], s, d, 2, 4, 0, sc, 0, 127);
    case 1: return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(o.q[t], s, d, 2, 4, 1, sc, 0, 127);
    case 2: return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(o.q[t], s, d, 2, 4, 2, sc, 0, 127);
    default: return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(o.q[t], s, d, 2, 4, 3, sc, 0, 127);
  }
}

// Operand register masks of a chunk with FG fine row-scale groups: a lane of operand row m keeps the columns of group
// m mod FG that its 32-column block g holds (element 8 j + n is column 4 n + j of the block).
template <int FG>
__device__ __forceinline__ void mx_fine_masks(int lane, uint32_t (&mask)[6]) {
  constexpr int GC = kChunk / FG;   // columns of a group: 8 or 16
  const int u = lane & (FG - 1), g = lane >> 4;
  const int first = u * GC - 32 * g;   // the group's first column within the block, if it holds it
  const bool in = first >= 0 && first < 32;
  // columns first .. first + GC - 1 are elements 8 j + first / 4 .. + GC / 4 - 1, six bits each
  const uint64_t run = in ? ((uint64_t(1) << (6 * (GC / 4))) - 1) << (6 * (first / 4)) : 0;   // within 48 bits
  const uint64_t a = run | (run << 48), b = (run >> 16) | (run << 32), c = (run >> 32) | (run << 16);
  mask[0] = uint32_t(a);
  mask[1] = uint32_t(a >> 32);
  mask[2] = uint32_t(b);
  mask[3] = uint32_t(b >> 32);
  mask[4] = uint32_t(c);
  mask[5] = uint32_t(c >> 32);
}

// Bit position of canonical bit u of a chunk in row's packed entry. FG > 0: a chunk with FG fine row-scale groups.
template <int MU, int FG>
__device__ __forceinline__ int mx_stored_bit(int u, int row) {
  if constexpr (FG == 8) {   // pairs of sub-vectors: the pairs rotated by row / 2, a pair's two swapped on odd rows
    const int sub = u >> 3;
    return ((((sub >> 1) - (row >> 1)) & 7) * 2 + ((sub - row) & 1)) * 8 + (u & 7);
  }
  return (u - MU * row) & 127;
}

// Adds a chunk's odd blocks (an infinity or NaN among a batch row's 32 products) of batch rows b0 .. b1-1 to the
// wavefront's sums red[m][row], in fp32: lane (n, g) takes 8 of a block's columns of row n of each row block.
template <int MU, int T, int FG>
__device__ __forceinline__ void mx_add_odd(const GemmArgs& a, int c, int b0, int b1, int row0, int n_rb, int lane,
                                           float* red, int rs) {
  const uint32_t* sc = reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(a.img) +
                                                         int64_t(c) * mx_chunk_bytes(T) + T * 1536);
  uint64_t marks = __builtin_amdgcn_ballot_w64((sc[T > 4 ? 2 * lane + 1 : lane] & kMxOdd) != 0 && (lane & 15) >= b0 &&
                                               (lane & 15) < b1);
  while (marks != 0) {
    const int l = __builtin_ctzll(marks), b = l & 15, u0 = 32 * (l >> 4) + 8 * (lane >> 4), v0 = c * kChunk + u0;
    marks &= marks - 1;
    for (int rb = 0; rb < n_rb; ++rb) {
      int row = row0 + 16 * rb + (lane & 15);
      row = row < a.Mp ? row : a.Mp - 1;
      const int64_t slot = MU == 8 ? ((c & 1) ^ ((row >> 4) & 1)) : (c & 1);
      const uint8_t* e = a.signs + ((int64_t(c >> 1) * 2 + slot) * a.Mp + row) * 16;
      float sum = 0.f;
      for (int k = 0; k < 8; ++k) {
        const uint32_t xi = a.xidx[v0 + k];
        if (xi == 0xFFFFu) continue;
        const int bit = mx_stored_bit<MU, FG>(u0 + k, row);
        const float p = h2f(a.colscale[v0 + k]) * h2f(a.x[b * a.ldx + xi]);
        sum += ((e[bit >> 3] >> (bit & 7)) & 1) != 0 ? p : -p;
      }
      const int64_t plane = int64_t(a.chunk_plane[c]) * a.Mp;
      if constexpr (FG == 0)
        sum *= h2f(a.rscale[plane + row]);
      else
        sum *= h2f(a.rscale[plane + int64_t(row) * FG + ((u0 / (kChunk / FG) - row / (16 / FG)) & (FG - 1))]);
      sum += __shfl_xor(sum, 16, 64);
      sum += __shfl_xor(sum, 32, 64);
      if (lane < 16) red[b * rs + 16 * rb + lane] += sum;
    }
  }
}

// The digits of batch row b's column block (the lane's lane >> 4) of chunk c, and its scale bytes and mark.
template <int NBP>
struct MxFineOperand {
  mx_i32x8 q[kDigits];   // six registers used
  uint32_t sc[2], mark;
};

template <int NBP>
__device__ __forceinline__ void mx_load_fine(const GemmArgs& a, int c, int b, int lane, MxFineOperand<NBP>& o) {
  constexpr int T = mx_t<NBP, true>(), DP = 16 / NBP;
  const uint8_t* img = reinterpret_cast<const uint8_t*>(a.img) + int64_t(c) * mx_chunk_bytes(T);
#pragma unroll
  for (int d = 0; d < kDigits; ++d) {
    const int t = d / DP, src = b + NBP * (d % DP) + (lane & 48);
    const mx_u32x4 lo = *reinterpret_cast<const mx_u32x4*>(img + t * 1024 + src * 16);
    const mx_u32x2 hi = *reinterpret_cast<const mx_u32x2*>(img + T * 1024 + t * 512 + src * 8);
    o.q[d] = mx_i32x8{int(lo[0]), int(lo[1]), int(lo[2]), int(lo[3]), int(hi[0]), int(hi[1]), 0, 0};
  }
  const uint32_t* sc = reinterpret_cast<const uint32_t*>(img + T * 1536) + (b + (lane & 48)) * (T > 4 ? 2 : 1);
  o.sc[0] = sc[0];
  o.mark = sc[T > 4 ? 1 : 0];
}

template <int NL>
struct MxSigns {
  mx_u32x4 e[NL];
  uint32_t rs[NL];
};

// Grid (row tiles, parts); W wavefronts. With several parts their sums go to a.partials, float [parts][B][Mp]. 28672x8192
// with 3 bases + 5% on one 256-CU device, us per call (three kernels fp16 -> image and this one): B = 8 48.1 -> 38.3.
//
// FG = 8 or 16 (mu = 8, RB = 4): layers whose salient chunks (from chunk nfc on) have FG row scales per row, one per 16
// or 8 columns (the paper's s16 and s8 configurations). There the 16 operand rows of an instruction are the FG groups of
// one or two batch rows (the operand masked to each group's columns), its six digits accumulate into one result, and
// each group's sum is multiplied by its scale: FG / 16 of the instructions per batch row instead of 1 / 16, on the few
// salient chunks. A quarter of the wavefronts takes a quarter of the batch rows, so that a layer's few such chunks
// are spread over enough wavefronts.
template <int MU, int NBP, int RB, int W, int FG>
__global__ void __launch_bounds__(64 * W) k_gemm_mx(GemmArgs a, int parts) {
  constexpr int T = mx_t<NBP, (FG > 0)>();
  static_assert(RB == 4 || RB == 8, "whole loads of four row blocks");
  constexpr int NL = RB / 4;         // loads per chunk
  // Chunks requested ahead: 4 KB (and the row scales) per wavefront. As compiled, 14 of the 16 instances wait for all
  // outstanding loads at the head of the loop over groups of D chunks (the loop may be left in the middle of a group, where
  // the last loads issued are the next ones used), the other two for all but two or three: the loads in flight drain once
  // per group.
  constexpr int D = 4 / NL;
  constexpr int RS = 16 * RB + 4;    // LDS row stride: the four lane groups' stores in different banks
  __shared__ float red[W][16][RS];
  const int lane = int(threadIdx.x) & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int n = lane & 15, q4 = lane >> 4;
  const int row0 = int(blockIdx.x) * 16 * RB;

  // this workgroup's part of the chunks with one row scale, and the wavefront's: c0 + wave, c0 + wave + W, ...
  const int ncc = FG > 0 ? a.nfc : a.NCP;
  const int c0 = ncc * int(blockIdx.y) / parts, c1 = ncc * int(blockIdx.y + 1) / parts;
  const int steps = (c1 - c0 - wave + W - 1) / W;   // may be <= 0

  // the row of the lane's entry of load l (rows past the padded rows read the last padded row; never stored)
  uint32_t rows[NL];
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    const int r = row0 + 64 * l + lane;
    rows[l] = uint32_t(r < a.Mp ? r : a.Mp - 1);
  }
  const int64_t plane_bytes = int64_t(a.Mp) * 16;
  const SignRot rot = sign_rot<MU>(rows[0]);   // the same for the rows of every load (64 rows apart)

  auto load_signs = [&](int c, int32_t plane, MxSigns<NL>& s) __attribute__((always_inline)) {
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      const uint32_t swap = MU == 8 ? (rows[l] >> 4) & 1u : 0u;
      const uint8_t* p = a.signs + int64_t(c & ~1) * plane_bytes + ((uint32_t(c & 1) ^ swap) ? plane_bytes : 0) +
                         rows[l] * 16u;
      s.e[l] = __builtin_nontemporal_load(reinterpret_cast<const mx_u32x4*>(p));
      s.rs[l] = a.rscale[int64_t(plane) * a.Mp + rows[l]];
    }
  };

  mx_f32x4 acc[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) acc[rb] = mx_f32x4{0.f, 0.f, 0.f, 0.f};

  uint32_t odd = 0;   // the marks of the operands used
  auto step = [&](int s, MxSigns<NL>& cur, MxOperand<T>& o, MxOperand<T>& on) __attribute__((always_inline)) {
    const int c = c0 + wave + s * W;
    const int cd = s + D < steps ? c + D * W : c, cn = s + 1 < steps ? c + W : c;
    const int32_t plane = load_uniform_i32(a.chunk_plane, cd);
    // canonical words and row scales of the chunk's RB tiles
    uint32_t w[NL][4], rs[4];
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      sign_unrotate(cur.e[l], rot, w[l]);
      sign_transpose(w[l]);
    }
    sign_broadcast(NL > 1 ? cur.rs[0] | (cur.rs[NL - 1] << 16) : cur.rs[0], rs);
    // the next chunk's digits first, then the signs D chunks ahead (within a group): loads return in order
    mx_load_operand<T>(a, cn, lane, on);
    load_signs(cd, plane, cur);
    asm volatile("" ::: "memory");   // the loads are issued here, not where their values are first used
    odd |= o.sc[T > 4 ? 1 : 0];
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      mx_i32x8 sgn[4] = {};
      mx_signs(w[l][0], w[l][1], sgn[0], sgn[1]);
      mx_signs(w[l][2], w[l][3], sgn[2], sgn[3]);
      mx_f32x4 d[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) d[q] = mx_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) d[q] = mx_mul<T>(o, t, sgn[q], d[q]);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float sc = h2f(uint16_t(rs[q] >> (16 * l)));
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[4 * l + q][i] = __builtin_fmaf(sc, d[q][i], acc[4 * l + q][i]);
      }
    }
  };

  if (steps > 0) {
    MxSigns<NL> sg[D];
    MxOperand<T> op[2];
    const int c = c0 + wave;
    mx_load_operand<T>(a, c, lane, op[0]);
#pragma unroll
    for (int k = 0; k < D; ++k) {
      const int ck = k < steps ? c + k * W : c;
      load_signs(ck, load_uniform_i32(a.chunk_plane, ck), sg[k]);
    }
    for (int s = 0; s < steps; s += D) {
#pragma unroll
      for (int k = 0; k < D; ++k) {
        if (s + k >= steps) break;
        step(s + k, sg[k], op[k & 1], op[(k + 1) & 1]);
      }
    }
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][4 * q4 + i][16 * rb + n] = acc[rb][i];
  if (__builtin_amdgcn_ballot_w64((odd & kMxOdd) != 0) != 0) {
    for (int c = c0 + wave; c < c1; c += W) mx_add_odd<MU, T, 0>(a, c, 0, NBP, row0, RB, lane, &red[wave][0][0], RS);
  }

  constexpr int SB = FG == 8 ? 2 : 1;                 // batch rows of one fine result
  constexpr int SQ = (NBP / SB + 3) / 4;              // results of one wavefront
  constexpr int QB = SQ * SB;                         // its batch rows: QB * (wave & 3) and on
  __shared__ float red_fine[FG > 0 ? W : 1][QB][FG > 0 ? 64 : 1];
  if constexpr (FG > 0) {
    static_assert(MU == 8 && RB == 4 && W % 4 == 0, "fine groups: mu = 8, 64-row workgroups");
    const int nf = a.NCP - ncc, b0 = QB * (wave & 3);
    const int f1 = ncc + nf * int(blockIdx.y + 1) / parts;
    const int fa = ncc + nf * int(blockIdx.y) / parts + (wave >> 2);
    float accf[SQ][4];
#pragma unroll
    for (int k = 0; k < SQ; ++k)
#pragma unroll
      for (int q = 0; q < 4; ++q) accf[k][q] = 0.f;
    uint32_t oddf = 0;
    if (fa < f1 && b0 < NBP) {
      uint32_t mask[6];
      mx_fine_masks<FG>(lane, mask);
      // the un-rotation of the entries: FG = 16 as in the other chunks; FG = 8 by row & ~1, then the bytes of each pair
      // swapped on odd rows
      const SignRot rotf = sign_rot<MU>(FG == 8 ? rows[0] & ~1u : rows[0]);
      const uint32_t pair = FG == 8 && (rows[0] & 1u) != 0 ? 0x02030001u : 0x03020100u;
      const int bl = FG == 8 ? (n >> 3) : 0;   // the lane's batch row within a result
      int64_t rrow[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = row0 + 16 * q + n;
        rrow[q] = r < a.Mp ? r : a.Mp - 1;
      }
      auto load_entry = [&](int c) __attribute__((always_inline)) {
        const uint32_t slot = uint32_t(c & 1) ^ ((rows[0] >> 4) & 1u);
        return __builtin_nontemporal_load(reinterpret_cast<const mx_u32x4*>(
            a.signs + int64_t(c & ~1) * plane_bytes + (slot ? plane_bytes : 0) + rows[0] * 16u));
      };
      auto load_scales = [&](int c, uint16_t (&sc)[4][4]) __attribute__((always_inline)) {
        const uint16_t* base = a.rscale + int64_t(load_uniform_i32(a.chunk_plane, c)) * a.Mp;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            sc[q][i] = base[rrow[q] * FG + ((4 * q4 + i - int(rrow[q]) / (16 / FG)) & (FG - 1))];
      };
      mx_u32x4 ent = load_entry(fa);
      uint16_t rsf[4][4], rsn[4][4];
      load_scales(fa, rsn);
      MxFineOperand<NBP> next;
      mx_load_fine<NBP>(a, fa, b0 + bl, lane, next);
      for (int c = fa; c < f1; c += W / 4) {
        const int cn = c + W / 4 < f1 ? c + W / 4 : c;
        uint32_t w[4];
        sign_unrotate(ent, rotf, w);
        if constexpr (FG == 8) {
#pragma unroll
          for (int m = 0; m < 4; ++m) w[m] = __builtin_amdgcn_perm(w[m], w[m], pair);
        }
        sign_transpose(w);
        mx_i32x8 sgn[4] = {};
        mx_signs(w[0], w[1], sgn[0], sgn[1]);
        mx_signs(w[2], w[3], sgn[2], sgn[3]);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) rsf[q][i] = rsn[q][i];
        ent = load_entry(cn);
        load_scales(cn, rsn);
#pragma unroll
        for (int k = 0; k < SQ; ++k) {
          MxFineOperand<NBP> o = next;
          mx_load_fine<NBP>(a, k + 1 < SQ ? c : cn, b0 + SB * (k + 1 < SQ ? k + 1 : 0) + bl, lane, next);
          asm volatile("" ::: "memory");   // requested before this result's instructions
          oddf |= o.mark;
          const uint32_t e0 = o.sc[0] & 0xFFu;
          // the digits' scale bytes e0 - 5 d
          const int sc0 = int(e0 * 0x01010101u - 0x0F0A0500u), sc1 = int(e0 * 0x0101u - 0x1914u);
#pragma unroll
          for (int d = 0; d < kDigits; ++d)
#pragma unroll
            for (int i = 0; i < 6; ++i) o.q[d][i] &= int(mask[i]);
          mx_f32x4 r[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) r[q] = mx_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            r[q] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(o.q[0], sgn[q], r[q], 2, 4, 0, sc0, 0, 127);
            r[q] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(o.q[1], sgn[q], r[q], 2, 4, 1, sc0, 0, 127);
            r[q] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(o.q[2], sgn[q], r[q], 2, 4, 2, sc0, 0, 127);
            r[q] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(o.q[3], sgn[q], r[q], 2, 4, 3, sc0, 0, 127);
            r[q] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(o.q[4], sgn[q], r[q], 2, 4, 0, sc1, 0, 127);
            r[q] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(o.q[5], sgn[q], r[q], 2, 4, 1, sc1, 0, 127);
          }
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) accf[k][q] = __builtin_fmaf(h2f(rsf[q][i]), r[q][i], accf[k][q]);
        }
      }
    }
    // the lane groups that hold the same batch row's groups
#pragma unroll
    for (int k = 0; k < SQ; ++k)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float v = accf[k][q];
        v += __shfl_xor(v, 16, 64);
        if constexpr (FG == 16) v += __shfl_xor(v, 32, 64);
        if ((q4 & (FG == 16 ? 3 : 1)) == 0) red_fine[wave][k * SB + (q4 >> 1)][16 * q + n] = v;
      }
    if (__builtin_amdgcn_ballot_w64((oddf & kMxOdd) != 0) != 0) {
      for (int c = fa; c < f1; c += W / 4)
        mx_add_odd<MU, T, FG>(a, c, b0, b0 + QB, row0, RB, lane, &red[wave][0][0], RS);
    }
  }
  __syncthreads();
  for (int e = int(threadIdx.x); e < a.B * 16 * RB; e += 64 * W) {
    const int b = e / (16 * RB), r = e - b * 16 * RB, row = row0 + r;
    float v = 0.f;
#pragma unroll
    for (int wv = 0; wv < W; ++wv) {
      // a wavefront's digit sums, the smallest first: their roundings stay below those of the one addition to v (added to
      // v one by one, at two rows 64 additions instead of 8, the results were 1.03 to 1.25 times as far off)
      float u = red[wv][16 - NBP + b][r];
#pragma unroll
      for (int m = 16 - 2 * NBP; m >= 0; m -= NBP) u += red[wv][m + b][r];
      v += u;
    }
    if constexpr (FG > 0) {
#pragma unroll
      for (int wv = 0; wv < W; wv += 4) v += red_fine[wv + b / QB][b % QB][r];
    }
    if (row >= a.M) continue;
    if (parts == 1)
      store_y(a, b, row, v);
    else
      a.partials[(int64_t(blockIdx.y) * a.B + b) * a.Mp + row] = v;
  }
}

template <int MU, int NBP, int FG>
bool launch_mx(const GemmArgs& a, int parts, hipStream_t stream) {
  const int x_aligned = ((reinterpret_cast<uintptr_t>(a.x) | uint64_t(a.ldx) * 2u) & 15u) == 0;
  if (parts < 1 || a.B < 1 || a.B > NBP) return false;
  hipLaunchKernelGGL((k_mx_image<NBP, (FG > 0)>), dim3(unsigned(ceil_div(int64_t(a.NCP) * 4 * NBP, 64))), dim3(64), 0,
                     stream, a, x_aligned);
  constexpr int RB = mx_rows(FG > 0) / 16;
  hipLaunchKernelGGL((k_gemm_mx<MU, NBP, RB, 8, FG>), dim3(unsigned(ceil_div(a.M, 16 * RB)), unsigned(parts)), dim3(512), 0,
                     stream, a, parts);
  if (parts > 1)
    launch_reduce_parts(a, parts, stream);
  return true;
}

template <int MU, int FG>
bool launch_mx_b(const GemmArgs& a, int nbp, int parts, hipStream_t stream) {
  switch (nbp) {
    case 2: return launch_mx<MU, 2, FG>(a, parts, stream);
    case 4: return launch_mx<MU, 4, FG>(a, parts, stream);
    case 8: return launch_mx<MU, 8, FG>(a, parts, stream);
    case 16: return launch_mx<MU, 16, FG>(a, parts, stream);
  }
  return false;
}

}  // namespace

bool launch_gemm_mx(const GemmArgs& a, int nbp, int mu, int fg, int parts, hipStream_t stream) {
  if (mu == 4) return fg == 0 && launch_mx_b<4, 0>(a, nbp, parts, stream);
  switch (fg) {
    case 0: return launch_mx_b<8, 0>(a, nbp, parts, stream);
    case 8: return launch_mx_b<8, 8>(a, nbp, parts, stream);
    case 16: return launch_mx_b<8, 16>(a, nbp, parts, stream);
  }
  return false;
}

}  // namespace fluxbin
