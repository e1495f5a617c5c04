// Many batch rows (prompt processing) on the matrix cores of gfx950.
//
// The product is the other kernels' (Eqs. 10-11 and 15). As in the fp16 small-batch kernel (fluxbin_gemm_mfma.hip) every 32
// columns of a chunk are a v_mfma_f32_16x16x32_f16 of signed column scales (+-alpha_c, exact in fp16) and activations, its
// products exact in the fp32 accumulation, and each chunk's sums are multiplied by the row scales once. There a decoded
// sign operand serves 32 batch rows, so a call of B rows decoded every sign B / 32 times (1.5 vector instructions per
// operand register) and was bound by that. Here it serves 64: a wavefront owns 64 rows x 64 batch rows, and the
// activation operands of a column block stay in registers for all the bases that read it.
//
// Work decomposition. A workgroup of four wavefronts takes 256 rows x 64 batch rows and a part of the column blocks (128
// columns of the global bases, or 128 dense salient columns): per column block the activations (16 KB) and the
// column-scale pairs of its bases go to LDS from images that a first kernel writes once per call, requested in the first
// step of the column block before; every base's chunk is one step: a 16-byte load per lane brings the chunk's 64 rows (one
// step ahead: a step takes the signs out of their registers before it requests the next), an un-rotation and a 4 x 4
// transpose put them into operand order, and 64 matrix instructions and 64 row-scale FMAs per lane follow: 1080 cycles of
// matrix work, about 830 of vector work. With parts > 1 the parts' sums are added by a second
// kernel in part order: deterministic. 128 rows x 128 batch rows per workgroup was 1 to 3% slower, other instruction
// orders (interleaved by scheduling barriers, raised wavefront priority) no faster.
//
// Rounding. One accumulator for all of a part's chunks, up to several hundred additions, was up to 2.2 times as far from 64
// bits as the 32-row launches, whose workgroups take 6 to 32 chunks each. So a run of chunks (pf_run) ends in an addition to
// the earlier runs' sums, in LDS and the registers left: no further off than those launches over nine layers (0.59 to 1.0
// times, 1.02 on one), for 3% of the time on average (28672x8192 at B = 256 327 -> 336 us).
//
// us per call, 32-row launches of the small-batch kernel -> this, on one 256-CU device: 28672x8192 with 3 bases + 5%
// B = 64 137 -> 112, B = 128 273 -> 192, B = 256 543 -> 336 (1.09 PFLOP/s; a large fp16 matrix product reaches 1.29 on
// the same device), 8192x28672 B = 256 570 -> 339, 4096x4096 with 2 bases + 2% B = 256 146 -> 42. Single calls apart from
// each other; among others the clock is lower (a kernel trace over three layers, B = 256: 374, and 9 for the image).
#include "fluxbin_device.h"
#include "fluxbin_signs.h"

namespace fluxbin {

namespace {

typedef _Float16 pf_f16x8 __attribute__((ext_vector_type(8)));

constexpr int NB = kPfBatch / 16;   // 16-row batch tiles of a workgroup
constexpr int kPfTile = 1024;   // dwords of the activations of a column block and 16 batch rows

// Chunk of base k of column block cb (cb < ncg: global; the first salient chunk is sal0).
__device__ __forceinline__ int pf_chunk(const GemmArgs& a, int cb, int k, int ncs, int sal0) {
  return cb < a.ncg ? k * a.ncg + cb : sal0 + k * ncs + (cb - a.ncg);
}

// Activation operands: dword q of lane (batch row m, group g) for K step t of a column block holds the fp16 pair
// x[b][32 g + j], x[b][32 g + j + 16], j = 4 t + q (the columns whose sign bits one shift brings to bits 15 and 31); zero
// for rows past B and columns without a source. One thread per (column block, 16 batch rows, t, lane); then the
// column-scale pairs in the same order, [column block][4 bases][4 groups][16].
__global__ void __launch_bounds__(256) k_pf_image(GemmArgs a, int ncs, int sal0, int kb, int ks, int btiles,
                                                  uint32_t* ximg, uint32_t* cimg) {
  const int cb = int(blockIdx.x), t = int(threadIdx.x) >> 6, lane = int(threadIdx.x) & 63, m = lane & 15, g = lane >> 4;
  const int b = int(blockIdx.y) * 16 + m;
  const uint16_t* idx = a.xidx + pf_chunk(a, cb, 0, ncs, sal0) * kChunk + 32 * g + 4 * t;
  const uint16_t* x = a.x + int64_t(b < a.B ? b : 0) * a.ldx;
  uint32_t xi[8];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    xi[q] = idx[q];
    xi[4 + q] = idx[16 + q];
  }
  uint16_t v[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = x[xi[q] == 0xFFFFu ? 0 : xi[q]];
  uint32_t o[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t lo = xi[q] == 0xFFFFu || b >= a.B ? 0u : v[q], hi = xi[4 + q] == 0xFFFFu || b >= a.B ? 0u : v[4 + q];
    o[q] = lo | (hi << 16);
  }
  *reinterpret_cast<uint4*>(ximg + (int64_t(cb) * btiles + blockIdx.y) * kPfTile + int(threadIdx.x) * 4) =
      make_uint4(o[0], o[1], o[2], o[3]);
  if (blockIdx.y == 0) {
    const int k = int(threadIdx.x) >> 6, e = int(threadIdx.x) & 63;   // base, 16 g + j
    uint32_t w = 0;
    if (k < (cb < a.ncg ? kb : ks)) {
      const uint16_t* c = a.colscale + pf_chunk(a, cb, k, ncs, sal0) * kChunk + 32 * (e >> 4) + (e & 15);
      w = uint32_t(c[0]) | (uint32_t(c[16]) << 16);
    }
    cimg[cb * 256 + int(threadIdx.x)] = w;
  }
}

// Roundings of a sum of n equal random terms added in runs of r whose sums are then added in turn: the number of terms in
// the running value, summed over the additions (the variance of the result's error, in that of one term's rounding).
int64_t pf_roundings(int64_t n, int64_t r) {
  if (n <= r) return n * (n + 1) / 2;
  const int64_t runs = n / r, rest = n % r;
  return runs * (r * (r + 1) / 2) + r * (runs * (runs + 1) / 2) + (rest > 0 ? rest * (rest + 1) / 2 + n : 0);
}

// Chunks that one accumulator takes, one after another, before its sum goes to the earlier runs': the most whose roundings,
// with those over the parts, are no more than the 32-row launches' of the small-batch kernel (workgroups of 3 to 16
// super-chunks, three per CU, their sums added in turn) less an eighth (runs end with a column block, up to three chunks
// late), or as many as leave the least where that cannot be.
int pf_run(int64_t n_chunks, int64_t row_tiles, int parts) {
  const int64_t units = row_tiles * ((n_chunks + 1) / 2);
  int64_t per = ceil_div(units, 3 * int64_t(device_cu_count()));
  per = per < 3 ? 3 : per > 16 ? 16 : per;
  const int64_t limit = pf_roundings(n_chunks, 2 * per) * 7 / 8, n = ceil_div(n_chunks, parts);
  int64_t best = n, least = -1;
  for (int64_t r = n; r >= 4; --r) {
    const int64_t e = parts * pf_roundings(n, r) + (parts > 1 ? n * parts * (parts + 1) / 2 : 0);
    if (e <= limit) return int(r);
    if (least < 0 || e < least) {
      least = e;
      best = r;
    }
  }
  return int(best);
}

// Copies 1 KB from src (lane l's 16 bytes at src + 4 l) to dst in LDS, without registers.
__device__ __forceinline__ void pf_copy_1k(const uint32_t* src, uint32_t* dst, int lane) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + 4 * lane),
                                   (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}

template <int MU>
__global__ void __launch_bounds__(256, 2) k_gemm_prefill(GemmArgs a, int parts, int ncs, int sal0, int kb, int ks, int run,
                                                         int btiles, const uint32_t* ximg, const uint32_t* cimg) {
  // 78 KB of the 80 that let two workgroups share a CU: the earlier runs' sums (of which the registers left hold the rest),
  // and the activations and column-scale pairs of two column blocks
  constexpr int kKept = 11;   // result vectors whose earlier sums are in LDS (the other five: in registers)
  __shared__ __attribute__((aligned(16))) sign_f32x4 sums[kKept][256];
  __shared__ __attribute__((aligned(16))) uint32_t xs[2][NB * kPfTile];
  __shared__ __attribute__((aligned(16))) uint32_t cs[2][256];
  static_assert(sizeof(sums) + sizeof(xs) + sizeof(cs) <= 80 * 1024, "two workgroups per CU");
  const int lane = int(threadIdx.x) & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int n = lane & 15, q4 = lane >> 4;
  const int row0 = int(blockIdx.x) * 256 + 64 * wave;
  const int bt0 = int(blockIdx.y) * NB;   // first 16-row batch tile
  const int ncb = a.ncg + ncs;
  const int cb0 = ncb * int(blockIdx.z) / parts, cb1 = ncb * int(blockIdx.z + 1) / parts;

  const int r = row0 + lane;
  const uint32_t row = uint32_t(r < a.Mp ? r : a.Mp - 1);   // rows past the padded rows: never stored
  const int64_t plane_bytes = int64_t(a.Mp) * 16;
  const SignRot rot = sign_rot<MU>(row);
  const uint32_t swap = MU == 8 ? (row >> 4) & 1u : 0u;

  struct Signs {
    sign_u32x4 e;
    uint32_t rs;
  };
  auto load_signs = [&](int cb, int k, Signs& s) __attribute__((always_inline)) {
    const int c = pf_chunk(a, cb, k, ncs, sal0);
    const uint8_t* p = a.signs + int64_t(c & ~1) * plane_bytes + ((uint32_t(c & 1) ^ swap) ? plane_bytes : 0) + row * 16u;
    s.e = *reinterpret_cast<const sign_u32x4*>(p);
    s.rs = a.rscale[int64_t(load_uniform_i32(a.chunk_plane, c)) * a.Mp + row];
  };
  auto bases = [&](int cb) __attribute__((always_inline)) { return cb < a.ncg ? kb : ks; };
  auto advance = [&](int& cb, int& k) __attribute__((always_inline)) {   // the next step (the last one repeats)
    if (k + 1 < bases(cb)) {
      ++k;
    } else if (cb + 1 < cb1) {
      ++cb;
      k = 0;
    }
  };
  auto stage = [&](int cb, int buf) __attribute__((always_inline)) {
    const uint32_t* src = ximg + (int64_t(cb) * btiles + bt0) * kPfTile;
#pragma unroll
    for (int i = 0; i < NB; ++i) pf_copy_1k(src + (4 * i + wave) * 256, &xs[buf][(4 * i + wave) * 256], lane);
    if (wave == 0) pf_copy_1k(cimg + cb * 256, &cs[buf][0], lane);
  };

  sign_f32x4 acc[4][NB];   // [row block][16 batch rows]
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[rb][nb] = sign_f32x4{0.f, 0.f, 0.f, 0.f};

  // The run's sums to the earlier runs' (if there are any), and back to zero.
  sign_f32x4 sums_reg[16 - kKept];
#pragma unroll
  for (int e = kKept; e < 16; ++e) sums_reg[e - kKept] = sign_f32x4{0.f, 0.f, 0.f, 0.f};
  const int tid = int(threadIdx.x);
  auto add_earlier = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e / NB][e % NB] += e < kKept ? sums[e][tid] : sums_reg[e - kKept];
  };
  auto keep = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      if (e < kKept)
        sums[e][tid] = acc[e / NB][e % NB];
      else
        sums_reg[e - kKept] = acc[e / NB][e % NB];
      acc[e / NB][e % NB] = sign_f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  static_assert(NB == 4, "16 result vectors");
  bool flushed = false;

  if (cb0 < cb1) {
    stage(cb0, 0);
    Signs sg;
    int cbn = cb0, kn = 0, left = run;
    load_signs(cbn, kn, sg);
    for (int cb = cb0; cb < cb1; ++cb) {
      const int buf = (cb - cb0) & 1;
      // The barrier waits for no memory operation: this wavefront's copies of the column block first (its outstanding
      // loads but the copies are the signs used next). After it every wavefront's copies have landed, and everyone is
      // done with the other buffer.
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      pf_f16x8 xf[4][NB];   // [K step][16 batch rows]
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          xf[t][nb] = *reinterpret_cast<const pf_f16x8*>(&xs[buf][nb * kPfTile + (t * 64 + lane) * 4]);
      const int nk = bases(cb);
      for (int k = 0; k < nk; ++k) {
        uint32_t w[4], rs[4];
        sign_unrotate(sg.e, rot, w);
        sign_transpose(w);
        sign_broadcast(sg.rs, rs);
        uint32_t cp[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const sign_u32x4 v = *reinterpret_cast<const sign_u32x4*>(&cs[buf][k * 64 + 16 * q4 + 4 * q]);
#pragma unroll
          for (int i = 0; i < 4; ++i) cp[4 * q + i] = v[i];
        }
        // after this step's LDS reads: the compiler, which cannot tell the buffers apart, waits for copies before reads
        if (k == 0 && cb + 1 < cb1) stage(cb + 1, buf ^ 1);
        advance(cbn, kn);
        load_signs(cbn, kn, sg);
#pragma unroll
        for (int r2 = 0; r2 < 4; r2 += 2) {   // two row blocks at a time
          const uint64_t ww = (uint64_t(w[r2 + 1]) << 32) | w[r2];
          sign_f32x4 d[2][NB];
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) d[0][nb] = d[1][nb] = sign_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            sign_u32x4 s[2];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int j = 4 * t + q;
              const uint64_t v = j < 15 ? sign_shl64(ww, 15 - j) : ww;
              s[0][q] = (~uint32_t(v) & 0x80008000u) ^ cp[j];
              s[1][q] = (~uint32_t(v >> 32) & 0x80008000u) ^ cp[j];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
              for (int nb = 0; nb < NB; ++nb)
                d[h][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xf[t][nb], __builtin_bit_cast(pf_f16x8, s[h]), d[h][nb],
                                                                  0, 0, 0);
          }
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const float sc = h2f(uint16_t(rs[r2 + h]));
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
              for (int i = 0; i < 4; ++i) acc[r2 + h][nb][i] = __builtin_fmaf(sc, d[h][nb][i], acc[r2 + h][nb][i]);
          }
        }
      }
      left -= nk;
      if (left <= 0 && cb + 1 < cb1) {
        if (flushed) add_earlier();
        keep();
        flushed = true;
        left = run;
      }
    }
  }
  if (flushed) add_earlier();
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int b = (bt0 + nb) * 16 + 4 * q4 + i;
      if (b >= a.B) continue;
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
        const int yr = row0 + 16 * rb + n;
        if (yr >= a.M) continue;
        if (parts == 1)
          store_y(a, b, yr, acc[rb][nb][i]);
        else
          a.partials[(int64_t(blockIdx.z) * a.B + b) * a.Mp + yr] = acc[rb][nb][i];
      }
    }
}

}  // namespace

bool launch_gemm_prefill(const GemmArgs& a, int mu, int kb, int ks, int ncs, int sal0, int parts, hipStream_t stream) {
  if ((mu != 4 && mu != 8) || parts < 1) return false;
  const int ncb = a.ncg + ncs;
  const int btiles = int(ceil_div(a.B, kPfBatch)) * NB;
  uint32_t* cimg = a.img;
  uint32_t* ximg = cimg + int64_t(ncb) * 256;
  hipLaunchKernelGGL(k_pf_image, dim3(unsigned(ncb), unsigned(btiles)), dim3(256), 0, stream, a, ncs, sal0, kb, ks, btiles,
                     ximg, cimg);
  const int run = pf_run(int64_t(kb) * a.ncg + ks * ncs, ceil_div(a.M, 256), parts);
  const dim3 grid(unsigned(ceil_div(a.M, 256)), unsigned(btiles / NB), unsigned(parts));
  if (mu == 8)
    hipLaunchKernelGGL(k_gemm_prefill<8>, grid, dim3(256), 0, stream, a, parts, ncs, sal0, kb, ks, run, btiles,
                       ximg, cimg);
  else
    hipLaunchKernelGGL(k_gemm_prefill<4>, grid, dim3(256), 0, stream, a, parts, ncs, sal0, kb, ks, run, btiles,
                       ximg, cimg);
  if (parts > 1) launch_reduce_parts(a, parts, stream);
  return true;
}

}  // namespace fluxbin
