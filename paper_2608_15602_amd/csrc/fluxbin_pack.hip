// Packing kernels of libfluxbin: canonical planes -> device format (relayout of the sign planes, VCM extraction of
// the salient columns, gather of their column scales), plus the layout-decoding kernels used by tests.
//
// VCM (Sec. 3.2, Def. VCM, Eqs. 12-13): the salient columns of each salient base are copied into a dense block of
// virtual columns (dense column t <- input column I_sal[t]) and their column scales are gathered once here, so the
// GEMV kernels read the salient refinement exactly like the global bases.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fluxbin_internal.h"

namespace fluxbin {

struct PackArgs {
  const uint32_t* signs;
  const uint32_t* sal_signs;
  const int32_t* sal_idx;
  const uint16_t* alpha_r;
  const uint16_t* alpha_c;
  const uint16_t* alpha_sr;
  const uint16_t* alpha_sc;
  uint8_t* base;
  int64_t M, N, W, g_r, S, g_s;
  int32_t Kb, Ks, mu, pad0;
  int64_t Npad, ncg, Sv, ncs, NC, NSC, NCP, V, Mp, Gr, Gs, NRP;
  int64_t Gcg, Gcs, ngcp, nfc, Pg;
  uint64_t off_signs, off_rscale, off_colscale, off_xidx, off_chunk_plane, off_sal_idx;
};

struct HeaderWords {
  uint32_t w[64];
};

// Kind of chunk c: 0 global, 1 salient, 2 pad (the separator after the global chunks, or the last chunk of an odd
// count); base k and the first local column.
__device__ inline int chunk_kind(const PackArgs& a, int64_t c, int64_t* k, int64_t* col0) {
  if (c < a.Kb * a.ncg) {
    *k = c / a.ncg;
    *col0 = (c % a.ncg) * kChunk;
    return 0;
  }
  if (c < a.ngcp) {
    *k = 0;
    *col0 = 0;
    return 2;
  }
  const int64_t c2 = c - a.ngcp;
  if (c2 < a.Ks * a.ncs) {
    *k = c2 / a.ncs;
    *col0 = (c2 % a.ncs) * kChunk;
    return 1;
  }
  *k = 0;
  *col0 = 0;
  return 2;
}

// Row scales per chunk c and row (1: one plane; G > 1: a block of G scales per row), by the chunk's scale layout.
__device__ inline int64_t chunk_G(const PackArgs& a, int64_t c) { return c < a.nfc ? a.Gcg : a.Gcs; }

// Position of sub-vector u in row i's 16-byte entry of a chunk with G scale groups (spc = 128/mu positions, n = spc/G per
// group): the groups are rotated by floor(i/n) and the positions within a group by i, so that any spc consecutive rows
// read spc different sub-vectors at every position (G = 1: sub-vector (q + i) mod spc at position q).
__device__ inline int pos_of(int u, int64_t i, int spc, int G) {
  const int n = spc / G;
  const int blk = int((((u / n) - (i / n)) % G + G) % G);
  const int w = int((((u % n) - i) % n + n) % n);
  return blk * n + w;
}

// 128 bits rotated right by rot: bit b of the result is bit (b + rot) mod 128.
__device__ inline void rotate_right(uint32_t w[4], uint32_t rot) {
  const uint32_t sb = rot & 31u;
  uint32_t f[4];
  for (int m = 0; m < 4; ++m) f[m] = __builtin_amdgcn_alignbit(w[(m + 1) & 3], w[m], sb);
  const bool r1 = (rot & 32u) != 0, r2 = (rot & 64u) != 0;
  uint32_t h[4];
  for (int m = 0; m < 4; ++m) h[m] = r1 ? f[(m + 1) & 3] : f[m];
  for (int m = 0; m < 4; ++m) w[m] = r2 ? h[(m + 2) & 3] : h[m];
}

// Every field of f bits (16, 32 or 64; 8 at mu = 4) of the 128 rotated right by rot < f.
__device__ inline void rotate_fields(uint32_t w[4], int f, uint32_t rot) {
  if (f == 64) {
    for (int p = 0; p < 4; p += 2) {
      const uint32_t lo = __builtin_amdgcn_alignbit(w[p + 1], w[p], rot & 31u);
      const uint32_t hi = __builtin_amdgcn_alignbit(w[p], w[p + 1], rot & 31u);
      w[p] = (rot & 32u) != 0 ? hi : lo;
      w[p + 1] = (rot & 32u) != 0 ? lo : hi;
    }
  } else if (f == 32) {
    for (int m = 0; m < 4; ++m) w[m] = __builtin_amdgcn_alignbit(w[m], w[m], rot);
  } else {
    const uint32_t low = ~0u / ((1u << f) - 1u) * ((1u << (f - rot)) - 1u);   // the f - rot low bits of every field
    for (int m = 0; m < 4; ++m) w[m] = ((w[m] >> rot) & low) | ((w[m] << (f - rot)) & ~low);
  }
}

constexpr int kPackRows = 64;   // rows of a workgroup's tile of packed entries

// A workgroup packs 64 rows x C chunks: a transpose of 16-byte pieces through LDS. A wavefront reads 16 C contiguous bytes
// of a row (the tile's chunks of a global base, one word per lane) and writes 1 KB runs of a chunk's rows. A salient
// chunk's bits are gathered 64 columns at a time, a lane each, and collected by a ballot: the column indices are read
// once per tile and the row's words come from the caches. Bound by memory: 28672 x 8192 with 3 bases + 5% (117 MB read,
// 90 MB written) 229 -> 58 us; one thread per entry read rows 1 KB apart and salient columns one after another. C = 16, or
// 4 where that leaves workgroups for fewer than the CUs (a tile's salient chunks follow one another: 64 x 4096, all columns
// salient, 4 bases, whole call 71 -> 48 us; 64 x 28672, half of them salient, 88 -> 66).
template <int C>
__global__ void __launch_bounds__(256) k_pack_signs(PackArgs a) {
  constexpr int LW = 4 * C, RL = 64 / LW;   // a wavefront's load: RL rows of LW words
  // halves of a salient chunk requested together: both where workgroups are few; at C = 16 they would cost 14 registers and
  // with them two of seven wavefronts per SIMD (28672 x 8192, 3 bases + 5%, whole call 98 -> 109 us)
  constexpr int H = C == 4 ? 2 : 1;
  __shared__ uint32_t tile[kPackRows][LW + 4];   // 4 words of padding: rows on different banks
  const int lane = int(threadIdx.x) & 63, wave = int(threadIdx.x) >> 6;
  // the last chunks first: the salient ones, whose workgroups take longest
  const int64_t i0 = int64_t(blockIdx.x) * kPackRows, c0 = int64_t(gridDim.y - 1 - blockIdx.y) * C;
  {
    // global chunks: lane l takes word l & 3 of chunk c0 + (l mod LW) / 4, of row l / LW of a load
    const int64_t c = c0 + (lane % LW >> 2);
    int64_t k = 0, col0 = 0;
    const bool global = c < a.NCP && chunk_kind(a, c, &k, &col0) == 0;
    const int64_t j0 = col0 + 32 * (lane & 3);
    const bool read = global && j0 < a.N;
    const uint32_t keep = a.N - j0 < 32 ? (1u << ((a.N - j0) & 31)) - 1u : ~0u;
    const uint32_t* src = a.signs + (read ? k * a.M * a.W + j0 / 32 : 0);
    uint32_t w[kPackRows / (4 * RL)];
#pragma unroll
    for (int r = 0; r < kPackRows / (4 * RL); ++r) {
      const int64_t i = i0 + (4 * r + wave) * RL + lane / LW;
      w[r] = read && i < a.M ? src[i * a.W] & keep : 0u;
    }
#pragma unroll
    for (int r = 0; r < kPackRows / (4 * RL); ++r) tile[(4 * r + wave) * RL + lane / LW][lane % LW] = w[r];
  }
  __syncthreads();
  const int64_t cs = a.ngcp > c0 ? a.ngcp : c0;
  const int64_t ce = c0 + C < a.NC ? c0 + C : a.NC;
  for (int64_t c = cs; c < ce; ++c) {   // salient chunks of the tile
    int64_t k, col0;
    if (chunk_kind(a, c, &k, &col0) != 1) continue;
    for (int half0 = 0; half0 < 2; half0 += H) {
      uint32_t w[H][kPackRows / 4];   // H halves' words in flight together
      int32_t j[H];
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const int64_t t = col0 + 64 * (half0 + h) + lane;
        j[h] = t < a.S ? a.sal_idx[t] : -1;
      }
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const uint32_t* src = a.sal_signs + k * a.M * a.W + (j[h] < 0 ? 0 : j[h] >> 5);
#pragma unroll
        for (int r = 0; r < kPackRows / 4; ++r) {
          const int64_t i = i0 + 4 * r + wave;
          w[h][r] = j[h] >= 0 && i < a.M ? src[i * a.W] : 0u;
        }
      }
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int r = 0; r < kPackRows / 4; ++r) {
          const uint64_t bits = __builtin_amdgcn_ballot_w64(((w[h][r] >> (j[h] & 31)) & 1u) != 0);
          if (lane < 2) tile[4 * r + wave][4 * (c - c0) + 2 * (half0 + h) + lane] = uint32_t(bits >> (32 * lane));
        }
    }
  }
  __syncthreads();
  const int64_t i = i0 + lane;   // Mp is a multiple of 64: every row of the tile is written
  for (int q = wave; q < C && c0 + q < a.NCP; q += 4) {
    const int64_t c = c0 + q;
    uint32_t bits[4];
    for (int m = 0; m < 4; ++m) bits[m] = tile[lane][4 * q + m];
    const int G = int(chunk_G(a, c));
    if (G == 1 || G == kChunk / a.mu) {
      rotate_right(bits, uint32_t(a.mu * i) & 127u);
    } else {   // the groups rotated by i / n, the sub-vectors of a group by i (pos_of)
      const int f = kChunk / G, n = f / a.mu;
      rotate_right(bits, uint32_t((i / n) % G * f));
      rotate_fields(bits, f, uint32_t(i % n * a.mu));
    }
    const int64_t h = a.mu == 8 ? (c & 1) ^ ((i & 31) >= 16 ? 1 : 0) : (c & 1);
    reinterpret_cast<uint4*>(a.base + a.off_signs)[((c & ~int64_t(1)) + h) * a.Mp + i] =
        make_uint4(bits[0], bits[1], bits[2], bits[3]);
  }
}

// Coarse row scales, a transpose of 64 rows x up to 64 groups through LDS: src [K][M][groups] -> planes [K * groups][Mp]
// from plane p0 (rows past M zero). The tile's source is read in memory order.
__global__ void __launch_bounds__(256) k_pack_rscale_planes(PackArgs a, const uint16_t* src, int64_t groups, int64_t p0) {
  __shared__ uint16_t tile[64][65];
  const int64_t i0 = int64_t(blockIdx.x) * 64, g0 = int64_t(blockIdx.y) * 64, k = blockIdx.z;
  const int ng = int(groups - g0 < 64 ? groups - g0 : 64), t = int(threadIdx.x);
  uint16_t v[16];
#pragma unroll
  for (int m = 0; m < 16; ++m) {   // 64 ng elements, the loads in flight together
    const int e = t + 256 * m, r = e / ng, g = e - r * ng;
    v[m] = r < 64 && i0 + r < a.M ? src[(k * a.M + i0 + r) * groups + g0 + g] : uint16_t(0);
  }
#pragma unroll
  for (int m = 0; m < 16; ++m) {
    const int e = t + 256 * m, r = e / ng, g = e - r * ng;
    if (r < 64) tile[g][r] = v[m];
  }
  __syncthreads();
  uint32_t* dst = reinterpret_cast<uint32_t*>(a.base + a.off_rscale) + ((p0 + k * groups + g0) * a.Mp + i0) / 2;
#pragma unroll
  for (int m = 0; m < 8; ++m) {   // two rows per store
    const int g = (t >> 5) + 8 * m, r = 2 * (t & 31);
    if (g < ng) dst[int64_t(g) * (a.Mp / 2) + (t & 31)] = uint32_t(tile[g][r]) | (uint32_t(tile[g][r + 1]) << 16);
  }
}

// Fine row scales, one thread per scale: a chunk's block of G planes holds, for each row, G consecutive scales; slot b is
// the scale of the chunk's group (b + floor(i/n)) mod G (n = spc/G sub-vectors per group), i.e. the group read at
// positions b*n .. b*n+n-1 of the row's rotated entry. src [K][M][groups], nc chunks per base, planes from p0.
__global__ void k_pack_rscale_fine(PackArgs a, const uint16_t* src, int64_t groups, int64_t nc, int64_t G, int64_t p0,
                                   int64_t count) {
  const int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (e >= count) return;
  const int64_t blk = e / (a.Mp * G);                 // (base, chunk within the base)
  const int64_t i = (e % (a.Mp * G)) / G;
  const int64_t b = e % G;
  const int64_t k = blk / nc, lc = blk % nc;
  const int64_t n = (kChunk / a.mu) / G;
  const int64_t grp = lc * G + (b + i / n) % G;
  reinterpret_cast<uint16_t*>(a.base + a.off_rscale)[p0 * a.Mp + e] =
      i < a.M && grp < groups ? src[(k * a.M + i) * groups + grp] : uint16_t(0);
}

// One thread per virtual column; the first NCP threads also write the chunk's row-scale plane, the first max(S,1)
// threads the 16-bit salient indices, the first 64 the header.
__global__ void k_pack_columns(PackArgs a, HeaderWords h) {
  const int64_t v = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (v < 64) reinterpret_cast<uint32_t*>(a.base)[v] = h.w[v];
  if (v < a.V) {
    const int64_t c = v / kChunk;
    const int64_t r = v % kChunk;
    int64_t k, col0;
    const int kind = chunk_kind(a, c, &k, &col0);
    uint16_t cs = 0, xi = 0xFFFFu;
    if (kind == 0 && col0 + r < a.N) {
      const int64_t j = col0 + r;
      cs = a.alpha_c[k * a.N + j];
      xi = uint16_t(j);
    } else if (kind == 1 && col0 + r < a.S) {
      const int64_t j = a.sal_idx[col0 + r];
      cs = a.alpha_sc[k * a.N + j];
      xi = uint16_t(j);
    }
    reinterpret_cast<uint16_t*>(a.base + a.off_colscale)[v] = cs;
    reinterpret_cast<uint16_t*>(a.base + a.off_xidx)[v] = xi;
  }
  if (v < a.NCP) {
    // first row-scale plane of chunk v; a pad chunk uses the planes of the chunk before it (its signs and column
    // scales are zero, so any finite scale gives it exactly zero)
    int64_t c = v;
    int64_t k, col0;
    int kind = chunk_kind(a, c, &k, &col0);
    while (kind == 2 && c > 0) kind = chunk_kind(a, --c, &k, &col0);
    int64_t plane = 0;
    if (kind == 0) plane = a.Gcg == 1 ? k * a.Gr + col0 / a.g_r : (k * a.ncg + col0 / kChunk) * a.Gcg;
    if (kind == 1) plane = a.Pg + (a.Gcs == 1 ? k * a.Gs + col0 / a.g_s : (k * a.ncs + col0 / kChunk) * a.Gcs);
    reinterpret_cast<int32_t*>(a.base + a.off_chunk_plane)[v] = int32_t(plane);
  }
  const int64_t ns = a.S > 1 ? a.S : 1;
  if (v < ns) {
    reinterpret_cast<uint16_t*>(a.base + a.off_sal_idx)[v] = (v < a.S) ? uint16_t(a.sal_idx[v]) : uint16_t(0);
  }
}

// Reads one virtual sign bit (chunk c, column r of the chunk, row i) back from the device layout.
__device__ inline uint32_t device_bit(const PackArgs& a, const uint8_t* signs, int64_t c, int r, int64_t i) {
  const int64_t Mp = a.Mp;
  const int mu = a.mu;
  const int G = int(chunk_G(a, c));
  const int64_t sc = c >> 1;
  if (mu == 8) {
    const int64_t h = (c & 1) ^ ((i & 31) >= 16 ? 1 : 0);
    const int u = r >> 3, n = r & 7;
    const int q = pos_of(u, i, 16, G);
    const uint8_t byte = signs[((sc * 2 + h) * Mp + i) * 16 + q];
    return (byte >> n) & 1u;
  }
  const int64_t h = c & 1;
  const int u = r >> 2, n = r & 3;
  const int q = pos_of(u, i, 32, G);
  const uint8_t byte = signs[((sc * 2 + h) * Mp + i) * 16 + (q >> 1)];
  return (byte >> (4 * (q & 1) + n)) & 1u;
}

// One thread per output word: global planes [Kb][M][W] then dense salient planes [Ks][M][ceil(S/32)].
__global__ void k_unpack(PackArgs a, uint32_t* d_signs, uint32_t* d_dense) {
  const int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  const uint8_t* signs = a.base + a.off_signs;
  const int64_t ng = a.Kb * a.M * a.W;
  const int64_t Ws = (a.S + 31) / 32;
  const int64_t ns = (d_dense && a.Ks > 0 && a.S > 0) ? a.Ks * a.M * Ws : 0;
  if (e < ng) {
    const int64_t w = e % a.W, i = (e / a.W) % a.M, k = e / (a.W * a.M);
    uint32_t word = 0;
    for (int b = 0; b < 32; ++b) {
      const int64_t j = 32 * w + b;
      if (j >= a.N) break;
      const int64_t vcol = k * a.Npad + j;
      word |= device_bit(a, signs, vcol / kChunk, int(vcol % kChunk), i) << b;
    }
    d_signs[e] = word;
  } else if (e < ng + ns) {
    const int64_t f = e - ng;
    const int64_t w = f % Ws, i = (f / Ws) % a.M, k = f / (Ws * a.M);
    uint32_t word = 0;
    for (int b = 0; b < 32; ++b) {
      const int64_t t = 32 * w + b;
      if (t >= a.S) break;
      const int64_t vcol = a.ngcp * kChunk + k * a.Sv + t;
      word |= device_bit(a, signs, vcol / kChunk, int(vcol % kChunk), i) << b;
    }
    d_dense[f] = word;
  }
}

// Pattern read at step q from the 16-byte entry of a row (the same byte/nibble selection the GEMV kernels make).
__device__ inline uint32_t pattern_at(const uint4& e, int q, int mu) {
  const uint32_t w[4] = {e.x, e.y, e.z, e.w};
  if (mu == 8) return (w[q >> 2] >> (8 * (q & 3))) & 0xFFu;
  return (w[q >> 3] >> (4 * (q & 7))) & 0xFu;
}

// One thread per (chunk c, row i < M, sub-vector u): the LUT index the kernels read for that sub-vector.
__global__ void k_debug_indices(PackArgs a, uint8_t* d_p) {
  const int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  const int per = kChunk / a.mu;
  if (e >= a.NCP * a.M * per) return;
  const int u = int(e % per);
  const int64_t i = (e / per) % a.M;
  const int64_t c = e / (per * a.M);
  const int64_t sc = c >> 1;
  int64_t h;
  int q;
  const int G = int(chunk_G(a, c));
  if (a.mu == 8) {
    h = (c & 1) ^ ((i & 31) >= 16 ? 1 : 0);
    q = pos_of(u, i, 16, G);
  } else {
    h = c & 1;
    q = pos_of(u, i, 32, G);
  }
  const uint4 entry = reinterpret_cast<const uint4*>(a.base + a.off_signs)[(sc * 2 + h) * a.Mp + i];
  d_p[e] = uint8_t(pattern_at(entry, q, a.mu));
}

__global__ void k_fill_zero(uint32_t* d, int64_t n) {
  const int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (e < n) d[e] = 0u;
}

static PackArgs make_args(const fluxbin_layer& L) {
  PackArgs a{};
  const fluxbin_shape& s = L.shape;
  const Derived d = derive(s);
  a.base = static_cast<uint8_t*>(L.d_base);
  a.M = s.M;
  a.N = s.N;
  a.W = (s.N + 31) / 32;
  a.g_r = s.g_r;
  a.S = s.S;
  a.g_s = s.g_s;
  a.Kb = s.Kb;
  a.Ks = s.Ks;
  a.mu = s.mu;
  a.Npad = d.Npad;
  a.ncg = d.ncg;
  a.Sv = d.Sv;
  a.ncs = d.ncs;
  a.NC = d.NC;
  a.NSC = d.NSC;
  a.NCP = d.NCP;
  a.V = d.V;
  a.Mp = d.Mp;
  a.Gr = d.Gr;
  a.Gs = d.Gs;
  a.NRP = d.NRP;
  a.Gcg = d.Gcg;
  a.Gcs = d.Gcs;
  a.ngcp = d.ngcp;
  a.nfc = d.nfc;
  a.Pg = d.Pg;
  a.off_signs = L.off_signs;
  a.off_rscale = L.off_rscale;
  a.off_colscale = L.off_colscale;
  a.off_xidx = L.off_xidx;
  a.off_chunk_plane = L.off_chunk_plane;
  a.off_sal_idx = L.off_sal_idx;
  return a;
}

static unsigned grid_for(int64_t n, int threads) { return unsigned((n + threads - 1) / threads); }

fluxbin_status launch_pack(const fluxbin_layer& L, const fluxbin_weights& w, const int32_t* d_sal_idx,
                           hipStream_t stream) {
  PackArgs a = make_args(L);
  a.signs = w.signs;
  a.sal_signs = w.sal_signs;
  a.sal_idx = d_sal_idx;
  a.alpha_r = w.alpha_r;
  a.alpha_c = w.alpha_c;
  a.alpha_sr = w.alpha_sr;
  a.alpha_sc = w.alpha_sc;
  const Derived d = derive(L.shape);
  const Offsets o = offsets(L.shape, d);
  Header h{};
  h.magic = kMagic;
  h.version = FLUXBIN_FORMAT_VERSION;
  h.shape = L.shape;
  h.Npad = d.Npad;
  h.Sv = d.Sv;
  h.NC = d.NC;
  h.NSC = d.NSC;
  h.Mp = d.Mp;
  h.Gr = d.Gr;
  h.Gs = d.Gs;
  h.NRP = d.NRP;
  h.off_signs = o.signs;
  h.off_rscale = o.rscale;
  h.off_colscale = o.colscale;
  h.off_xidx = o.xidx;
  h.off_chunk_plane = o.chunk_plane;
  h.off_sal_idx = o.sal_idx;
  h.total = o.total;
  HeaderWords hw;
  static_assert(sizeof(hw) == sizeof(h), "header size");
  __builtin_memcpy(&hw, &h, sizeof(h));

  const int T = 256;
  const bool sal = d.NRP > d.Pg;
  const auto signs = [&](auto chunks) {
    constexpr int C = decltype(chunks)::value;
    hipLaunchKernelGGL(k_pack_signs<C>, dim3(unsigned(d.Mp / kPackRows), grid_for(d.NCP, C)), dim3(T), 0, stream, a);
  };
  if (d.Mp / kPackRows * ceil_div(d.NCP, 16) >= device_cu_count())
    signs(std::integral_constant<int, 16>());
  else
    signs(std::integral_constant<int, 4>());
  auto rscale = [&](const uint16_t* src, int64_t K, int64_t groups, int64_t nc, int64_t G, int64_t p0) {
    if (G == 1) {
      hipLaunchKernelGGL(k_pack_rscale_planes, dim3(unsigned(d.Mp / 64), grid_for(groups, 64), unsigned(K)), dim3(T), 0,
                         stream, a, src, groups, p0);
    } else {
      const int64_t n = K * nc * G * d.Mp;
      hipLaunchKernelGGL(k_pack_rscale_fine, dim3(grid_for(n, T)), dim3(T), 0, stream, a, src, groups, nc, G, p0, n);
    }
  };
  rscale(a.alpha_r, L.shape.Kb, d.Gr, d.ncg, d.Gcg, 0);
  if (sal) rscale(a.alpha_sr, L.shape.Ks, d.Gs, d.ncs, d.Gcs, d.Pg);
  int64_t n_col = d.V;
  if (L.shape.S > n_col) n_col = L.shape.S;
  hipLaunchKernelGGL(k_pack_columns, dim3(grid_for(n_col, T)), dim3(T), 0, stream, a, hw);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "launching the packing kernels");
  return FLUXBIN_OK;
}

fluxbin_status launch_unpack(const fluxbin_layer& L, uint32_t* d_signs, uint32_t* d_dense, hipStream_t stream) {
  PackArgs a = make_args(L);
  const int64_t ng = a.Kb * a.M * a.W;
  const int64_t ns = (d_dense && a.Ks > 0 && a.S > 0) ? a.Ks * a.M * ((a.S + 31) / 32) : 0;
  const int T = 256;
  hipLaunchKernelGGL(k_unpack, dim3(grid_for(ng + ns, T)), dim3(T), 0, stream, a, d_signs, d_dense);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "launching the unpack kernel");
  return FLUXBIN_OK;
}

fluxbin_status launch_debug_indices(const fluxbin_layer& L, uint8_t* d_p, hipStream_t stream) {
  PackArgs a = make_args(L);
  const int64_t n = a.NCP * a.M * (kChunk / a.mu);
  const int T = 256;
  hipLaunchKernelGGL(k_debug_indices, dim3(grid_for(n, T)), dim3(T), 0, stream, a, d_p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "launching the debug-indices kernel");
  return FLUXBIN_OK;
}

fluxbin_status launch_fill_zero(void* d, size_t bytes, hipStream_t stream) {
  const int64_t n = int64_t(bytes / 4);
  const int T = 256;
  hipLaunchKernelGGL(k_fill_zero, dim3(grid_for(n, T)), dim3(T), 0, stream, static_cast<uint32_t*>(d), n);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "launching the fill kernel");
  return FLUXBIN_OK;
}

}  // namespace fluxbin
