// PRISM window sum (Eq. PRISMfinal over the window of Eq. RegionBounds) on
// a packed, pixel-major copy of the active beams of S: with 16-bit (BF16 or
// FP16) operands for callers that accept their rounding, or with FP32
// operands. Accumulation is FP32 in both.
//
//  * FP16: every active beam plane S_a is multiplied by an exact power of two
//    scale[a] that brings its largest component below 1, and alpha_a is
//    divided by the same factor, so the product is unchanged in exact
//    arithmetic and FP16 stays in range. BF16 has FP32's range: a power of
//    two only shifts the operands' exponents there, every product is the
//    same, and the pass over S that finds the scales is left out.
//  * S is packed once per call into a pixel-major copy s16[pixel][beam] =
//    (Re, Im), beam rows padded to whole K blocks, so that one 32-beam K
//    block of a pixel is 128 contiguous bytes. Calls of few probes pack only
//    the pixel tiles that some window meets.
//  * alpha is written by k_alpha16 directly in the MFMA A layout per probe
//    group and K block: FP32 real-ified (rows 2g: (Re, -Im), rows 2g+1: (Im,
//    Re)); 16-bit one row (Re, -Im) per probe, from which the matrix core's
//    (Im, Re) operand is made in registers (a half swap and a sign).
//  * v_mfma_f32_16x16x32_{bf16,f16}: lane l holds A[l%16][8(l/16)+j],
//    B[8(l/16)+j][l%16] (j < 8) and D[4(l/16)+i][l%16] (i < 4).
//  * FP32: a K block is 16 beams (the same 128 bytes per row). Each lane
//    reads 16 bytes = 4 K' values and feeds four v_mfma_f32_16x16x4f32
//    steps; K' is visited as 4 (l/16) + 16 ks + s on both operands, a
//    permutation of the block's 32 real K' indices, so the sum is the same.
//    The scale is 1.
//  * Staging: K blocks go straight from global memory into XOR-swizzled LDS rows
//    (global_load_lds_dwordx4), one block ahead of the products, in both forms.
//    FP32 waves read both K steps' operands of a block before its products;
//    16-bit ones load the first block of the workgroup's next tile during the
//    last products of this one.
//  * The 1 / (W sqrt(B_A)) normalisation is applied in FP32 at the end.
#include <algorithm>

#include "fft_lds.hpp"
#include "kernels.hpp"

namespace prism {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int wrap_mod16(long long v, int m) {
  long long r = v % m;
  return (int)(r < 0 ? r + m : r);
}

// Difference d of two origins in [0, ns) (ns even) wrapped to [-ns/2, ns/2).
__device__ __forceinline__ int wrap_near(int d, int ns) {
  return d >= ns / 2 ? d - ns : (d < -ns / 2 ? d + ns : d);
}

template <Prec P>
__device__ __forceinline__ uint32_t pack16(float lo, float hi) {
  uint16_t a, b;
  if constexpr (P == Prec::kBF16) {
    a = __builtin_bit_cast(uint16_t, (__bf16)lo);
    b = __builtin_bit_cast(uint16_t, (__bf16)hi);
  } else {
    a = __builtin_bit_cast(uint16_t, (_Float16)lo);
    b = __builtin_bit_cast(uint16_t, (_Float16)hi);
  }
  return (uint32_t)a | ((uint32_t)b << 16);
}

// One 16-byte operand pair: one 16x16x32 MFMA (16-bit) or four 16x16x4
// steps (FP32).
template <Prec P>
__device__ __forceinline__ floatx4 mfma16(u32x4 a, u32x4 b, floatx4 c) {
  if constexpr (P == Prec::kF32) {
    const floatx4 af = __builtin_bit_cast(floatx4, a), bf = __builtin_bit_cast(floatx4, b);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(af.x, bf.x, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(af.y, bf.y, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(af.z, bf.z, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(af.w, bf.w, c, 0, 0, 0);
    return c;
  }
  if constexpr (P == Prec::kBF16) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  } else if constexpr (P == Prec::kFP16) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, a),
                                                  __builtin_bit_cast(halfx8, b), c, 0, 0, 0);
  }
}

// ---------------------------------------------------------------------------
// Largest |Re|, |Im| of each active plane: kScaleSplit blocks per plane
// (enough blocks to fill the GPU even for a few beams), then one thread per
// beam folds the partial maxima into the power-of-two scale.
__global__ __launch_bounds__(256) void k_s16_absmax(const float2* __restrict__ S,
                                                    const ActiveBeam* __restrict__ act, int ns,
                                                    float* __restrict__ partial) {
  const int a = blockIdx.x, part = blockIdx.y, tid = threadIdx.x;
  const size_t per = (size_t)ns * ns / kScaleSplit;  // complex values per block (even)
  const float4* pl = reinterpret_cast<const float4*>(S + (size_t)act[a].plane * ns * ns +
                                                     (size_t)part * per);
  float m = 0.f;
  for (size_t i = tid; i < per / 2; i += 256) {
    const float4 v = pl[i];
    m = fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  __shared__ float red[4];
  if ((tid & 63) == 0) red[tid >> 6] = m;
  __syncthreads();
  if (tid == 0)
    partial[(size_t)a * kScaleSplit + part] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

__global__ __launch_bounds__(256) void k_s16_scale(const float* __restrict__ partial, int n_act,
                                                   float* __restrict__ scale) {
  const int a = blockIdx.x * 256 + threadIdx.x;
  if (a >= n_act) return;
  float mm = 0.f;
  for (int k = 0; k < kScaleSplit; ++k) mm = fmaxf(mm, partial[(size_t)a * kScaleSplit + k]);
  float sc = 1.f;
  if (mm > 0.f) {
    int e;
    frexpf(mm, &e);  // mm = fr * 2^e with fr in [0.5, 1), so mm < 2^e
    sc = ldexpf(1.f, -e);
  }
  scale[a] = sc;
}

// Whether some window (of side w, origins org[0 .. np) in [0, ns)) holds a
// pixel of the 64 from pix0 on (one answer per workgroup of 256 threads).
__device__ __forceinline__ bool tile_met(const int2* __restrict__ org, int np, int w, int ns,
                                         int pix0) {
  const int y0 = pix0 / ns, x0 = pix0 - y0 * ns;
  const int len = min(64, ns - x0);  // pixels in row y0; the rest (ns not a multiple of 64) below
  bool met = false;
  for (int p = threadIdx.x; p < np; p += 256) {
    const int2 o = org[p];
    // row y meets when y - o.y (wrapped) is in [0, w); pixels [x, x + n) of
    // a row meet when x - o.x (wrapped) is in [0, w) or o.x is among them
    auto hit = [&](int y, int x, int n) {
      const int dy = y - o.y + (y < o.y ? ns : 0), dx = x - o.x + (x < o.x ? ns : 0);
      return dy < w && (dx < w || dx + n > ns);
    };
    met = met || hit(y0, x0, len);
    for (int y = y0 + 1, left = 64 - len; left > 0; ++y, left -= ns)  // ns = 48, 96, ...
      met = met || (y < ns && hit(y, 0, min(left, ns)));
  }
  return __syncthreads_or(met) != 0;
}

// FP32: 16 beams x 64 pixels per workgroup, transposed through LDS; a pixel
// row holds n_actp (re, im) float pairs, zero past the active beams. org !=
// nullptr: only the pixel tiles that one of np windows meets (the window sum
// multiplies other pixels too, but stores none of those sums). blockIdx.y
// walks the beam blocks.
__global__ __launch_bounds__(256) void k_s32_pack(const float2* __restrict__ S,
                                                  const ActiveBeam* __restrict__ act, int n_act,
                                                  int n_actp, int ns, const int2* __restrict__ org,
                                                  int np, int w, float2* __restrict__ s32) {
  __shared__ float2 tile[64][17];
  const int tid = threadIdx.x;
  const size_t pix0 = (size_t)blockIdx.x * 64;
  if (org && !tile_met(org, np, w, ns, (int)pix0)) return;
  const size_t npix = (size_t)ns * ns;
  float2 v[4];
  auto load = [&](int a0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int a = a0 + (tid + 256 * i) / 64, px = tid % 64;
      v[i] = a < n_act ? S[(size_t)act[a].plane * npix + pix0 + px] : make_float2(0.f, 0.f);
    }
  };
  const int step = 16 * gridDim.y;
  load(blockIdx.y * 16);
  for (int a0 = blockIdx.y * 16; a0 < n_actp; a0 += step) {
#pragma unroll
    for (int i = 0; i < 4; ++i) tile[tid % 64][(tid + 256 * i) / 64] = v[i];
    __syncthreads();
    if (a0 + step < n_actp) load(a0 + step);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = tid + 256 * i;
      const int px = idx / 16, j = idx % 16;
      s32[(pix0 + px) * n_actp + a0 + j] = tile[px][j];
    }
    __syncthreads();
  }
}

// 32 beams x 64 pixels per workgroup, transposed through LDS.
template <Prec P>
__global__ __launch_bounds__(256) void k_s16_pack(const float2* __restrict__ S,
                                                  const ActiveBeam* __restrict__ act, int n_act,
                                                  int n_actp, int ns, const float* __restrict__ scale,
                                                  const int2* __restrict__ org, int np, int w,
                                                  uint32_t* __restrict__ s16) {
  __shared__ uint32_t tile[64][33];
  const int tid = threadIdx.x;
  const size_t pix0 = (size_t)blockIdx.x * 64;
  if (org && !tile_met(org, np, w, ns, (int)pix0)) return;
  const size_t npix = (size_t)ns * ns;
  uint32_t v[8];
  auto load = [&](int a0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int a = a0 + (tid + 256 * i) / 64, px = tid % 64;
      v[i] = 0u;
      if (a < n_act) {
        const float2 z = S[(size_t)act[a].plane * npix + pix0 + px];
        const float sc = prec_scaled(P) ? scale[a] : 1.f;
        v[i] = pack16<P>(z.x * sc, z.y * sc);
      }
    }
  };
  const int step = 32 * gridDim.y;
  load(blockIdx.y * 32);
  for (int a0 = blockIdx.y * 32; a0 < n_actp; a0 += step) {
#pragma unroll
    for (int i = 0; i < 8; ++i) tile[tid % 64][(tid + 256 * i) / 64] = v[i];
    __syncthreads();
    if (a0 + step < n_actp) load(a0 + step);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int idx = tid + 256 * i;
      const int px = idx / 32, j = idx % 32;
      s16[(pix0 + px) * n_actp + a0 + j] = tile[px][j];
    }
    __syncthreads();
  }
}

// One thread per (probe group, K block, probe g, beam bl): the A entries of
// alpha'' = exp(i phase) / scale[a] (scale 1 for FP32), zero outside the
// probe / beam range.
template <Prec P>
__global__ void k_alpha16(const double* __restrict__ probe_xy, int p0, int np,
                          const ActiveBeam* __restrict__ act, int n_act, int f, int ns, int w,
                          ProbeOptics po, const float* __restrict__ scale, int group, int nblk,
                          size_t total, uint32_t* __restrict__ a16, int2* __restrict__ origin) {
  constexpr int KB = prec_block_beams(P);
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int bl = (int)(i % KB);
  const int g = (int)((i / KB) % group);
  const int blk = (int)((i / ((size_t)KB * group)) % nblk);
  const size_t grp = i / ((size_t)KB * group * nblk);
  const size_t p = grp * group + g;
  const int a = blk * KB + bl;
  float re = 0.f, im = 0.f;
  if (p < (size_t)np && a < n_act) {
    const double x0 = probe_xy[2 * (p0 + p)], y0 = probe_xy[2 * (p0 + p) + 1];
    if (a == 0) {
      const double dxs = po.cell / (double)ns;
      const int cx = wrap_mod16((long long)floor(x0 / dxs + 0.5), ns);
      const int cy = wrap_mod16((long long)floor(y0 / dxs + 0.5), ns);
      origin[p] = make_int2(wrap_mod16((long long)cx - w / 2, ns),
                            wrap_mod16((long long)cy - w / 2, ns));
    }
    const double kx = (double)act[a].m * f, ky = (double)act[a].n * f;
    const double dx = kx - po.ktx, dy = ky - po.kty;
    const double q2 = (dx * dx + dy * dy) * (po.dq * po.dq);
    double t = -(0.5 * po.lam * q2 * po.C1 + 0.25 * po.lam * po.lam * po.lam * q2 * q2 * po.C3) -
               (kx * (x0 - po.sx) + ky * (y0 - po.sy)) * po.dq;
    t -= floor(t);
    double s, c;
    sincospi(2.0 * t, &s, &c);
    const double inv = prec_scaled(P) ? 1.0 / (double)scale[a] : 1.0;
    re = (float)(c * inv);
    im = (float)(s * inv);
  }
  const size_t blk0 = (grp * nblk + blk) * (size_t)group;  // probe rows before this block's
  if constexpr (P == Prec::kF32) {
    uint32_t* r0 = a16 + (blk0 + g) * (2 * kC16KB);
    uint32_t* r1 = r0 + kC16KB;
    // row 2g: (Re a, -Im a), row 2g+1: (Im a, Re a) as float pairs
    r0[2 * bl] = __builtin_bit_cast(uint32_t, re);
    r0[2 * bl + 1] = __builtin_bit_cast(uint32_t, -im);
    r1[2 * bl] = __builtin_bit_cast(uint32_t, im);
    r1[2 * bl + 1] = __builtin_bit_cast(uint32_t, re);
  } else {
    a16[(blk0 + g) * kC16KB + bl] = pack16<P>(re, -im);
  }
}

// Four waves cover the 128 pixels of a union tile. FP32 (bound by the matrix
// cores): each wave multiplies every probe row by two 16-pixel column tiles.
// 16 bits (bound by operand reads from LDS): the waves form a grid of WM x WN,
// each PT tiles of 16 probes by CT tiles of 16 pixels; a probe tile is one
// operand read for two products per column (its real and its imaginary rows,
// see C16), so a wave reads PT + CT operands for 2 PT CT products (G = 64: 6
// for 16; eight waves of all 128 real-ified rows by one column read 9 for 8).
constexpr int kNT16 = 256;
template <int G>
struct C16 {
  static constexpr int WM = G == 64 ? 2 : 1, WN = 4 / WM;
  static constexpr int PT = G / WM / 16, CT = 8 / WN;
};
constexpr int kCT32 = 2;
constexpr int kTile16 = 128;  // union pixels per workgroup

// What a workgroup sums: a list of items, each one union tile of 128 pixels
// for the whole group, or (mode 1) one tile of one probe's own window.
struct UnionGeom16 {
  int y0, x0, uy, ux;  // union origin on the S-matrix, rows and columns
  float rux;           // 1 / ux
  // row of linear union pixel up: the float quotient is off by at most one
  __device__ __forceinline__ int row(int up, int& col) const {
    int a = (int)((float)up * rux);
    col = up - a * ux;
    if (col < 0) {
      --a;
      col += ux;
    } else if (col >= ux) {
      ++a;
      col -= ux;
    }
    return a;
  }
};
__device__ __forceinline__ UnionGeom16 union_geom(int y0, int x0, int uy, int ux) {
  return UnionGeom16{y0, x0, uy, ux, 1.0f / (float)ux};
}

struct GroupWork {
  const uint32_t* s16;   // packed S
  const uint32_t* a16g;  // the group's A blocks
  const int2* origin;    // the group's window origins
  float2* window;        // the group's windows
  int rowlen, ns, w, gcount, nblk;
  float out_scale;
  const int *offx, *offy, *zero;  // window offsets from the union origin (LDS)
  UnionGeom16 U;                  // mode 0
  int mode, first, stride, items;

  __device__ __forceinline__ UnionGeom16 item(int k, int& tile, int& only) const {
    if (mode == 0) {
      tile = first + k * stride;
      only = -1;
      return U;
    }
    only = k % gcount;
    tile = first + k / gcount * stride;
    const int2 o = origin[only];
    return union_geom(o.y, o.x, w, w);
  }
};

// S pixels a thread stages for item k: tile columns (tid + 256 i) / 8. Columns
// past the union read pixel 0 instead; their outputs are never stored, and a
// B column only reaches its own output column, so nothing needs clearing.
// Rows of absent probes and beams are zero in the packed A.
template <int NBQ>
__device__ __forceinline__ void tile_pixels(const GroupWork& wk, int k, int (&spix)[NBQ]) {
  int tile, only;
  const UnionGeom16 U = wk.item(k, tile, only);
  const int npix = U.uy * U.ux, ns = wk.ns;
#pragma unroll
  for (int i = 0; i < NBQ; ++i) {
    const int up = tile * kTile16 + (((int)threadIdx.x + kNT16 * i) >> 3);
    int off = 0;
    if (up < npix) {
      int b;
      int y = U.y0 + U.row(up, b), x = U.x0 + b;
      // origins are below ns, unions at most 2 ns wide (W <= ns, spread <= ns)
      y -= y >= 2 * ns ? 2 * ns : (y >= ns ? ns : 0);
      x -= x >= 2 * ns ? 2 * ns : (x >= ns ? ns : 0);
      off = y * ns + x;
    }
    spix[i] = off;
  }
}

// FP32 sums of the workgroup's items.
template <int G>
__device__ __forceinline__ void contract32(const GroupWork& wk, const int* rylo, const int* ryhi,
                                           uint32_t* buf0, uint32_t* buf1) {
  constexpr int RT = G / 8;
  constexpr int AROWS = prec_rows(Prec::kF32) * G;
  static_assert(AROWS * 8 % kNT16 == 0 && kTile16 * 8 % kNT16 == 0,
                "every thread stages whole 16-byte segments of A and B");
  constexpr int NAQ = AROWS * 8 / kNT16;     // u32x4 of the A block per thread
  constexpr int NBQ = kTile16 * 8 / kNT16;   // u32x4 of the B block per thread
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int krow = lane >> 4, mcol = lane & 15;

  // Operands go from global memory straight into LDS
  // (global_load_lds_dwordx4: lane i of a wave's instruction writes its 16
  // bytes at the wave's LDS base + 16 i), one K block ahead of the
  // products, into two buffers that are separate LDS arrays (so the
  // compiler sees that reads of one never wait for loads into the other);
  // no registers stage them. An LDS row holds the 8 16-byte segments of
  // one A row or of one pixel's K block, segment s stored at s ^ (row & 7),
  // so the rows that one read instruction's lanes meet fall in different
  // banks.
  constexpr int P32 = kC16KB;  // LDS row: 32 words, no padding
  constexpr int AOFF = 0, BOFF = AROWS * P32;
  typedef __attribute__((address_space(3))) void* lds_ptr;
  auto issue = [&](uint32_t* buf, int blk, const int (&spix)[NBQ]) {
    const uint32_t* ab = wk.a16g + (size_t)blk * AROWS * kC16KB;
#pragma unroll
    for (int i = 0; i < NAQ; ++i) {
      const int row = (tid + kNT16 * i) >> 3;
      const int seg = (tid & 7) ^ (row & 7);
      __builtin_amdgcn_global_load_lds(ab + (size_t)row * kC16KB + 4 * seg,
                                       (lds_ptr)(buf + AOFF + 4 * (kNT16 * i + 64 * wv)), 16, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < NBQ; ++i) {
      const int row = (tid + kNT16 * i) >> 3;
      const int seg = (tid & 7) ^ (row & 7);
      __builtin_amdgcn_global_load_lds(
          wk.s16 + (size_t)spix[i] * wk.rowlen + blk * kC16KB + 4 * seg,
          (lds_ptr)(buf + BOFF + 4 * (kNT16 * i + 64 * wv)), 16, 0, 0);
    }
  };

#pragma unroll 1
  for (int k = 0; k < wk.items; ++k) {
    int tile, only;
    const UnionGeom16 U = wk.item(k, tile, only);
    const int npix = U.uy * U.ux;
    int spix[NBQ];
    tile_pixels<NBQ>(wk, k, spix);

    // Row tiles (8 probes each) this wave multiplies: those holding a probe
    // whose window meets a union row of the wave's 32 pixels. The skipped
    // products only reach outputs the epilogue never stores, so the stored
    // sums are the same.
    unsigned rmask = 0;
    if (only >= 0) {
      rmask = 1u << (only / 8);
    } else {
      const int up0 = tile * kTile16 + 16 * kCT32 * wv;
      if (up0 < npix) {
        int c;
        const int a0 = U.row(up0, c), a1 = U.row(min(up0 + 16 * kCT32, npix) - 1, c);
#pragma unroll
        for (int r = 0; r < RT; ++r)
          if (rylo[r] <= a1 && ryhi[r] >= a0) rmask |= 1u << r;
      }
    }
    rmask = __builtin_amdgcn_readfirstlane(rmask);

    floatx4 acc[RT][kCT32];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int c = 0; c < kCT32; ++c) acc[r][c] = floatx4{0.f, 0.f, 0.f, 0.f};
    // both K steps' operands are read before the products, so the second
    // step's reads overlap the first step's products
    auto compute = [&](const uint32_t* buf) {
      const uint32_t* A = buf + AOFF + mcol * P32;
      const uint32_t* Bm = buf + BOFF + (16 * kCT32 * wv + mcol) * P32;
      u32x4 av[2][RT], bv[2][kCT32];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const int seg = 4 * ((krow + 4 * ks) ^ (mcol & 7));
#pragma unroll
        for (int r = 0; r < RT; ++r)
          av[ks][r] = *reinterpret_cast<const u32x4*>(A + 16 * r * P32 + seg);
#pragma unroll
        for (int c = 0; c < kCT32; ++c)
          bv[ks][c] = *reinterpret_cast<const u32x4*>(Bm + 16 * c * P32 + seg);
      }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int r = 0; r < RT; ++r)
          if (rmask >> r & 1u)
#pragma unroll
            for (int c = 0; c < kCT32; ++c)
              acc[r][c] = mfma16<Prec::kF32>(av[ks][r], bv[ks][c], acc[r][c]);
    };
    // block 2j in buf0, 2j + 1 in buf1
    issue(buf0, 0, spix);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's loads are in LDS
    __syncthreads();
    for (int blk = 0; blk < wk.nblk; blk += 2) {
      const bool pair = blk + 1 < wk.nblk;
      if (pair) issue(buf1, blk + 1, spix);
      compute(buf0);
      __builtin_amdgcn_s_waitcnt(0x0F70);
      // every wave's block blk + 1 is in LDS and no wave still reads buf0
      __syncthreads();
      if (!pair) break;
      if (blk + 2 < wk.nblk) issue(buf0, blk + 2, spix);
      compute(buf1);
      __builtin_amdgcn_s_waitcnt(0x0F70);
      __syncthreads();
    }

    const int w = wk.w;
    const size_t w2 = (size_t)w * w;
    const int* ox = only >= 0 ? wk.zero : wk.offx;
    const int* oy = only >= 0 ? wk.zero : wk.offy;
#pragma unroll
    for (int c = 0; c < kCT32; ++c) {
      const int up = tile * kTile16 + 16 * kCT32 * wv + 16 * c + mcol;
      if (up >= npix) continue;
      int b;
      const int a = U.row(up, b);
#pragma unroll
      for (int r = 0; r < RT; ++r) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int g = 8 * r + 2 * krow + h;
          if (g >= wk.gcount || (only >= 0 && g != only)) continue;
          const int v = a - oy[g], u = b - ox[g];
          if (v < 0 || v >= w || u < 0 || u >= w) continue;
          wk.window[(size_t)g * w2 + (size_t)v * w + u] =
              make_float2(acc[r][c][2 * h] * wk.out_scale, acc[r][c][2 * h + 1] * wk.out_scale);
        }
      }
    }
  }
}

// 16-bit sums of the workgroup's items. Probe tile r of a wave: the operand
// read holds (Re, -Im) of 16 probes; swapping the halves of each word and
// flipping the low one's sign gives (Im, Re), so the wave's two products are
// the real and the imaginary parts of the sums. The next item's first K block
// is fetched during the last products of this one. Bound: the L2 /
// Infinity Cache traffic and latency of the pixel rows.
template <int G, Prec P>
__device__ __forceinline__ void contract16(const GroupWork& wk, uint32_t* buf0, uint32_t* buf1) {
  using C = C16<G>;
  constexpr int PT = C::PT, CT = C::CT, P32 = kC16KB;
  constexpr int AQ = G * 8;                         // 16-byte segments of the A block
  constexpr int NAQ = (AQ + kNT16 - 1) / kNT16;     // of them per thread
  constexpr int NBQ = kTile16 * 8 / kNT16;          // segments of the B block per thread
  constexpr int BOFF = G * P32;
  typedef __attribute__((address_space(3))) void* lds_ptr;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wv / C::WN, wn = wv % C::WN;
  const int krow = lane >> 4, mcol = lane & 15;
  const int seg = 4 * ((tid & 7) ^ ((tid >> 3) & 7));  // this thread's source segment (words)
  const uint32_t* asrc = wk.a16g + (tid >> 3) * P32 + seg;
  const size_t row = (size_t)wk.rowlen;

  const uint32_t* bsrc[NBQ];
  auto pixels = [&](int k) {
    int spix[NBQ];
    tile_pixels<NBQ>(wk, k, spix);
#pragma unroll
    for (int i = 0; i < NBQ; ++i) bsrc[i] = wk.s16 + spix[i] * row + seg;
  };
  // K block blk of the current item into buf; bsrc steps to the next block
  auto issue = [&](uint32_t* buf, int blk) {
    const uint32_t* ab = asrc + (size_t)blk * (G * P32);
#pragma unroll
    for (int i = 0; i < NAQ; ++i)
      if (AQ >= kNT16 || wv < AQ / 64)
        __builtin_amdgcn_global_load_lds(ab + i * (kNT16 / 8) * P32,
                                         (lds_ptr)(buf + 4 * (kNT16 * i + 64 * wv)), 16, 0, 0);
#pragma unroll
    for (int i = 0; i < NBQ; ++i) {
      __builtin_amdgcn_global_load_lds(bsrc[i], (lds_ptr)(buf + BOFF + 4 * (kNT16 * i + 64 * wv)),
                                       16, 0, 0);
      bsrc[i] += P32;
    }
  };

  pixels(0);
  issue(buf0, 0);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's loads are in LDS
  __syncthreads();
#pragma unroll 1
  for (int k = 0; k < wk.items; ++k) {
    floatx4 re[PT][CT], im[PT][CT];
#pragma unroll
    for (int r = 0; r < PT; ++r)
#pragma unroll
      for (int c = 0; c < CT; ++c) re[r][c] = im[r][c] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto compute = [&](const uint32_t* buf) {
      const uint32_t* A = buf + (16 * PT * wm + mcol) * P32;
      const uint32_t* Bm = buf + BOFF + (16 * CT * wn + mcol) * P32;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const int sg = 4 * ((krow + 4 * ks) ^ (mcol & 7));
        u32x4 av[PT], bv[CT];
#pragma unroll
        for (int r = 0; r < PT; ++r)
          av[r] = *reinterpret_cast<const u32x4*>(A + 16 * r * P32 + sg);
#pragma unroll
        for (int c = 0; c < CT; ++c)
          bv[c] = *reinterpret_cast<const u32x4*>(Bm + 16 * c * P32 + sg);
#pragma unroll
        for (int r = 0; r < PT; ++r) {
          u32x4 aw;
#pragma unroll
          for (int q = 0; q < 4; ++q)
            aw[q] = __builtin_amdgcn_alignbit(av[r][q], av[r][q], 16) ^ 0x8000u;
#pragma unroll
          for (int c = 0; c < CT; ++c) {
            re[r][c] = mfma16<P>(av[r], bv[c], re[r][c]);
            im[r][c] = mfma16<P>(aw, bv[c], im[r][c]);
          }
        }
      }
    };
#pragma unroll 1
    for (int blk = 0; blk < wk.nblk; blk += 2) {
      const bool pair = blk + 1 < wk.nblk;
      if (pair) issue(buf1, blk + 1);
      compute(buf0);
      __builtin_amdgcn_s_waitcnt(0x0F70);
      // every wave's block blk + 1 is in LDS and no wave still reads buf0
      __syncthreads();
      if (blk + 2 < wk.nblk) {
        issue(buf0, blk + 2);
      } else if (k + 1 < wk.items) {
        pixels(k + 1);
        issue(buf0, 0);
      }
      if (pair) compute(buf1);
      __builtin_amdgcn_s_waitcnt(0x0F70);
      __syncthreads();
    }

    int tile, only;
    const UnionGeom16 U = wk.item(k, tile, only);
    const int npix = U.uy * U.ux;
    const unsigned w = (unsigned)wk.w;
    int ca[CT], cb[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const int up = tile * kTile16 + 16 * CT * wn + 16 * c + mcol;
      ca[c] = U.row(up, cb[c]);
      if (up >= npix) ca[c] = -(1 << 20);  // outside every window
    }
#pragma unroll
    for (int r = 0; r < PT; ++r) {
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const int g = 16 * (PT * wm + r) + 4 * krow + h;
        if (g >= wk.gcount || (only >= 0 && g != only)) continue;
        const int oy = only >= 0 ? 0 : wk.offy[g], ox = only >= 0 ? 0 : wk.offx[g];
        float2* win = wk.window + (size_t)g * w * w;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          const unsigned v = (unsigned)(ca[c] - oy), u = (unsigned)(cb[c] - ox);
          if (v < w && u < w)
            win[v * w + u] = make_float2(re[r][c][h] * wk.out_scale, im[r][c][h] * wk.out_scale);
        }
      }
    }
  }
}

// Grid: one dimension of (group, slot) pairs over the probe groups of every
// segment (segment k owns groups g_begin .. g_begin + ceil(np / G)); the slots of
// a group share its union tiles round-robin. set == 0: slots of a group adjacent.
// set > 0: `set` neighbouring groups and all their slots run on one XCD
// (workgroups are dealt to the 8 XCDs by blockIdx % 8), one group of the set
// after the other at the same slot, so that its L2 serves the pixels they share.
template <int G, Prec P>
__global__ __launch_bounds__(kNT16)
__attribute__((amdgpu_waves_per_eu(P == Prec::kF32 ? 2 : 3))) void k_contract16(
    const ContractSegs segs, int w, int slots, int set) {
  // two arrays, one per buffer (A block, then B block)
  constexpr bool F32 = P == Prec::kF32;
  constexpr int LDSB = (prec_rows(P) * G + kTile16) * kC16KB;
  __shared__ uint32_t sbuf0[LDSB], sbuf1[LDSB];
  __shared__ int offx[G], offy[G];
  __shared__ int zero[G];
  __shared__ int ginfo[6];
  __shared__ int rylo[G / 8], ryhi[G / 8];  // union rows each row tile's windows span
  const int tid = threadIdx.x;
  // which group, and which of its slots
  int gidx, slot;
  if (set == 0) {
    gidx = blockIdx.x / slots;
    slot = blockIdx.x % slots;
  } else {
    const int i = blockIdx.x >> 3, per = set * slots;
    gidx = ((i / per) * 8 + (blockIdx.x & 7)) * set + i % set;
    slot = i % per / set;
    if (gidx >= segs.groups) return;
  }
  int k = 0;  // segment of this group (uniform)
  while (k + 1 < segs.n && gidx >= segs.s[k + 1].g_begin) ++k;
  const ContractSeg& sg = segs.s[k];
  const uint32_t* __restrict__ s16 = sg.s16;
  const int2* __restrict__ origin = sg.origin;
  const int rowlen = sg.rowlen, ns = sg.ns, np = sg.np;
  const int grp = gidx - sg.g_begin;
  const int p_base = grp * G;
  const int gcount = min(G, np - p_base);
  const int nblk = rowlen / kC16KB;
  const uint32_t* a16g = sg.a16 + (size_t)grp * nblk * (prec_rows(P) * G) * kC16KB;
  if (tid < 64) {
    // group geometry in wave 0, one lane per probe (G <= 64): offsets of
    // each window from the first, their extent, and the union origin
    const int2 o0 = origin[p_base];
    int rx = 0, ry = 0;
    if (tid < gcount) {
      const int2 o = origin[p_base + tid];
      rx = wrap_near(o.x - o0.x, ns);
      ry = wrap_near(o.y - o0.y, ns);
    }
    int minx = rx, maxx = rx, miny = ry, maxy = ry;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      minx = min(minx, __shfl_xor(minx, off, 64));
      maxx = max(maxx, __shfl_xor(maxx, off, 64));
      miny = min(miny, __shfl_xor(miny, off, 64));
      maxy = max(maxy, __shfl_xor(maxy, off, 64));
    }
    if (tid < G) {
      offx[tid] = rx - minx;
      offy[tid] = ry - miny;
    }
    if (tid == 0) {
      // one pass over the union of the windows costs (w + sx)(w + sy)
      // pixels, one pass per probe costs gcount w^2: take the cheaper (each
      // output pixel gets the same sum either way)
      const long long uni = (long long)(w + maxx - minx) * (w + maxy - miny);
      ginfo[0] = uni <= (long long)gcount * w * w ? 0 : 1;
      ginfo[1] = o0.y + miny < 0 ? o0.y + miny + ns : o0.y + miny;  // minx, miny in [-ns/2, 0]
      ginfo[2] = o0.x + minx < 0 ? o0.x + minx + ns : o0.x + minx;
      ginfo[3] = w + (maxy - miny);
      ginfo[4] = w + (maxx - minx);
    }
  }
  for (int g = tid; g < G; g += kNT16) zero[g] = 0;
  __syncthreads();
  if (tid < G / 8) {
    int lo = 1 << 30, hi = -1;
    for (int j = 0; j < 8; ++j) {
      const int g = 8 * tid + j;
      if (g < gcount) {
        lo = min(lo, offy[g]);
        hi = max(hi, offy[g] + w - 1);
      }
    }
    rylo[tid] = lo;
    ryhi[tid] = hi;
  }
  __syncthreads();
  // the workgroups of a group share its tiles round-robin
  GroupWork wk;
  wk.s16 = s16;
  wk.a16g = a16g;
  wk.origin = origin + p_base;
  wk.window = sg.window + (size_t)p_base * w * w;
  wk.rowlen = rowlen;
  wk.ns = ns;
  wk.w = w;
  wk.gcount = gcount;
  wk.nblk = nblk;
  wk.out_scale = sg.out_scale;
  wk.offx = offx;
  wk.offy = offy;
  wk.zero = zero;
  wk.mode = __builtin_amdgcn_readfirstlane(ginfo[0]);
  wk.U = union_geom(__builtin_amdgcn_readfirstlane(ginfo[1]),
                    __builtin_amdgcn_readfirstlane(ginfo[2]),
                    __builtin_amdgcn_readfirstlane(ginfo[3]),
                    __builtin_amdgcn_readfirstlane(ginfo[4]));
  wk.first = slot;
  wk.stride = slots;
  const int tiles = ((wk.mode == 0 ? wk.U.uy * wk.U.ux : w * w) + kTile16 - 1) / kTile16;
  const int mine = (tiles - wk.first + wk.stride - 1) / wk.stride;
  wk.items = mine * (wk.mode == 0 ? 1 : gcount);
  if (wk.first >= tiles) return;
  if constexpr (F32) contract32<G>(wk, rylo, ryhi, sbuf0, sbuf1);
  else contract16<G, P>(wk, sbuf0, sbuf1);
}

inline unsigned blocks16(size_t n, unsigned bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

hipError_t launch_s16_scale(const float2* smatrix, const ActiveBeam* act, int n_act, int ns,
                            float* partial, float* scale, hipStream_t st) {
  hipLaunchKernelGGL(k_s16_absmax, dim3((unsigned)n_act, (unsigned)kScaleSplit), dim3(256), 0, st,
                     smatrix, act, ns, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_s16_scale, dim3((unsigned)((n_act + 255) / 256)), dim3(256), 0, st, partial,
                     n_act, scale);
  return hipGetLastError();
}

hipError_t launch_s16_pack(const float2* smatrix, const ActiveBeam* act, int n_act, int n_actp,
                           int ns, const float* scale, const int2* org, int np, int w, void* s16,
                           Prec prec, hipStream_t st) {
  const int nblk = n_actp / prec_block_beams(prec);
  const int tiles = ns * ns / 64;
  // The workgroups of a tile that packs selectively repeat its window test, so
  // each walks more beam blocks the longer that test is (4, 2 per 256 probes),
  // as long as 4096 workgroups are left to find the tiles that are met.
  int gy = nblk;
  if (org) {
    const int walk = std::max(4, 2 * ((np + 255) / 256));
    gy = std::max((nblk + walk - 1) / walk, std::min(nblk, (4096 + tiles - 1) / tiles));
  }
  const dim3 grid((unsigned)tiles, (unsigned)gy);
  if (prec == Prec::kF32) {
    hipLaunchKernelGGL(k_s32_pack, grid, dim3(256), 0, st, smatrix, act, n_act, n_actp, ns, org,
                       np, w, static_cast<float2*>(s16));
  } else if (prec == Prec::kBF16) {
    hipLaunchKernelGGL(k_s16_pack<Prec::kBF16>, grid, dim3(256), 0, st, smatrix, act, n_act,
                       n_actp, ns, scale, org, np, w, static_cast<uint32_t*>(s16));
  } else {
    hipLaunchKernelGGL(k_s16_pack<Prec::kFP16>, grid, dim3(256), 0, st, smatrix, act, n_act,
                       n_actp, ns, scale, org, np, w, static_cast<uint32_t*>(s16));
  }
  return hipGetLastError();
}

hipError_t launch_alpha16(const double* probe_xy, int p0, int np, const ActiveBeam* act,
                          int n_act, int n_actp, int f, int ns, int w, const ProbeOptics& po,
                          const float* scale, int group, void* a16, int2* origin, Prec prec,
                          hipStream_t st) {
  const int ngrp = (np + group - 1) / group;
  const int kb = prec_block_beams(prec);
  const int nblk = n_actp / kb;
  const size_t total = (size_t)ngrp * nblk * group * kb;
#define A16(PP)                                                                                \
  hipLaunchKernelGGL(k_alpha16<PP>, dim3(blocks16(total, 256)), dim3(256), 0, st, probe_xy, p0, \
                     np, act, n_act, f, ns, w, po, scale, group, nblk, total,                  \
                     static_cast<uint32_t*>(a16), origin)
  if (prec == Prec::kF32) A16(Prec::kF32);
  else if (prec == Prec::kBF16) A16(Prec::kBF16);
  else A16(Prec::kFP16);
#undef A16
  return hipGetLastError();
}

hipError_t launch_contract16(const ContractSegs& segs, int w, int group, Prec prec,
                             int window_tile_div, hipStream_t st) {
  if (segs.n < 1 || segs.n > kMaxSeg || segs.groups < 1) return hipErrorInvalidValue;
  const int slots = contract_tile_slots(w, window_tile_div, segs.groups, group, prec);
  int set = segs.groups >= 128 ? 4 : 0;
  const int wgs = set == 0 ? slots * segs.groups
                           : ((segs.groups + set - 1) / set + 7) / 8 * 8 * set * slots;
  const dim3 grid((unsigned)wgs);
#define C16(GG, PP) \
  hipLaunchKernelGGL((k_contract16<GG, PP>), grid, dim3(kNT16), 0, st, segs, w, slots, set)
#define C16G(PP)                          \
  switch (group) {                        \
    case 16: C16(16, PP); break;          \
    case 32: C16(32, PP); break;          \
    case 64: C16(64, PP); break;          \
    default: return hipErrorInvalidValue; \
  }
  if (prec == Prec::kF32) {
    C16G(Prec::kF32)
  } else if (prec == Prec::kBF16) {
    C16G(Prec::kBF16)
  } else {
    C16G(Prec::kFP16)
  }
#undef C16G
#undef C16
  return hipGetLastError();
}

}  // namespace prism
