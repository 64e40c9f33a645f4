// Transforms of length N = R1 R2 R3 shared by L = R2 R3 lanes, R1 complex
// values per lane, for the slice passes on grids that are not a square of a
// register DFT length (a two-step N = R1 R2 has R3 = 1).
//
// Natural index of an element, and who holds it:
//   comb order : L a + b            lane b, register a            (a < R1)
//   block order: p + (R1 R2) d      lane p mod L, registers (p / L, d)
//                p = c + R1 c2      (c < R1, c2 < R2, d < R3)
//                (two-step: c + R1 d, lane c mod L, registers (c / L, d))
// comb_to_block transforms from comb to block order:
//   DFT_R1 over a -> c, twiddle w_N^{bc}; with b = R3 a2 + b2, DFT_R2 over
//   a2 -> c2, twiddle w_L^{b2 c2}; DFT_R3 over b2 -> d.
// block_to_comb is its mirror image (DFT_R3, w_L, DFT_R2, w_N, DFT_R1), so
// both use the same per-lane twiddles: R1 - 1 values w_N^{bc} and R2 - 1
// values w_L^{b2 c2} (b2 = b / R2), kept in registers by the callers (the
// w_L in LDS for R1 = 32, where registers run out). Each step's exchange goes through LDS once. Zero inputs passed as literals and
// unused outputs fold away, which is how the half band is pruned.
//
// LDS of one sequence: S1 = float2 stride of c in the first exchange, S2 of
// b2 in the second. A step over c2 pairs lane b with c = b % R2 + R2 i,
// b2 = b / R2. SYNC orders the LDS accesses of the lanes of a sequence: one
// wave's (wave_sync) or a workgroup's (__syncthreads).
#pragma once

#include "fft_reg.hpp"

namespace prism {

// Orders LDS accesses of one wave (compiler barrier; LDS executes a wave's
// instructions in order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Use every value of an array here, so that loads into it have completed at
// this point. Vector memory operations complete in order: a load still
// pending at the head of a loop would be waited for in every iteration,
// together with the previous iteration's stores.
template <int K>
__device__ __forceinline__ void settle(float2 (&v)[K]) {
#pragma unroll
  for (int i = 0; i < K; ++i) asm volatile("" : "+v"(v[i].x), "+v"(v[i].y));
}

template <int R1_, int R2_, int R3_, int S1_, int S2_, bool WAVE_>
struct Steps {
  static constexpr int R1 = R1_, R2 = R2_, R3 = R3_, S1 = S1_, S2 = S2_;
  static constexpr int N = R1 * R2 * R3, L = R2 * R3;
  static constexpr int M2 = R1 / R2, M3 = R1 / R3;  // DFTs per lane of steps 2 and 3
  static constexpr bool TWO = R3 == 1;
  // w_L twiddles: per lane in registers, or as an LDS table [b2][c2]
  static constexpr bool TLDS = !TWO && R1 >= 32;
  static constexpr int TL = TWO || TLDS ? 1 : R2 - 1, TLN = TLDS ? L : 1;
  struct Tw {
    float2 n[R1 - 1], l[TL];
    const float2* lds;  // TLDS: this lane's row of the table
    __device__ __forceinline__ float2 wl(int c2) const { return TLDS ? lds[c2] : l[c2 - 1]; }
  };
  // float2 of LDS per sequence, without padding between sequences
  static constexpr int E1 = (R1 - 1) * S1 + L, E2 = TWO ? 0 : (R3 - 1) * S2 + R1 * R2;
  static constexpr int SIZE = E1 > E2 ? E1 : E2;
  // registers of the block-order step: v[i * D + d] is element p + (N / D) d,
  // p = lane + L i
  static constexpr int D = TWO ? R2 : R3, MB = R1 / D;
  static_assert(R1 % R2 == 0 && R1 % R3 == 0, "whole DFTs per lane in every step");

  __device__ __forceinline__ static void sync() {
    if constexpr (WAVE_) wave_sync();
    else __syncthreads();
  }

  // twN: exp(-2 pi i k / N); tab: TLN float2 of LDS, written by the workgroup's
  // nt threads (the caller synchronises before the first transform)
  __device__ __forceinline__ static void load_twiddles(const float2* __restrict__ twN, int b,
                                                       float2* tab, int tid, int nt, Tw& t) {
#pragma unroll
    for (int c = 1; c < R1; ++c) t.n[c - 1] = twN[b * c];
    t.l[0] = make_float2(1.f, 0.f);
    if constexpr (TLDS) {
      for (int i = tid; i < L; i += nt) tab[i] = twN[(i / R2) * (i % R2) * R1];
    } else if constexpr (!TWO) {
#pragma unroll
      for (int c2 = 1; c2 < R2; ++c2) t.l[c2 - 1] = twN[(b / R2) * c2 * R1];
    }
    t.lds = tab + (b / R2) * R2;
    settle(t.n);
    settle(t.l);
  }

  template <int R, int M, bool INV>
  __device__ __forceinline__ static void dfts(float2 (&v)[R1]) {
#pragma unroll
    for (int i = 0; i < M; ++i) {
      float2 z[R];
#pragma unroll
      for (int r = 0; r < R; ++r) z[r] = v[i * R + r];
      dft_reg<R, INV>(z);
#pragma unroll
      for (int r = 0; r < R; ++r) v[i * R + r] = z[r];
    }
  }
  template <bool INV>
  __device__ __forceinline__ static float2 mul(float2 a, float2 w) {
    return INV ? cmulc(a, w) : cmul(a, w);
  }

  template <bool INV>
  __device__ __forceinline__ static void comb_to_block(float2 (&v)[R1], float2* lds, int b,
                                                       const Tw& t) {
    dft_reg<R1, INV>(v);
    sync();
#pragma unroll
    for (int c = 0; c < R1; ++c) lds[c * S1 + b] = c ? mul<INV>(v[c], t.n[c - 1]) : v[c];
    sync();
    if constexpr (TWO) {
#pragma unroll
      for (int i = 0; i < M2; ++i)
#pragma unroll
        for (int r = 0; r < R2; ++r) v[i * R2 + r] = lds[(b + L * i) * S1 + r];
      dfts<R2, M2, INV>(v);
    } else {
      const int cl = b % R2, b2 = b / R2;
#pragma unroll
      for (int i = 0; i < M2; ++i)
#pragma unroll
        for (int a2 = 0; a2 < R2; ++a2) v[i * R2 + a2] = lds[(cl + R2 * i) * S1 + R3 * a2 + b2];
      dfts<R2, M2, INV>(v);
      sync();
#pragma unroll
      for (int i = 0; i < M2; ++i)
#pragma unroll
        for (int c2 = 0; c2 < R2; ++c2)
          lds[b2 * S2 + R1 * c2 + cl + R2 * i] =
              c2 ? mul<INV>(v[i * R2 + c2], t.wl(c2)) : v[i * R2 + c2];
      sync();
#pragma unroll
      for (int i = 0; i < M3; ++i)
#pragma unroll
        for (int r = 0; r < R3; ++r) v[i * R3 + r] = lds[r * S2 + b + L * i];
      dfts<R3, M3, INV>(v);
    }
  }

  template <bool INV>
  __device__ __forceinline__ static void block_to_comb(float2 (&v)[R1], float2* lds, int b,
                                                       const Tw& t) {
    if constexpr (TWO) {
      dfts<R2, M2, INV>(v);
      sync();
#pragma unroll
      for (int i = 0; i < M2; ++i)
#pragma unroll
        for (int r = 0; r < R2; ++r) lds[(b + L * i) * S1 + r] = v[i * R2 + r];
    } else {
      const int cl = b % R2, b2 = b / R2;
      dfts<R3, M3, INV>(v);
      sync();
#pragma unroll
      for (int i = 0; i < M3; ++i)
#pragma unroll
        for (int r = 0; r < R3; ++r) lds[r * S2 + b + L * i] = v[i * R3 + r];
      sync();
#pragma unroll
      for (int i = 0; i < M2; ++i)
#pragma unroll
        for (int c2 = 0; c2 < R2; ++c2) {
          const float2 z = lds[b2 * S2 + R1 * c2 + cl + R2 * i];
          v[i * R2 + c2] = c2 ? mul<INV>(z, t.wl(c2)) : z;
        }
      dfts<R2, M2, INV>(v);
      sync();
#pragma unroll
      for (int i = 0; i < M2; ++i)
#pragma unroll
        for (int a2 = 0; a2 < R2; ++a2) lds[(cl + R2 * i) * S1 + R3 * a2 + b2] = v[i * R2 + a2];
    }
    sync();
#pragma unroll
    for (int c = 0; c < R1; ++c) {
      const float2 z = lds[c * S1 + b];
      v[c] = c ? mul<INV>(z, t.n[c - 1]) : z;
    }
    dft_reg<R1, INV>(v);
  }
};

// Radices and LDS strides of each grid side's row pass (a sequence is a row,
// consecutive lanes hold consecutive elements) and column pass (consecutive
// lanes hold the TC columns of a tile). The strides keep the 16 lanes that
// LDS serves together on distinct 8-byte banks: RS is the distance between
// sequences.
__host__ __device__ constexpr int steps_wgs(int nt, int lds) {
  return 512 / nt < 163840 / lds ? (512 / nt > 0 ? 512 / nt : 1) : 163840 / lds;
}
template <int N>
struct GridSteps;
#define PRISM_GRID_STEPS(N_, R1_, R2_, R3_, RP1, RP2, RRS, TC_, CP1, CP2, CRS)                \
  template <>                                                                                 \
  struct GridSteps<N_> {                                                                      \
    static constexpr int L = R2_ * R3_;                                                       \
    static constexpr bool WAVE = 64 % L == 0; /* a row never crosses a wave */                \
    using Row = Steps<R1_, R2_, R3_, L + RP1, R1_ * R2_ + RP2, WAVE>;                         \
    using Col = Steps<R1_, R2_, R3_, L + CP1, R1_ * R2_ + CP2, false>;                        \
    static constexpr int ROW_NT = WAVE ? 256 : 192, ROW_RS = RRS, TC = TC_, COL_RS = CRS;     \
    /* workgroups per compute unit: two waves per SIMD, 160 KiB of LDS */                     \
    static constexpr int ROW_WGS = steps_wgs(ROW_NT, ROW_NT / L * RRS * 8);                   \
    static constexpr int COL_WGS = steps_wgs(TC_ * L, (TC_ * CRS + N_ / 2) * 8);              \
    static_assert(R1_ * R2_ * R3_ == N_, "radices");                                          \
    static_assert(Row::SIZE <= RRS && Col::SIZE <= CRS, "LDS of a sequence");                 \
    static_assert(ROW_NT % L == 0 && R1_ % 4 == 0 && Row::D % 4 == 0, "half-band pruning");   \
  };
//               N    R1  R2  R3  row: +S1 +S2 RS    col: TC +S1 +S2 RS
PRISM_GRID_STEPS(2048, 32, 8, 8, 2, 8, 2110, 8, 1, 0, 2082)
PRISM_GRID_STEPS(1536, 24, 8, 8, 2, 8, 1592, 8, 1, 0, 1562)
PRISM_GRID_STEPS(1152, 24, 6, 8, 2, 6, 1200, 8, 1, 4, 1182)
PRISM_GRID_STEPS(768, 24, 8, 4, 2, 8, 814, 16, 0, 0, 769)
PRISM_GRID_STEPS(576, 24, 24, 1, 1, 0, 600, 16, 0, 0, 577)
PRISM_GRID_STEPS(512, 32, 16, 1, 1, 0, 560, 16, 0, 0, 513)
PRISM_GRID_STEPS(384, 24, 4, 4, 4, 4, 496, 16, 0, 0, 385)
PRISM_GRID_STEPS(192, 24, 8, 1, 1, 0, 216, 16, 8, 0, 377)
PRISM_GRID_STEPS(128, 16, 8, 1, 1, 0, 152, 16, 8, 0, 249)
#undef PRISM_GRID_STEPS

}  // namespace prism
