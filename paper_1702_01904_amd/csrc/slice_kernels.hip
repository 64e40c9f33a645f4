// Multislice kernels (Eqs. 3-5) shared by the PRISM S-matrix build (Fig. 1c)
// and by conventional multislice STEM.
//
// One slice step psi <- iFFT2( FFT2(psi t_p) P_p M ) is split into two
// HBM passes over the compact state X(y, kx) (layout in kernels.hpp):
//   row pass    : X -> iFFT_x -> * t_p / n -> FFT_x -> keep |kx| < n/4 -> X'
//   column pass : X' -> FFT_y -> * P_p(kx) P_p(ky) M / n -> iFFT_y -> X''
// P_p is separable, so it comes from a 1D table per slice; M is the
// half-band anti-aliasing aperture kx^2 + ky^2 < (n/4)^2. Each pass reads
// and writes n^2/2 complex values per wave.
#include <algorithm>

#include "fft_lds.hpp"
#include "fft_reg.hpp"
#include "fft_steps.hpp"
#include "kernels.hpp"

namespace prism {

namespace {

// Launch shapes (tuned on MI355X; overridable at build time).
#ifndef PRISM_COL_E
#define PRISM_COL_E 8          // complex values per LDS column-pass thread
#endif
#ifndef PRISM_ROW_ELEMS
#define PRISM_ROW_ELEMS 2048   // complex values per LDS row-pass workgroup
#endif

// Largest power of two p with p n <= cap (at least 1): rows per workgroup
// that divide every wave's n rows (n = 2^k, 3 2^k or 9 2^k).
__host__ __device__ constexpr int pow2_rows(int n, int cap) {
  return 2 * n <= cap ? 2 * pow2_rows(2 * n, cap) : 1;
}
__host__ __device__ constexpr int col_tc(int n) { return 8; }
__host__ __device__ constexpr int col_nt(int n) {
  return (col_tc(n) * n / PRISM_COL_E) < 64
             ? 64
             : (col_tc(n) * n / PRISM_COL_E > 1024 ? 1024 : col_tc(n) * n / PRISM_COL_E);
}
constexpr int kRowNT = PRISM_ROW_ELEMS / 8;
__host__ __device__ constexpr int row_nseq(int n) { return pow2_rows(n, PRISM_ROW_ELEMS); }
__host__ __device__ constexpr int ext_nseq(int n) { return pow2_rows(n, 4096); }

// Map launch order onto tiles so that consecutive tiles run on the same
// XCD (workgroups are dealt to the 8 XCDs round-robin) and share its L2.
__device__ __forceinline__ int xcd_tile(int bid, int nb) {
  if ((nb & 7) != 0) return bid;
  return (bid & 7) * (nb >> 3) + (bid >> 3);
}

__device__ __forceinline__ int signed_k(int idx, int n) { return idx < n / 2 ? idx : idx - n; }

// ---------------------------------------------------------------------------
__global__ void k_twiddles(float2* tw, int L) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < L) {
    double s, c;
    sincospi(-2.0 * (double)i / (double)L, &s, &c);
    tw[i] = make_float2((float)c, (float)s);
  }
}

// tw2[m][j] = exp(-2 pi i j m / n) for j, m < R, n = R^2 (four-step passes).
__global__ void k_twiddles2(float2* tw2, int R) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < R * R) {
    const int m = i / R, j = i % R;
    double s, c;
    sincospi(-2.0 * (double)(j * m) / (double)(R * R), &s, &c);
    tw2[i] = make_float2((float)c, (float)s);
  }
}

// t_p = exp(i phi_p) / n, the 1/n belonging to the row pass' inverse FFT.
__global__ void k_transmission(const float* __restrict__ phase, float2* __restrict__ trans,
                               size_t count, float scale) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) {
    double s, c;
    sincos((double)phase[i], &s, &c);
    trans[i] = make_float2((float)(c * scale), (float)(s * scale));
  }
}

__global__ void k_prop_lut(float2* lut, int n, int H, const double* __restrict__ thick, double lam,
                           double dq) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * H) return;
  const int p = i / n, idx = i % n;
  const double k = (double)signed_k(idx, n);
  double s, c;
  sincospi(-lam * thick[p] * (k * dq) * (k * dq), &s, &c);
  lut[i] = make_float2((float)c, (float)s);
}

// ---------------------------------------------------------------------------
// Four-step row pass for n = R^2 (R = 16, 32). Row element x = R a + b sits
// with lane b (R lanes per row, 64 / R rows per wave):
//   inverse: lane b transforms over a (only a < R/4 and a >= 3R/4 are
//            nonzero: the compact half band), twiddles by w_n^{-bc}, one LDS
//            transpose, lane c transforms over b -> psi(c + R d);
//   t_p / n multiplies psi in registers;
//   forward: lane c transforms over d (the same registers), twiddles by
//            w_n^{ce}, one LDS transpose, lane e transforms over c and
//            stores the outputs e + R g with |kx| < n/4.
// Each wave owns its LDS rows, so the transposes need only wave-level
// ordering. Each lane keeps its R - 1 twiddles w_n^{jc} in registers for the
// whole kernel (no table reads between the transforms). A workgroup walks row
// groups (gridDim.x apart); each wave loads the next row's inputs and the
// current row's t_p while it computes.

// Raw buffer resource over count complex values at p (gfx9 word 3), and
// 8-byte loads / stores at vector offset voff + scalar offset soff (bytes).
// Accesses past the resource read zero / are dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t wave_rsrc(const float2* p, int count) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float2*>(p), 0, count * 8, 0x00020000);
}
typedef int int2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float2 buf_load(__amdgpu_buffer_rsrc_t r, unsigned voff, int soff) {
  return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, unsigned voff, int soff,
                                          float2 v) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(int2v, v), r, voff, soff, 0);
}

// Row y of plane wave w of a build in compact form: exp(2 pi i (m f x + n f
// y) / n) has X(y, kx) = n exp(2 pi i ((n f y) mod n) / n) at kx = m f and
// zero elsewhere. k = kx mod n. The first row pass of a build forms its
// inputs from this instead of reading a written state: one read and one
// write of the state less per build.
struct PlaneRow {
  int k;
  float2 z;
};
template <int N>
__device__ __forceinline__ PlaneRow row_wave(const BeamWaves& beams, int w, int y,
                                             const float2* __restrict__ twN) {
  const int kx = beams.mn[2 * (beams.b0 + w)] * beams.f;
  const int ky = beams.mn[2 * (beams.b0 + w) + 1] * beams.f;
  int idx = (ky * y) % N;  // |ky| < n/4, y < n <= 2048: fits 32 bits
  if (idx < 0) idx += N;
  const float2 t = twN[idx];  // exp(-2 pi i idx / n)
  return PlaneRow{kx < 0 ? kx + N : kx, make_float2(t.x * (float)N, -t.y * (float)N)};
}

// WT: each wave w reads its own transmission wtrans[w] + soff (waves of
// several specimens in one launch); otherwise every wave reads trans.
// INIT: first slice of a build, the inputs are plane waves (row_wave).
template <int R, bool WT, bool INIT>
__global__ __launch_bounds__(256) void k_row_pass4(float2* __restrict__ state,
                                                   const float2* __restrict__ trans,
                                                   const float2* const* __restrict__ wtrans,
                                                   size_t soff,
                                                   const float2* __restrict__ twN,
                                                   const float2* __restrict__ tw2, BeamWaves beams,
                                                   int groups) {
  constexpr int N = R * R, H2 = N / 2, Q = R / 4, LS = R + 1;
  constexpr int RPW = 64 / R;             // rows per wave
  constexpr int RS = R * LS + 8;          // LDS row stride (float2)
  constexpr int GROUP = 4 * RPW;          // rows per workgroup iteration
  __shared__ float2 lds[4 * RPW * RS];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int j = lane % R, rw = lane / R;
  float2* L = lds + (wv * RPW + rw) * RS;
  float2 s[2 * Q];  // compact inputs of the next row: a < Q, then a >= R - Q
  // Buffer loads from a group's first row; live == false gives a
  // zero-length resource (zeros, no memory traffic).
  const unsigned lane_off = (unsigned)(((wv * RPW + rw) * H2 + j) * 8);
  auto load_src = [&](int g, bool live) {
    const __amdgpu_buffer_rsrc_t rs =
        wave_rsrc(state + (size_t)g * GROUP * H2, live ? GROUP * H2 : 0);
#pragma unroll
    for (int a = 0; a < Q; ++a) s[a] = buf_load(rs, lane_off, R * a * 8);
#pragma unroll
    for (int a = 0; a < Q; ++a) s[Q + a] = buf_load(rs, lane_off, (R * (R - Q + a) - H2) * 8);
  };
  int g = blockIdx.x;
  if constexpr (!INIT) load_src(g, true);
  // this lane's four-step twiddles w_n^{jc}, c = 1 .. R-1 (the same values
  // serve the inverse, conjugated, and the forward transform), held in
  // registers for the whole loop
  float2 tw[R - 1];
#pragma unroll
  for (int c = 1; c < R; ++c) tw[c - 1] = tw2[c * R + j];
  // wait here for the first row and the twiddles (s_waitcnt vmcnt(0)) so
  // that the loop head
  // carries no pending load and never waits for the previous row's stores
  __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll 1
  for (; g < groups; g += gridDim.x) {
    const size_t row = (size_t)g * GROUP + wv * RPW + rw;
    float2 v[R];
    if constexpr (INIT) {
      const PlaneRow pr = row_wave<N>(beams, (int)(row / N), (int)(row & (size_t)(N - 1)), twN);
#pragma unroll
      for (int a = 0; a < R; ++a) {
        const bool on = (a < Q || a >= R - Q) && R * a + j == pr.k;
        v[a] = make_float2(on ? pr.z.x : 0.f, on ? pr.z.y : 0.f);
      }
    } else {
#pragma unroll
      for (int a = 0; a < R; ++a)
        v[a] = a < Q ? s[a] : (a >= R - Q ? s[a - (R - 2 * Q)] : make_float2(0.f, 0.f));
      // Next row's inputs first, then this row's t_p: both are waited for
      // together at the t_p product, after the inverse transform, so no load
      // is still pending (and no store waited for) at the top of the loop.
      const int gn = g + (int)gridDim.x;
      load_src(min(gn, groups - 1), gn < groups);
    }
    float2 tt[R];
    {
      const float2* tb = WT ? wtrans[row / N] + soff : trans;
      const float2* t = tb + (row & (size_t)(N - 1)) * N + j;
#pragma unroll
      for (int d = 0; d < R; ++d) tt[d] = t[R * d];
    }
    dft_reg<R, true>(v);
#pragma unroll
    for (int c = 0; c < R; ++c) L[c * LS + j] = c ? cmulc(v[c], tw[c - 1]) : v[c];
    wave_sync();
#pragma unroll
    for (int b = 0; b < R; ++b) v[b] = L[j * LS + b];
    dft_reg<R, true>(v);
#pragma unroll
    for (int d = 0; d < R; ++d) v[d] = cmul(v[d], tt[d]);
    dft_reg<R, false>(v);
    wave_sync();
#pragma unroll
    for (int e = 0; e < R; ++e) L[e * LS + j] = e ? cmul(v[e], tw[e - 1]) : v[e];
    wave_sync();
#pragma unroll
    for (int c = 0; c < R; ++c) v[c] = L[j * LS + c];
    dft_reg<R, false>(v);
    float2* dst = state + row * H2 + j;
#pragma unroll
    for (int g = 0; g < R; ++g) {
      if (g < Q) dst[R * g] = v[g];
      else if (g >= R - Q) dst[R * g - H2] = v[g];
    }
    wave_sync();
  }
}

// ---------------------------------------------------------------------------
// Four-step column pass for n = R^2 over tiles of TC adjacent compact
// columns (TC R threads); lane (b, c) = (tid / TC, tid % TC), so each load or
// store instruction covers TC contiguous columns of 64 / TC rows.
//   forward : lane (b, c) transforms y = R a + b over a, twiddles by
//             w_n^{b k1}, LDS transpose, lane (k1, c) transforms over b and
//             keeps ky = k1 + R k2 with |ky| < n/4 (the rest is cut by M);
//   P_p(kx) P_p(ky) M / n in registers;
//   inverse : lane (k1, c) transforms over k2 (inputs outside the half band
//             are zero), twiddles by w_n^{-k1 m1}, LDS transpose, lane
//             (m1, c) transforms over k1 and stores y = m1 + R m2.
// A workgroup walks tiles (gridDim.x apart), loading the next tile while it
// computes the current one.
#ifndef PRISM_COL4_TC32
#define PRISM_COL4_TC32 16   // columns per tile at n = 1024
#endif

template <int R, int TC>
__global__ __launch_bounds__(TC * R) __attribute__((amdgpu_waves_per_eu(2))) void k_col_pass4(float2* __restrict__ state,
                                                   const float2* __restrict__ prop,
                                                   const float2* __restrict__ tw2, int tiles) {
  constexpr int N = R * R, H2 = N / 2, Q = R / 4, LS = R + 1;
  constexpr int NT = TC * R;
  constexpr int TILES = H2 / TC;         // tiles per wave
  constexpr int CS = R * LS + 16 / TC;   // LDS column stride (float2): the TC
                                         // columns of a 16-lane group hit
                                         // distinct banks
  __shared__ float2 twl[R * R];
  __shared__ float2 pyl[H2];  // P_p(ky) for |ky| < n/4, compact order
  __shared__ float2 lds[TC * CS];
  const int tid = threadIdx.x, c = tid % TC, b = tid / TC;
  for (int i = tid; i < R * R; i += NT) twl[i] = tw2[i];
  for (int i = tid; i < H2; i += NT) pyl[i] = prop[i < H2 / 2 ? i : i + H2];
  float2* L = lds + c * CS;
  const float2* twb = twl + b;
  const float inv_n = 1.0f / (float)N;

  // Buffer accesses: one wave function per resource, lane (b, c) at a fixed
  // vector byte offset, the row and tile offsets in scalar registers.
  const unsigned lane_off = (unsigned)(b * H2 + c) * 8u;
  float2 s[R];  // next tile's column elements y = R a + b
  // live == false: a zero-length resource, the loads return zeros and
  // touch no memory (keeps the instruction stream of every iteration alike)
  auto load_tile = [&](int tile, bool live) {
    const int w = tile / TILES, c0 = (tile % TILES) * TC;
    const __amdgpu_buffer_rsrc_t rs =
        wave_rsrc(state + (size_t)w * N * H2, live ? N * H2 : 0);
#pragma unroll
    for (int a = 0; a < R; ++a) s[a] = buf_load(rs, lane_off, (c0 + R * a * H2) * 8);
  };
  // Tiles g, g + gridDim.x, ..., with g the XCD-grouped workgroup index: workgroups resident on one XCD at the same time take
  // adjacent tiles, which share the 128-byte lines of every row.
  const int g = xcd_tile(blockIdx.x, gridDim.x), nwg = gridDim.x;
  load_tile(g, true);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): no load pending at the loop head
  __syncthreads();
#pragma unroll 1
  for (int tile = g; tile < tiles; tile += nwg) {
    const int w = tile / TILES, c0 = (tile % TILES) * TC;
    float2 v[R];
#pragma unroll
    for (int a = 0; a < R; ++a) v[a] = s[a];
    // the next tile is in flight during this one
    load_tile(min(tile + nwg, tiles - 1), tile + nwg < tiles);
    dft_reg<R, false>(v);
#pragma unroll
    for (int k1 = 0; k1 < R; ++k1) L[k1 * LS + b] = v[k1];
    __syncthreads();
    const int jj = c0 + c;
    const int kx = jj < H2 / 2 ? jj : jj - H2;
    // P_p(kx) from the same LDS table as P_p(ky) (compact index jj): a
    // global load here would be waited for together with the next tile's
    // loads (vector memory counts complete in order)
    const float2 px = cscale(pyl[jj], inv_n);
    // the twiddle w_n^{bb k1} is applied on the reading side (the table is
    // symmetric, so the reading lane k1 = b indexes it by bb): the element
    // and twiddle reads go out together instead of one twiddle read waited
    // for per LDS write
    {
      float2 tw[R - 1];
#pragma unroll
      for (int bb = 0; bb < R; ++bb) v[bb] = L[b * LS + bb];
#pragma unroll
      for (int bb = 1; bb < R; ++bb) tw[bb - 1] = twb[bb * R];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int bb = 1; bb < R; ++bb) v[bb] = cmul(v[bb], tw[bb - 1]);
    }
    dft_reg<R, false>(v);  // lane (k1 = b, c): ky index b + R k2
    {
      // P_p(ky) of the kept rows, read together; the band limit is a select
      // on the computed product (no branch per element)
      float2 p2[2 * Q];
#pragma unroll
      for (int k2 = 0; k2 < 2 * Q; ++k2) {
        const int kyi = b + R * (k2 < Q ? k2 : k2 + R - 2 * Q);
        p2[k2] = pyl[k2 < Q ? kyi : kyi - H2];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k2 = 0; k2 < R; ++k2) {
        if (k2 < Q || k2 >= R - Q) {
          const int kyi = b + R * k2;
          const int ky = kyi < H2 ? kyi : kyi - N;
          float2 m = cmul(cmul(v[k2], px), p2[k2 < Q ? k2 : k2 - (R - 2 * Q)]);
          asm volatile("" : "+v"(m.x), "+v"(m.y));
          const bool keep = 16 * (kx * kx + ky * ky) < N * N;
          v[k2] = make_float2(keep ? m.x : 0.f, keep ? m.y : 0.f);
        } else {
          v[k2] = make_float2(0.f, 0.f);
        }
      }
    }
    dft_reg<R, true>(v);  // over k2 -> m1
    __syncthreads();
#pragma unroll
    for (int m1 = 0; m1 < R; ++m1) L[m1 * LS + b] = v[m1];
    __syncthreads();
    {
      float2 tw[R - 1];
#pragma unroll
      for (int k1 = 0; k1 < R; ++k1) v[k1] = L[b * LS + k1];
#pragma unroll
      for (int k1 = 1; k1 < R; ++k1) tw[k1 - 1] = twb[k1 * R];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k1 = 1; k1 < R; ++k1) v[k1] = cmulc(v[k1], tw[k1 - 1]);
    }
    dft_reg<R, true>(v);  // lane (m1 = b, c): y = b + R m2
    const __amdgpu_buffer_rsrc_t rd = wave_rsrc(state + (size_t)w * N * H2, N * H2);
#pragma unroll
    for (int m2 = 0; m2 < R; ++m2) buf_store(rd, lane_off, (c0 + R * m2 * H2) * 8, v[m2]);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Row pass for the grids that are not a square of a register DFT length
// (fft_steps.hpp: three or two register DFT steps per transform, one LDS
// exchange between them). L lanes hold a row:
//   inverse: comb order in (only |kx| < n/4, i.e. registers a < R1/4 and
//            a >= 3 R1/4, are nonzero), block order out;
//   t_p / n multiplies psi in registers;
//   forward: block order in, comb order out, the half band stored.
// Twiddles stay in registers for the whole kernel; a workgroup walks row
// groups (gridDim.x apart) with the next group's inputs and the current
// group's t_p in flight during the transforms.
// Bound: VALU issue and memory together (n = 1536: 64 VALU instructions per row
// element, issue 70 % busy at 5.4 TB/s in a launch of 10 waves alone; n = 2048:
// 56 % at 5.8 TB/s, half of it t_p). R1 values per lane keep the exchanges at
// two per transform, against three LDS round trips and a workgroup barrier pair
// each for the radix-8 LDS stages this replaces: 99 instead of 209 us per 20-
// and 27-wave launch at n = 1536 (3.8 against 2.6 TB/s), 123 instead of 208 us
// for 11 and 14 waves at n = 2048.
// WT and INIT as in the four-step pass.
template <int N, bool WT, bool INIT>
__global__ __launch_bounds__(GridSteps<N>::ROW_NT) __attribute__((amdgpu_waves_per_eu(2)))
void k_row_steps(float2* __restrict__ state, const float2* __restrict__ trans,
                 const float2* const* __restrict__ wtrans, size_t soff,
                 const float2* __restrict__ twN, BeamWaves beams, int groups) {
  using GS = GridSteps<N>;
  using ST = typename GS::Row;
  constexpr int H2 = N / 2, R1 = ST::R1, L = ST::L, Q = R1 / 4, D = ST::D, MB = ST::MB;
  constexpr int GROUP = GS::ROW_NT / L;  // rows per workgroup iteration
  static_assert(N % GROUP == 0, "a row group lies inside one wave function");
  __shared__ float2 lds[GROUP * GS::ROW_RS];
  __shared__ float2 tab[ST::TLN];
  const int tid = threadIdx.x, b = tid % L, rw = tid / L;
  float2* Lr = lds + rw * GS::ROW_RS;
  const unsigned row_off = (unsigned)(rw * H2 + b) * 8u, t_off = (unsigned)(rw * N + b) * 8u;

  float2 s[2 * Q];  // compact inputs of the next row: a < Q, then a >= R1 - Q
  auto load_src = [&](int g, bool live) {
    const __amdgpu_buffer_rsrc_t rs =
        wave_rsrc(state + (size_t)g * GROUP * H2, live ? GROUP * H2 : 0);
#pragma unroll
    for (int a = 0; a < Q; ++a) s[a] = buf_load(rs, row_off, L * a * 8);
#pragma unroll
    for (int a = 0; a < Q; ++a) s[Q + a] = buf_load(rs, row_off, (L * (R1 - Q + a) - H2) * 8);
  };
  int g = blockIdx.x;
  if constexpr (!INIT) load_src(g, true);
  typename ST::Tw tw;
  ST::load_twiddles(twN, b, tab, tid, GS::ROW_NT, tw);
  if constexpr (!INIT) settle(s);
  if constexpr (ST::TLDS) __syncthreads();
#pragma unroll 1
  for (; g < groups; g += gridDim.x) {
    const int w = g * GROUP / N, y0 = g * GROUP - w * N;  // uniform
    float2 v[R1];
    if constexpr (INIT) {
      const PlaneRow pr = row_wave<N>(beams, w, y0 + rw, twN);
#pragma unroll
      for (int a = 0; a < R1; ++a) {
        const bool on = (a < Q || a >= R1 - Q) && L * a + b == pr.k;
        v[a] = make_float2(on ? pr.z.x : 0.f, on ? pr.z.y : 0.f);
      }
    } else {
#pragma unroll
      for (int a = 0; a < R1; ++a)
        v[a] = a < Q ? s[a] : (a >= R1 - Q ? s[a - (R1 - 2 * Q)] : make_float2(0.f, 0.f));
      const int gn = g + (int)gridDim.x;
      load_src(min(gn, groups - 1), gn < groups);
    }
    float2 tt[R1];
    {
      const float2* tb = (WT ? wtrans[w] + soff : trans) + (size_t)y0 * N;
      const __amdgpu_buffer_rsrc_t rt = wave_rsrc(tb, GROUP * N);
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int d = 0; d < D; ++d) tt[i * D + d] = buf_load(rt, t_off, (L * i + N / D * d) * 8);
    }
    if constexpr (!(ST::TWO && R1 == 32))  // (no registers left for it)
      __builtin_amdgcn_sched_barrier(0);   // the loads go out before the first transform
    ST::template comb_to_block<true>(v, Lr, b, tw);
#pragma unroll
    for (int e = 0; e < R1; ++e) v[e] = cmul(v[e], tt[e]);
    ST::template block_to_comb<false>(v, Lr, b, tw);
    const __amdgpu_buffer_rsrc_t rd = wave_rsrc(state + (size_t)g * GROUP * H2, GROUP * H2);
#pragma unroll
    for (int a = 0; a < R1; ++a) {
      if (a < Q) buf_store(rd, row_off, L * a * 8, v[a]);
      else if (a >= R1 - Q) buf_store(rd, row_off, (L * a - H2) * 8, v[a]);
    }
  }
}

// Column pass of the same grids over tiles of TC adjacent compact columns
// (lane (b, c) = (tid / TC, tid % TC)): forward y-transform from comb to
// block order, P_p(kx) P_p(ky) M / n in registers with the rows |ky| >= n/4
// cut, inverse back to comb order. Workgroups walk tiles (gridDim.x apart,
// XCD-grouped as in the four-step pass) with the next tile in flight.
// Bound: the workgroup's phases (loads, VALU, LDS exchanges) overlap only
// through the prefetch, since one workgroup fills a compute unit's registers
// (n = 1536: VALU issue 32 % busy, 3.4 TB/s, waves waiting for loads or at
// barriers 30 % of their cycles); 102 instead of 174 us per 20- and
// 27-wave launch at n = 1536, 101 instead of 155 us for 11 and 14 waves at n =
// 2048, against the radix-8 LDS stages this replaces.
template <int N>
__global__ __launch_bounds__(GridSteps<N>::TC * GridSteps<N>::L)
__attribute__((amdgpu_waves_per_eu(2))) void k_col_steps(float2* __restrict__ state,
                                                         const float2* __restrict__ prop,
                                                         const float2* __restrict__ twN,
                                                         int tiles) {
  using GS = GridSteps<N>;
  using ST = typename GS::Col;
  constexpr int H2 = N / 2, R1 = ST::R1, L = ST::L, D = ST::D, MB = ST::MB, QD = D / 4;
  constexpr int TC = GS::TC, NT = TC * L, TILES = H2 / TC;
  static_assert(H2 % TC == 0, "whole tiles");
  __shared__ float2 pyl[H2];  // P_p(ky) for |ky| < n/4, compact order
  __shared__ float2 lds[TC * GS::COL_RS];
  __shared__ float2 tab[ST::TLN];
  const int tid = threadIdx.x, c = tid % TC, b = tid / TC;
  for (int i = tid; i < H2; i += NT) pyl[i] = prop[i < H2 / 2 ? i : i + H2];
  float2* Lc = lds + c * GS::COL_RS;
  const float inv_n = 1.0f / (float)N;
  const unsigned lane_off = (unsigned)(b * H2 + c) * 8u;
  float2 s[R1];  // next tile's column elements y = L a + b
  auto load_tile = [&](int tile, bool live) {
    const int w = tile / TILES, c0 = (tile % TILES) * TC;
    const __amdgpu_buffer_rsrc_t rs =
        wave_rsrc(state + (size_t)w * N * H2, live ? N * H2 : 0);
#pragma unroll
    for (int a = 0; a < R1; ++a) s[a] = buf_load(rs, lane_off, (c0 + L * a * H2) * 8);
  };
  int tile = xcd_tile(blockIdx.x, gridDim.x);
  load_tile(tile, true);
  typename ST::Tw tw;
  ST::load_twiddles(twN, b, tab, tid, NT, tw);
  settle(s);
  __syncthreads();
#pragma unroll 1
  for (; tile < tiles; tile += gridDim.x) {
    const int w = tile / TILES, c0 = (tile % TILES) * TC;
    float2 v[R1];
#pragma unroll
    for (int a = 0; a < R1; ++a) v[a] = s[a];
    const int next = tile + (int)gridDim.x;
    load_tile(min(next, tiles - 1), next < tiles);
    if constexpr (!(ST::TWO && R1 == 32))  // (no registers left for it)
      __builtin_amdgcn_sched_barrier(0);   // the loads go out before the first transform
    ST::template comb_to_block<false>(v, Lc, b, tw);
    const int jj = c0 + c;
    const int kx = jj < H2 / 2 ? jj : jj - H2;
    const float2 px = cscale(pyl[jj], inv_n);
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (d < QD || d >= D - QD) {
          const int kyi = b + L * i + N / D * d;
          const int ky = d < QD ? kyi : kyi - N;
          const float2 m = cmul(cmul(v[i * D + d], px), pyl[d < QD ? kyi : kyi - H2]);
          const bool keep = 16 * (kx * kx + ky * ky) < N * N;
          v[i * D + d] = make_float2(keep ? m.x : 0.f, keep ? m.y : 0.f);
        } else {
          v[i * D + d] = make_float2(0.f, 0.f);
        }
      }
    ST::template block_to_comb<true>(v, Lc, b, tw);
    const __amdgpu_buffer_rsrc_t rd = wave_rsrc(state + (size_t)w * N * H2, N * H2);
#pragma unroll
    for (int a = 0; a < R1; ++a) buf_store(rd, lane_off, (c0 + L * a * H2) * 8, v[a]);
  }
}

// ---------------------------------------------------------------------------
// LDS passes: the row and column pass of few waves on the grids of k_row_steps /
// k_col_steps (multislice of a few probes, few_waves), and the last column pass
// of multislice on every grid. 8 values per thread: a single wave's pass is a
// chain of short stages over many threads, where the step passes have 16 to 32
// values per lane and a wave function gives them few workgroups (n = 512, one
// wave: row pass 7 us instead of 12, column pass 9 instead of 13). Their
// arithmetic is the exact form (EX) of fft_lds.hpp: with the products of table
// twiddles and plain constants the detector sums' error is three times larger (n =
// 768, 40 slices: 9.0e-6; exact 1.2e-6; step passes 5.2e-6).
//
// Row pass: NSEQ rows of length n per workgroup (PRISM_ROW_ELEMS complex in
// LDS). The inverse x-transform runs 8, 8^MID, RL and the forward one
// RL, 8^MID, 8 (PairedPlan): the inverse's first stage reads the compact row
// straight from HBM (its inputs at |kx| >= n/4 are zero), its last stage
// stays in registers, is multiplied by t_p / n and feeds the forward's first
// stage, and the forward's last stage stores only the kept half band.
template <int N>
__global__ __launch_bounds__(kRowNT) void k_row_lds(float2* __restrict__ state,
                                                    const float2* __restrict__ trans,
                                                    const float2* __restrict__ twN) {
  constexpr int NT = kRowNT;
  constexpr int NSEQ = row_nseq(N);
  constexpr int H2 = N / 2, E8 = N / 8;
  using B = RowBatch<N, NSEQ>;
  using PP = PairedPlan<N>;
  constexpr int RL = PP::RL, NSL = N / PP::RL;
  using S8 = StageShape<B, 8, NT>;
  using SL = StageShape<B, RL, NT>;
  __shared__ float2 lds[lds_padded(NSEQ * N)];
  __shared__ float2 tw[N];
  const int tid = threadIdx.x;
  const size_t row0 = (size_t)blockIdx.x * NSEQ;
  load_twiddles<N, NT>(tw, twN, tid);
  {
    // inverse, first stage (span 1): inputs j + r n/8, nonzero for r in {0,1,6,7}
    float2 v[S8::PER][8];
#pragma unroll
    for (int p = 0; p < S8::PER; ++p) {
      const int b = tid + p * NT;
      v[p][2] = v[p][3] = v[p][4] = v[p][5] = make_float2(0.f, 0.f);
      if (S8::GUARD && b >= S8::TOT) continue;  // no butterfly (stage_out skips it too)
      int sq, j;
      stage_coords<B, S8::NB>(b, sq, j);
      const float2* src = state + (row0 + sq) * H2 + j;
      v[p][0] = src[0];
      v[p][1] = src[E8];
      v[p][6] = src[2 * E8];
      v[p][7] = src[3 * E8];
    }
    stage_out<B, 8, 1, NT, true, true>(lds, tid, v);
  }
  __syncthreads();
  fft_radix8_run<B, NT, true, 8, PP::MID, true>(lds, tw, tid);
  float2 v[SL::PER][RL];
  stage_in<B, RL, NSL, NT, true, true>(lds, tw, tid, v);
#pragma unroll
  for (int p = 0; p < SL::PER; ++p) {
    const int b = tid + p * NT;
    if (SL::GUARD && b >= SL::TOT) continue;
    int sq, j;
    stage_coords<B, SL::NB>(b, sq, j);
    dft<RL, true, true>(v[p]);
    const float2* t = trans + (size_t)((row0 + sq) % (size_t)N) * N + j;
#pragma unroll
    for (int r = 0; r < RL; ++r) v[p][r] = cmul(v[p][r], t[r * NSL]);
  }
  __syncthreads();
  stage_out<B, RL, 1, NT, false, true>(lds, tid, v);
  __syncthreads();
  fft_radix8_run<B, NT, false, RL, PP::MID, true>(lds, tw, tid);
  {
    // forward, last stage (span n/8): outputs j + r n/8, kept for r in {0,1,6,7}
    float2 w[S8::PER][8];
    stage_in<B, 8, E8, NT, false, true>(lds, tw, tid, w);
#pragma unroll
    for (int p = 0; p < S8::PER; ++p) {
      const int b = tid + p * NT;
      if (S8::GUARD && b >= S8::TOT) continue;
      int sq, j;
      stage_coords<B, S8::NB>(b, sq, j);
      dft8<false, true>(w[p]);
      float2* dst = state + (row0 + sq) * H2 + j;
      dst[0] = w[p][0];
      dst[E8] = w[p][1];
      dst[2 * E8] = w[p][6];
      dst[3 * E8] = w[p][7];
    }
  }
}

// Column pass over a tile of TC adjacent compact columns, held [y][c] in LDS:
// the forward y-transform reads straight from HBM, its last stage stays in
// registers for the propagator and band limit and feeds the inverse, whose last
// stage stores. DETECT (last slice of multislice): instead of the inverse, I =
// |Psi|^2 / n^2 gives per-tile detector partial sums.
template <int N, bool DETECT>
__global__ __launch_bounds__(col_nt(N)) void k_col_lds(float2* __restrict__ state,
                                                       const float2* __restrict__ prop,
                                                       const float2* __restrict__ twN, DetBins bins,
                                                       double* __restrict__ partial) {
  constexpr int TC = col_tc(N), NT = col_nt(N);
  constexpr int H2 = N / 2, Q = N / 4, E8 = N / 8;
  constexpr int TILES = H2 / TC;
  constexpr int NW = NT / 64;
  using B = Batch<N, TC, TC, 0, 1, TC, true>;
  using PP = PairedPlan<N>;
  constexpr int RL = PP::RL, NSL = N / PP::RL;
  using S8 = StageShape<B, 8, NT>;
  using SL = StageShape<B, RL, NT>;
  __shared__ float2 lds[lds_padded(TC * N)];
  __shared__ float2 tw[N];
  const int tid = threadIdx.x;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int w = tile / TILES, c0 = (tile % TILES) * TC;
  float2* base = state + (size_t)w * N * H2 + c0;
  load_twiddles<N, NT>(tw, twN, tid);
  {
    float2 v[S8::PER][8];
#pragma unroll
    for (int p = 0; p < S8::PER; ++p) {
      const int b = tid + p * NT;
      if (S8::GUARD && b >= S8::TOT) continue;  // no butterfly (stage_out skips it too)
      int c, j;
      stage_coords<B, S8::NB>(b, c, j);
#pragma unroll
      for (int r = 0; r < 8; ++r) v[p][r] = base[(size_t)(j + r * E8) * H2 + c];
    }
    stage_out<B, 8, 1, NT, false, !DETECT>(lds, tid, v);
  }
  __syncthreads();
  fft_radix8_run<B, NT, false, 8, PP::MID, !DETECT>(lds, tw, tid);
  float2 v[SL::PER][RL];
  stage_in<B, RL, NSL, NT, false, !DETECT>(lds, tw, tid, v);
  const float inv_n = 1.0f / (float)N;
#pragma unroll
  for (int p = 0; p < SL::PER; ++p) {
    const int b = tid + p * NT;
    if (SL::GUARD && b >= SL::TOT) continue;
    int c, j;
    stage_coords<B, SL::NB>(b, c, j);
    dft<RL, false, !DETECT>(v[p]);
    const int jj = c0 + c;
    const int kx = jj < Q ? jj : jj - H2;
    const float2 px = prop[kx < 0 ? kx + N : kx];
#pragma unroll
    for (int r = 0; r < RL; ++r) {
      const int yi = j + r * NSL;
      const int ky = signed_k(yi, N);
      const int k2 = kx * kx + ky * ky;
      if (16 * k2 < N * N) {
        float2 z = cmul(cmul(v[p][r], px), prop[yi]);
        v[p][r] = DETECT ? z : cscale(z, inv_n);
      } else {
        v[p][r] = make_float2(0.f, 0.f);
      }
    }
  }
  if constexpr (!DETECT) {
    __syncthreads();
    stage_out<B, RL, 1, NT, true, true>(lds, tid, v);
    __syncthreads();
    fft_radix8_run<B, NT, true, RL, PP::MID, true>(lds, tw, tid);
    float2 u[S8::PER][8];
    stage_in<B, 8, E8, NT, true, true>(lds, tw, tid, u);
#pragma unroll
    for (int p = 0; p < S8::PER; ++p) {
      const int b = tid + p * NT;
      if (S8::GUARD && b >= S8::TOT) continue;
      int c, j;
      stage_coords<B, S8::NB>(b, c, j);
      dft8<true, true>(u[p]);
#pragma unroll
      for (int r = 0; r < 8; ++r) base[(size_t)(j + r * E8) * H2 + c] = u[p][r];
    }
  } else {
    __shared__ double red[8][NW];
    const double inv_n2 = 1.0 / ((double)N * (double)N);
    for (int j0 = 0; j0 < bins.n; j0 += 8) {
      double acc[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[q] = 0.0;
#pragma unroll
      for (int p = 0; p < SL::PER; ++p) {
        const int b = tid + p * NT;
        if (SL::GUARD && b >= SL::TOT) continue;
        int c, j;
        stage_coords<B, SL::NB>(b, c, j);
        const int jj = c0 + c;
        const int kx = jj < Q ? jj : jj - H2;
#pragma unroll
        for (int r = 0; r < RL; ++r) {
          const int ky = signed_k(j + r * NSL, N);
          const int k2 = kx * kx + ky * ky;
          const double I = ((double)v[p][r].x * v[p][r].x + (double)v[p][r].y * v[p][r].y) * inv_n2;
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const int jb = j0 + q;
            if (jb < bins.n && k2 >= bins.lo[jb] && k2 < bins.hi[jb]) acc[q] += I;
          }
        }
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const double sum = wave_sum(acc[q]);
        if ((tid & 63) == 0) red[q][tid >> 6] = sum;
      }
      __syncthreads();
      if (tid < 8 && j0 + tid < bins.n) {
        double sum = 0.0;
        for (int wv = 0; wv < NW; ++wv) sum += red[tid][wv];
        partial[((size_t)w * TILES + (tile % TILES)) * bins.n + j0 + tid] = sum;
      }
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// Incident multislice probe, built per compact column in Fourier space and
// brought to X(y, kx) by an inverse FFT along y:
//   X0(y, kx) = norm * sum_ky A e^{-i chi} e^{-2 pi i q.(r0 - s)} e^{2 pi i ky y / n}
// with norm = 1 / sqrt(N_A), chi at k - k_t and s the tilt's entrance offset.
// The aperture comes as one kx interval per row (decided on the host).
// Phases are evaluated in FP64.
template <int N>
__global__ __launch_bounds__(col_nt(N)) void k_probe_init(float2* __restrict__ state,
                                                          const double* __restrict__ probe_xy,
                                                          int p0, ProbeOptics po,
                                                          const int2* __restrict__ aper,
                                                          const float2* __restrict__ twN) {
  constexpr int TC = col_tc(N), NT = col_nt(N);
  constexpr int H2 = N / 2, Q = N / 4;
  constexpr int TILES = H2 / TC;
  using B = Batch<N, TC, TC, 0, 1, TC, true>;
  __shared__ float2 lds[lds_padded(TC * N)];
  __shared__ float2 tw[N];
  const int tid = threadIdx.x;
  const int tile = blockIdx.x;
  const int w = tile / TILES, c0 = (tile % TILES) * TC;
  const double x0 = probe_xy[2 * (size_t)(p0 + w)] - po.sx;
  const double y0 = probe_xy[2 * (size_t)(p0 + w) + 1] - po.sy;
  load_twiddles<N, NT>(tw, twN, tid);
  const double dq2 = po.dq * po.dq;
  for (int e = tid; e < TC * N; e += NT) {
    const int y = e / TC, c = e % TC;
    const int jj = c0 + c;
    const int kx = jj < Q ? jj : jj - H2;
    const int ky = signed_k(y, N);
    const int2 row = aper[ky + N / 2];
    float2 v = make_float2(0.f, 0.f);
    if (kx >= row.x && kx <= row.y) {
      const double dx = (double)kx - po.ktx, dy = (double)ky - po.kty;
      const double q2 = (dx * dx + dy * dy) * dq2;
      double t = -(0.5 * po.lam * q2 * po.C1 + 0.25 * po.lam * po.lam * po.lam * q2 * q2 * po.C3) -
                 ((double)kx * x0 + (double)ky * y0) * po.dq;
      t -= floor(t);
      double s, co;
      sincospi(2.0 * t, &s, &co);
      v = make_float2((float)(co * po.norm), (float)(s * po.norm));
    }
    lds[lpad(e)] = v;
  }
  __syncthreads();
  fft_lds<B, NT, true>(lds, tw, tid);
  float2* base = state + (size_t)w * N * H2 + c0;
  for (int e = tid; e < TC * N; e += NT) {
    const int y = e / TC, c = e % TC;
    base[(size_t)y * H2 + c] = lds[lpad(e)];
  }
}

// ---------------------------------------------------------------------------
// Quarter-size exit wave: S(i', j') = psi_H(2 i', 2 j')
//   = (1/n) sum_kx X(2 j', kx) exp(2 pi i kx i' / (n/2)),
// an n/2-point inverse FFT of the even compact rows (already in n/2
// fftfreq order).
template <int N>
__global__ __launch_bounds__(256) void k_extract(const float2* __restrict__ state,
                                                 float2* __restrict__ S,
                                                 const float2* __restrict__ twH) {
  constexpr int NT = 256;
  constexpr int H2 = N / 2;
  constexpr int NSEQ = ext_nseq(N);
  using B = RowBatch<H2, NSEQ>;
  __shared__ float2 lds[lds_padded(NSEQ * H2)];
  __shared__ float2 tw[H2];
  const int tid = threadIdx.x;
  const size_t g0 = (size_t)blockIdx.x * NSEQ;
  load_twiddles<H2, NT>(tw, twH, tid);
  for (int e = tid; e < NSEQ * H2; e += NT) {
    const int s = e / H2, i = e % H2;
    const size_t g = g0 + s;
    const size_t w = g / H2, jp = g % H2;
    lds[lpad(e)] = state[(w * N + 2 * jp) * H2 + i];
  }
  __syncthreads();
  fft_lds<B, NT, true>(lds, tw, tid);
  const float inv_n = 1.0f / (float)N;
  for (int e = tid; e < NSEQ * H2; e += NT) {
    const int s = e / H2, i = e % H2;
    S[(g0 + s) * H2 + i] = cscale(lds[lpad(e)], inv_n);
  }
}

__global__ void k_reduce_partials(const double* __restrict__ partial, int nwaves, int tiles,
                                  int n_det, double* __restrict__ out, OutAcc acc) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nwaves * n_det) return;
  const int w = i / n_det, j = i % n_det;
  double s = 0.0;
  for (int t = 0; t < tiles; ++t) s += partial[((size_t)w * tiles + t) * n_det + j];
  put_out(out + i, s, acc);
}

inline unsigned blocks_for(size_t n, unsigned bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

// ---------------------------------------------------------------------------
// Launchers (sizes are validated by the host plan before any call).

hipError_t launch_twiddles(float2* tw, int L, hipStream_t st) {
  hipLaunchKernelGGL(k_twiddles, dim3(blocks_for(L, 256)), dim3(256), 0, st, tw, L);
  return hipGetLastError();
}

hipError_t launch_transmission(const float* phase, float2* trans, size_t count, float scale,
                               hipStream_t st) {
  hipLaunchKernelGGL(k_transmission, dim3(blocks_for(count, 256)), dim3(256), 0, st, phase, trans,
                     count, scale);
  return hipGetLastError();
}

hipError_t launch_prop_lut(float2* lut, int n, int H, const double* thick_dev, double lam,
                           double dq, hipStream_t st) {
  hipLaunchKernelGGL(k_prop_lut, dim3(blocks_for((size_t)n * H, 256)), dim3(256), 0, st, lut, n,
                     H, thick_dev, lam, dq);
  return hipGetLastError();
}

#define PRISM_DISPATCH_N(n, CALL) \
  switch (n) {                    \
    case 128: CALL(128); break;   \
    case 192: CALL(192); break;   \
    case 256: CALL(256); break;   \
    case 384: CALL(384); break;   \
    case 512: CALL(512); break;   \
    case 576: CALL(576); break;   \
    case 768: CALL(768); break;   \
    case 1024: CALL(1024); break; \
    case 1152: CALL(1152); break; \
    case 1536: CALL(1536); break; \
    case 2048: CALL(2048); break; \
    default: return hipErrorInvalidValue; \
  }

// The grids of k_row_steps / k_col_steps.
#define PRISM_DISPATCH_STEPS(n, CALL) \
  switch (n) {                        \
    case 128: CALL(128); break;       \
    case 192: CALL(192); break;       \
    case 384: CALL(384); break;       \
    case 512: CALL(512); break;       \
    case 576: CALL(576); break;       \
    case 768: CALL(768); break;       \
    case 1152: CALL(1152); break;     \
    case 1536: CALL(1536); break;     \
    case 2048: CALL(2048); break;     \
    default: return hipErrorInvalidValue; \
  }

// The grids of k_row_lds / k_col_lds<N, false> (few_waves).
#define PRISM_DISPATCH_FEW(n, CALL) \
  switch (n) {                      \
    case 128: CALL(128); break;     \
    case 192: CALL(192); break;     \
    case 384: CALL(384); break;     \
    case 512: CALL(512); break;     \
    case 576: CALL(576); break;     \
    case 768: CALL(768); break;     \
    case 1152: CALL(1152); break;   \
    case 1536: CALL(1536); break;   \
    default: return hipErrorInvalidValue; \
  }

hipError_t launch_twiddles2(float2* tw2, int n, hipStream_t st) {
  const int R = four_step_radix(n);
  if (R == 0) return hipSuccess;
  hipLaunchKernelGGL(k_twiddles2, dim3(blocks_for((size_t)R * R, 256)), dim3(256), 0, st, tw2, R);
  return hipGetLastError();
}

int four_step_radix(int n) { return n == 1024 ? 32 : (n == 256 ? 16 : 0); }

// Most waves of a multislice call for which the LDS passes are faster than the
// step passes of the same grid: the step passes' longer chain per lane is hidden
// once a launch has about two workgroups per compute unit, sooner where their
// rows are long and LDS tiles take most of a compute unit's LDS. Measured with 12
// slices, step / LDS passes in us: n = 128, 8 probes 138 / 127, 48 probes 162 /
// 162; n = 192, 8 probes 182 / 151, 96 probes 387 / 403; n = 384, 1 probe 234 /
// 179, 64 probes 611 / 608; n = 512, 1 probe 266 / 180, 16 probes 477 / 440, 64
// probes 794 / 856; n = 576, 1 probe 241 / 209, 8 probes 399 / 405; n = 768, 1
// probe 322 / 247, 16 probes 700 / 660, 32 probes 1074 / 1137; n = 1152, 1 probe
// 398 / 356, 4 probes 642 / 656; n = 1536, 1 probe 531 / 514, 2 probes 563 / 616;
// n = 2048, 1 probe 741 / 744.
bool few_waves(int n, int nwaves) {
  const int most = n == 128 ? 32 : n == 192 ? 64 : n == 384 || n == 512 ? 48
                 : n == 576 ? 6 : n == 768 ? 16 : n == 1152 ? 2 : n == 1536 ? 1 : 0;
  return nwaves <= most;
}

// Workgroups of a slice-pass launch over `units` row groups or tiles: the 256
// compute units times the workgroups one holds (per_cu), so that every
// workgroup walks units / grid of them and no last round runs nearly empty;
// a whole multiple of that where one would walk over maxit units or fewer
// than min_wgs would be launched; at most one per unit.
static unsigned pass_grid(int units, int per_cu, int maxit, int min_wgs) {
  const long long slots = 256LL * per_cu;
  const long long rounds = std::max((units + slots * maxit - 1) / (slots * maxit),
                                    (min_wgs + slots - 1) / slots);
  return (unsigned)std::min<long long>(units, slots * rounds);
}

hipError_t launch_row_pass(float2* state, int nwaves, int n, const float2* trans_p,
                           const float2* twN, const float2* tw2, const LaunchTuning& tune,
                           hipStream_t st, const BeamWaves* init, const float2* const* wtrans,
                           size_t soff, bool few) {
  const bool wt = wtrans != nullptr;
  const BeamWaves bw = init ? *init : BeamWaves{nullptr, 0, 0};
  if (init && wt) return hipErrorInvalidValue;  // first slices run one specimen at a time
  if (n == 1024 || n == 256) {
    // row groups of 4 waves x 64/R rows; two (R = 32) or three workgroups fit
    // a compute unit's registers
    const int R = n == 1024 ? 32 : 16;
    const int groups = nwaves * n / (4 * 64 / R);
    const dim3 grid(pass_grid(groups, R == 32 ? 2 : 3, tune.row_iters, tune.row_min_wg));
#define ROW4(RR, WW, II)                                                                      \
  hipLaunchKernelGGL((k_row_pass4<RR, WW, II>), grid, dim3(256), 0, st, state, trans_p, wtrans, \
                     soff, twN, tw2, bw, groups)
    if (R == 32) {
      if (init) ROW4(32, false, true);
      else if (wt) ROW4(32, true, false);
      else ROW4(32, false, false);
    } else {
      if (init) ROW4(16, false, true);
      else if (wt) ROW4(16, true, false);
      else ROW4(16, false, false);
    }
#undef ROW4
    return hipGetLastError();
  }
  if (few && (wt || init)) return hipErrorInvalidValue;  // multislice only
  if (few) {
#define ROWL(NN)                                                                               \
  hipLaunchKernelGGL(k_row_lds<NN>, dim3((unsigned)((size_t)nwaves * NN / row_nseq(NN))),      \
                     dim3(kRowNT), 0, st, state, trans_p, twN)
    PRISM_DISPATCH_FEW(n, ROWL)
#undef ROWL
    return hipGetLastError();
  }
#define ROW1(NN, WW, II)                                                                        \
  hipLaunchKernelGGL((k_row_steps<NN, WW, II>), grid, dim3(GridSteps<NN>::ROW_NT), 0, st, state, \
                     trans_p, wtrans, soff, twN, bw, groups)
#define ROW(NN)                                                                                \
  {                                                                                            \
    const int groups = nwaves * (NN / (GridSteps<NN>::ROW_NT / GridSteps<NN>::L));             \
    const dim3 grid(pass_grid(groups, GridSteps<NN>::ROW_WGS, tune.row_iters, tune.row_min_wg)); \
    if (init) ROW1(NN, false, true);                                                           \
    else if (wt) ROW1(NN, true, false);                                                        \
    else ROW1(NN, false, false);                                                               \
  }
  PRISM_DISPATCH_STEPS(n, ROW)
#undef ROW
#undef ROW1
  return hipGetLastError();
}

int col_tiles(int n) { return (n / 2) / col_tc(n); }

hipError_t launch_col_pass(float2* state, int nwaves, int n, const float2* prop_p,
                           const float2* twN, const float2* tw2, const LaunchTuning& tune,
                           hipStream_t st, bool few) {
  if (n == 1024) {
    constexpr int TC = PRISM_COL4_TC32;
    const int tiles = nwaves * (512 / TC);
    hipLaunchKernelGGL((k_col_pass4<32, TC>),
                       dim3(pass_grid(tiles, 16 / TC, tune.col_iters, tune.col_min_wg)),
                       dim3(TC * 32), 0, st, state, prop_p, tw2, tiles);
    return hipGetLastError();
  }
  if (n == 256) {
    const int tiles = nwaves * 8;
    hipLaunchKernelGGL((k_col_pass4<16, 16>),
                       dim3(pass_grid(tiles, 4, tune.col_iters, tune.col_min_wg)), dim3(256), 0, st,
                       state, prop_p, tw2, tiles);
    return hipGetLastError();
  }
  if (few) {
    const DetBins none{};
#define COLL(NN)                                                                          \
  hipLaunchKernelGGL((k_col_lds<NN, false>), dim3((unsigned)(nwaves * col_tiles(NN))),    \
                     dim3(col_nt(NN)), 0, st, state, prop_p, twN, none, (double*)nullptr)
    PRISM_DISPATCH_FEW(n, COLL)
#undef COLL
    return hipGetLastError();
  }
#define COL(NN)                                                                                 \
  {                                                                                             \
    const int tiles = nwaves * (NN / 2 / GridSteps<NN>::TC);                                    \
    hipLaunchKernelGGL((k_col_steps<NN>),                                                       \
                       dim3(pass_grid(tiles, GridSteps<NN>::COL_WGS, tune.col_iters,           \
                                       tune.col_min_wg)),                                       \
                       dim3(GridSteps<NN>::TC * GridSteps<NN>::L), 0, st, state, prop_p, twN,   \
                       tiles);                                                                  \
  }
  PRISM_DISPATCH_STEPS(n, COL)
#undef COL
  return hipGetLastError();
}

hipError_t launch_col_detect(const float2* state, int nwaves, int n, const float2* prop_p,
                             const float2* twN, const DetBins& bins, double* partial,
                             hipStream_t st) {
#define COLD(NN)                                                                                 \
  hipLaunchKernelGGL((k_col_lds<NN, true>), dim3((unsigned)(nwaves * col_tiles(NN))),            \
                     dim3(col_nt(NN)), 0, st, const_cast<float2*>(state), prop_p, twN, bins,    \
                     partial)
  PRISM_DISPATCH_N(n, COLD)
#undef COLD
  return hipGetLastError();
}

hipError_t launch_probe_init(float2* state, const double* probe_xy, int p0, int np, int n,
                             const ProbeOptics& po, const int2* aper, const float2* twN,
                             hipStream_t st) {
#define PINIT(NN)                                                                                \
  hipLaunchKernelGGL(k_probe_init<NN>, dim3((unsigned)(np * col_tiles(NN))), dim3(col_nt(NN)), 0, \
                     st, state, probe_xy, p0, po, aper, twN)
  PRISM_DISPATCH_N(n, PINIT)
#undef PINIT
  return hipGetLastError();
}

hipError_t launch_reduce_partials(const double* partial, int nwaves, int tiles, int n_det,
                                  double* out, OutAcc acc, hipStream_t st) {
  hipLaunchKernelGGL(k_reduce_partials, dim3(blocks_for((size_t)nwaves * n_det, 256)), dim3(256),
                     0, st, partial, nwaves, tiles, n_det, out, acc);
  return hipGetLastError();
}

hipError_t launch_extract(const float2* state, int nwaves, int n, float2* smatrix,
                          const float2* twH, hipStream_t st) {
#define EXT(NN)                                                                                  \
  hipLaunchKernelGGL(k_extract<NN>, dim3((unsigned)((size_t)nwaves * (NN / 2) / ext_nseq(NN))),  \
                     dim3(256), 0, st, state, smatrix, twH)
  PRISM_DISPATCH_N(n, EXT)
#undef EXT
  return hipGetLastError();
}

}  // namespace prism
