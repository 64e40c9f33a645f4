// PRISM probe step (Fig. 1d-f), second half: the window FFT, |Psi|^2 and
// the detector sums.
//
//   alpha_{m,n}(r0) = A(q) e^{-i chi(q)} e^{-2 pi i q.r0} / (W sqrt(B_A))
//   psi(r, r0)      = sum_{m,n} S_{m,n}(r) alpha_{m,n}(r0)      (Eq. PRISMfinal)
// inside the W x W window of Eq. RegionBounds (coefficients and window sum:
// probe16_kernels.hip), then |FFT_W psi|^2 / W^2 integrated per detector
// bin here, or stored whole (CBED).
#include <algorithm>

#include "fft_lds.hpp"
#include "fft_reg.hpp"
#include "kernels.hpp"

namespace prism {

namespace {

// Probe grouping of the window sum (shared with probe16_kernels.hip): probes
// per group for W >= 128, and the union tiles of 128 pixels.
constexpr int kCG128 = 64;
constexpr int kCTile = 128;
// ---------------------------------------------------------------------------
// W = 256 windows (too large for one workgroup's LDS): the 2D FFT runs as
// two four-step passes over the window buffer, 256 = 16 x 16.
//   rows : 16 lanes per row, lane j holds x = 16 a + j; DFT over a, twiddle
//          w_256^{jc}, LDS transpose, DFT over b -> row[c + 16 d], in place;
//   cols : tiles of 16 columns, lane (b, c) holds y = 16 a + b of column c;
//          the same steps along y, then I = |Psi|^2 / W^2 at full-grid
//          frequency f k_w is summed per detector bin (FP64) into one partial
//          per (probe, tile).
constexpr int kW4 = 256, kR4 = 16;

__device__ __forceinline__ void load_tw16(float2* twl, const float2* __restrict__ twW, int tid) {
  // twl[m][j] = w_256^{j m}
  twl[tid] = twW[((tid & 15) * (tid >> 4)) & (kW4 - 1)];
}

__global__ __launch_bounds__(256) void k_window_rows256(float2* __restrict__ window,
                                                        const float2* __restrict__ twW) {
  constexpr int R = kR4, LS = R + 1;
  __shared__ float2 twl[R * R];
  __shared__ float2 lds[R * R * LS];
  const int tid = threadIdx.x, j = tid % R, rr = tid / R;
  load_tw16(twl, twW, tid);
  __syncthreads();
  float2* row = window + ((size_t)blockIdx.x * R + rr) * kW4;
  float2* L = lds + rr * R * LS;
  float2 v[R];
#pragma unroll
  for (int a = 0; a < R; ++a) v[a] = row[R * a + j];
  dft_reg<R, false>(v);
#pragma unroll
  for (int c = 0; c < R; ++c) L[c * LS + j] = c ? cmul(v[c], twl[c * R + j]) : v[c];
  __syncthreads();
#pragma unroll
  for (int b = 0; b < R; ++b) v[b] = L[j * LS + b];
  dft_reg<R, false>(v);
#pragma unroll
  for (int d = 0; d < R; ++d) row[j + R * d] = v[d];
}

template <bool CBED, int NB>
__global__ __launch_bounds__(256) void k_window_cols256_detect(const float2* __restrict__ window,
                                                               const float2* __restrict__ twW,
                                                               int f, DetBins bins,
                                                               double* __restrict__ partial,
                                                               float* __restrict__ cbed,
                                                               OutAcc oa) {
  constexpr int R = kR4, LS = R + 1, TC = 16, TILES = kW4 / TC;
  constexpr int CS = R * LS + 1;  // column stride: 16 columns on distinct banks
  __shared__ float2 twl[R * R];
  __shared__ float2 lds[TC * CS];
  __shared__ double red[NB][4];
  const int tid = threadIdx.x, c = tid % TC, b = tid / TC;
  load_tw16(twl, twW, tid);
  __syncthreads();
  const size_t p = blockIdx.x / TILES;
  const int tile = blockIdx.x % TILES, col = tile * TC + c;
  const float2* src = window + p * kW4 * kW4 + col;
  float2* L = lds + c * CS;
  float2 v[R];
#pragma unroll
  for (int a = 0; a < R; ++a) v[a] = src[(size_t)(R * a + b) * kW4];
  dft_reg<R, false>(v);
#pragma unroll
  for (int k1 = 0; k1 < R; ++k1) L[k1 * LS + b] = k1 ? cmul(v[k1], twl[k1 * R + b]) : v[k1];
  __syncthreads();
#pragma unroll
  for (int bb = 0; bb < R; ++bb) v[bb] = L[b * LS + bb];
  dft_reg<R, false>(v);  // lane (k1 = b, c): ky index b + R k2
  const double inv_w2 = 1.0 / ((double)kW4 * (double)kW4);
  if constexpr (CBED) {
    float* dst = cbed + p * kW4 * kW4 + col;
#pragma unroll
    for (int k2 = 0; k2 < R; ++k2)
      put_out(dst + (size_t)(b + R * k2) * kW4,
              ((double)v[k2].x * v[k2].x + (double)v[k2].y * v[k2].y) * inv_w2, oa);
    return;
  }
  const long long kx = col < kW4 / 2 ? col : col - kW4;
  double acc[NB];
#pragma unroll
  for (int q = 0; q < NB; ++q) acc[q] = 0.0;
#pragma unroll
  for (int k2 = 0; k2 < R; ++k2) {
    const int kyi = b + R * k2;
    const long long ky = kyi < kW4 / 2 ? kyi : kyi - kW4;
    const long long kk = (long long)f * f * (kx * kx + ky * ky);
    const double I = ((double)v[k2].x * v[k2].x + (double)v[k2].y * v[k2].y) * inv_w2;
#pragma unroll
    for (int q = 0; q < NB; ++q)
      if (q < bins.n && kk >= bins.lo[q] && kk < bins.hi[q]) acc[q] += I;
  }
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    if (q < bins.n) {  // uniform
      const double sum = wave_sum(acc[q]);
      if ((tid & 63) == 0) red[q][tid >> 6] = sum;
    }
  }
  __syncthreads();
  if (tid < bins.n)
    partial[((size_t)p * TILES + tile) * bins.n + tid] =
        red[tid][0] + red[tid][1] + red[tid][2] + red[tid][3];
}

// ---------------------------------------------------------------------------
// W = 144 and 192 (more than one workgroup's LDS, not a square of a register
// DFT length): the same two passes over the window buffer with the LDS
// Stockham transforms: rows (kBigRows per workgroup) in place, then tiles of
// 16 columns with |Psi|^2 / W^2 and per-element binning (or CBED) as for
// W = 256.
constexpr int kBigRows = 8, kBigTC = 16, kBigNT = 256;

template <int W>
__global__ __launch_bounds__(kBigNT) void k_window_rows_lds(float2* __restrict__ window,
                                                            const float2* __restrict__ twW) {
  using B = RowBatch<W, kBigRows>;
  __shared__ float2 lds[lds_padded(W * kBigRows)];
  __shared__ float2 tw[W];
  const int tid = threadIdx.x;
  load_twiddles<W, kBigNT>(tw, twW, tid);
  float2* rows = window + (size_t)blockIdx.x * kBigRows * W;
  for (int e = tid; e < kBigRows * W; e += kBigNT) lds[lpad(e)] = rows[e];
  __syncthreads();
  fft_lds<B, kBigNT, false>(lds, tw, tid);
  for (int e = tid; e < kBigRows * W; e += kBigNT) rows[e] = lds[lpad(e)];
}

template <int W, bool CBED, int NB>
__global__ __launch_bounds__(kBigNT) void k_window_cols_lds(const float2* __restrict__ window,
                                                            const float2* __restrict__ twW, int f,
                                                            DetBins bins,
                                                            double* __restrict__ partial,
                                                            float* __restrict__ cbed, OutAcc oa) {
  constexpr int TILES = W / kBigTC;
  using B = Batch<W, kBigTC, kBigTC, 0, 1, kBigTC, true>;  // [y][c], column c is sequence c
  __shared__ float2 lds[lds_padded(W * kBigTC)];
  __shared__ float2 tw[W];
  __shared__ double red[CBED ? 1 : NB][kBigNT / 64];
  const int tid = threadIdx.x;
  load_twiddles<W, kBigNT>(tw, twW, tid);
  const size_t p = blockIdx.x / TILES;
  const int tile = blockIdx.x % TILES;
  const float2* src = window + p * W * W + tile * kBigTC;
  for (int e = tid; e < W * kBigTC; e += kBigNT) lds[lpad(e)] = src[(e / kBigTC) * W + e % kBigTC];
  __syncthreads();
  fft_lds<B, kBigNT, false>(lds, tw, tid);
  const double inv_w2 = 1.0 / ((double)W * (double)W);
  if constexpr (CBED) {
    float* dst = cbed + p * W * W + tile * kBigTC;
    for (int e = tid; e < W * kBigTC; e += kBigNT) {
      const float2 z = lds[lpad(e)];
      put_out(dst + (e / kBigTC) * W + e % kBigTC, ((double)z.x * z.x + (double)z.y * z.y) * inv_w2,
              oa);
    }
    return;
  }
  double acc[NB];
#pragma unroll
  for (int q = 0; q < NB; ++q) acc[q] = 0.0;
  for (int e = tid; e < W * kBigTC; e += kBigNT) {
    const int kyi = e / kBigTC, col = tile * kBigTC + e % kBigTC;
    const long long kx = col < W / 2 ? col : col - W, ky = kyi < W / 2 ? kyi : kyi - W;
    const long long kk = (long long)f * f * (kx * kx + ky * ky);
    const float2 z = lds[lpad(e)];
    const double I = ((double)z.x * z.x + (double)z.y * z.y) * inv_w2;
#pragma unroll
    for (int q = 0; q < NB; ++q)
      if (q < bins.n && kk >= bins.lo[q] && kk < bins.hi[q]) acc[q] += I;
  }
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    if (q < bins.n) {  // uniform
      const double sum = wave_sum(acc[q]);
      if ((tid & 63) == 0) red[q][tid >> 6] = sum;
    }
  }
  __syncthreads();
  if (tid < bins.n) {
    double sm = 0.0;
    for (int w = 0; w < kBigNT / 64; ++w) sm += red[tid][w];
    partial[((size_t)p * TILES + tile) * bins.n + tid] = sm;
  }
}

// ---------------------------------------------------------------------------
constexpr int kWdChunks = 16;  // bin-list chunks whose pixel indices load together

// Threads per window workgroup: W^2 / 16 rounded up to whole waves.
__host__ __device__ constexpr int wd_nt(int w) {
  return w * w / 16 < 64 ? 64 : (w * w / 16 + 63) / 64 * 64;
}
// Waves per SIMD the registers are limited for: at W = 128 two workgroups of
// 16 waves (64 registers).
__host__ __device__ constexpr int wd_wpe(int w) { return w == 128 ? 8 : 6; }

// The window transforms keep the window in registers and pass it from stage to
// stage through LDS, as whole complex values or one component at a time (real
// parts, then imaginary parts). By components a window needs half of the LDS, at
// four barriers per exchange instead of two and two walks of the bin lists. That
// pays where LDS or its traffic limits the waves in flight: at W = 128, where
// whole values let one workgroup per compute unit run instead of two (8192
// windows, 16 bins: 583 -> 485 us), and, with registers for two workgroups of
// nine waves either way, still at W = 96 (12800 windows, 3 bins: 589 us against
// 608 whole; patterns 412 against 482). Below, whole values are faster: W = 8, 16
// bins 26.6 us against 46.9; W = 32, 16 bins 56.6 against 92.5; W = 36, 3 bins
// 55 against 82; W = 64, 3 bins 116 against 137; W = 72, 3 bins 269 against 330,
// though patterns of W = 72 take 220 against 208 (12800 windows each).
__host__ __device__ constexpr bool wd_whole(int w, bool cbed) { return w <= (cbed ? 64 : 72); }
enum class Part { kRe, kIm, kWhole };
template <Part PT>
struct LdsPart {
  using T = float;
  static constexpr int SH = 5;  // padding: one element in 2^SH
  __device__ __forceinline__ static T of(float2 z) { return PT == Part::kRe ? z.x : z.y; }
  __device__ __forceinline__ static void to(float2& z, T x) {
    if (PT == Part::kRe) z.x = x;
    else z.y = x;
  }
};
template <>
struct LdsPart<Part::kWhole> {
  using T = float2;
  static constexpr int SH = 4;
  __device__ __forceinline__ static T of(float2 z) { return z; }
  __device__ __forceinline__ static void to(float2& z, T x) { z = x; }
};
template <int SH>
__host__ __device__ constexpr int padded(int i) {
  return i + (i >> SH);
}
// Padded address of base + r STEP for the elements of one butterfly (r < R of
// a sequence of length L): a compile-time offset from the padded base where
// the elements' blocks of P = 2^SH do not depend on the base, i.e. STEP is a
// multiple of P, or base = m (R STEP) + k with k < STEP (Stockham stages of
// rows) and R STEP divides P or is a multiple of it.
template <int SH, int STEP, int R, int L>
__device__ __forceinline__ int padded_step(int base_padded, int base, int r) {
  constexpr int P = 1 << SH;
  constexpr bool P2 = (STEP & (STEP - 1)) == 0 && (R & (R - 1)) == 0;
  if constexpr (STEP % P == 0 || (P2 && P % (STEP * R) == 0) ||
                (P2 && STEP * R % P == 0 && L % P == 0))
    return base_padded + r * STEP + ((r * STEP) >> SH);
  else
    return padded<SH>(base + r * STEP);
}

// Radix of the stage with span NS of a length-L transform (as fft_from).
__host__ __device__ constexpr int next_radix(int rem) {
  return rem % 8 == 0 ? 8 : (rem % 4 == 0 ? 4 : (rem % 2 == 0 ? 2 : 3));
}

// Flat index of element r of butterfly b's outputs / inputs in a stage.
template <class B, int R, int NS>
__host__ __device__ constexpr int out_index(int b, int r) {
  constexpr int NB = B::L / R;
  const int s = B::SEQ_FAST ? b % B::NSEQ : b / NB, j = B::SEQ_FAST ? b / B::NSEQ : b % NB;
  const int k = j % NS, e = (j - k) * R + k + r * NS;
  return (s / B::SPB) * B::BSTR + (s % B::SPB) * B::SSTR + e * B::ESTR;
}
template <class B, int R>
__host__ __device__ constexpr int in_index(int b, int r) {
  constexpr int NB = B::L / R;
  const int s = B::SEQ_FAST ? b % B::NSEQ : b / NB, j = B::SEQ_FAST ? b / B::NSEQ : b % NB;
  return (s / B::SPB) * B::BSTR + (s % B::SPB) * B::SSTR + (j + r * NB) * B::ESTR;
}
// Powers of two throughout: thread, butterfly and element numbers are
// disjoint bit fields of the index, so padded addresses add up and all but
// the thread's own part is a compile-time offset.
template <class B, int NT>
__host__ __device__ constexpr bool bit_fields() {
  return (B::L & (B::L - 1)) == 0 && (B::NSEQ & (B::NSEQ - 1)) == 0 && (NT & (NT - 1)) == 0 &&
         B::L * B::NSEQ >= 8 * NT;
}

// The window transforms' arithmetic with every multiply-add written out, so
// that their results do not depend on what the compiler contracts in the code
// around it: a b, and the 8- and 3-point DFTs of fft_lds.hpp (2 and 4 points
// have no products). xb says which of the imaginary part's two products is
// rounded on its own. Neither form is the more exact one (FP32, W = 128, against
// 64 bits: 2.4e-7 with the choice below, 2.2e-7 with one form throughout). The
// choice per butterfly (WinFft) follows what the compiler once contracted, so
// that the FP64 detector sums repeat earlier versions' to 1e-15 (W <= 72: the
// same additions; above, squares of real and imaginary parts are added apart);
// one form throughout moves them by 2e-8.
__device__ __forceinline__ float2 cmul_fma(float2 a, float2 b, bool xb) {
  const float fx = xb ? a.x : a.y, fy = xb ? b.y : b.x;  // the fused pair
  const float rx = xb ? a.y : a.x, ry = xb ? b.x : b.y;  // the rounded one
  return make_float2(__builtin_fmaf(a.x, b.x, -(a.y * b.y)), __builtin_fmaf(fx, fy, rx * ry));
}
// z + s (x, y)
__device__ __forceinline__ float2 madd(float2 z, float s, float x, float y) {
  return make_float2(__builtin_fmaf(s, x, z.x), __builtin_fmaf(s, y, z.y));
}
template <int R>
__device__ __forceinline__ void dft_fma(float2 (&v)[R]) {
  if constexpr (R == 8) {
    float2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
    float2 o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
    dft4v<false>(e0, e1, e2, e3);
    dft4v<false>(o0, o1, o2, o3);
    constexpr float r = 0.70710678118654752440f;
    const float2 p = make_float2(o1.x + o1.y, o1.y - o1.x);      // o1 w / r
    const float2 q = make_float2(o3.y - o3.x, -(o3.x + o3.y));   // o3 w^3 / r
    o2 = mul_mi<false>(o2);
    v[0] = cadd(e0, o0);
    v[4] = csub(e0, o0);
    v[1] = madd(e1, r, p.x, p.y);
    v[5] = madd(e1, -r, p.x, p.y);
    v[2] = cadd(e2, o2);
    v[6] = csub(e2, o2);
    v[3] = madd(e3, r, q.x, q.y);
    v[7] = madd(e3, -r, q.x, q.y);
  } else if constexpr (R == 3) {
    constexpr float h = 0.86602540378443864676f;  // sqrt(3) / 2
    const float2 t1 = cadd(v[1], v[2]), t2 = csub(v[1], v[2]);
    const float2 m = madd(v[0], -0.5f, t1.x, t1.y);
    v[0] = cadd(v[0], t1);
    v[1] = madd(m, h, t2.y, -t2.x);
    v[2] = madd(m, -h, t2.y, -t2.x);
  } else {
    dft<R, false>(v);
  }
}

// Inputs of one butterfly times w^r, w = exp(-2 pi i k / (NS R)): w, w^2, w^4
// from the table, the other powers as products (as stage_in).
template <class B, int R, int NS>
__device__ __forceinline__ void stage_twiddle(const float2* tw, int k, bool xb, float2 (&v)[R]) {
  constexpr int TWS = B::L / (NS * R);
  float2 w[R];
  if constexpr (R == 2 || R == 4 || R == 8) {
    w[1] = tw[k * TWS];
    if constexpr (R >= 4) w[2] = tw[2 * k * TWS];
    if constexpr (R == 4) w[3] = cmul_fma(w[1], w[2], false);
    if constexpr (R == 8) {
      w[4] = tw[4 * k * TWS];
      w[3] = cmul_fma(w[1], w[2], false);
      w[5] = cmul_fma(w[1], w[4], false);
      w[6] = cmul_fma(w[2], w[4], false);
      w[7] = cmul_fma(w[3], w[4], false);
    }
  } else {
#pragma unroll
    for (int r = 1; r < R; ++r) w[r] = tw[r * k * TWS];
  }
#pragma unroll
  for (int r = 1; r < R; ++r)
    v[r] = cmul_fma(v[r], w[r], xb && !(B::L == 128 && r == 4));
}

// Part PT of a stage's outputs to LDS / of its inputs from LDS (element
// numbering of stage_out / stage_in).
template <class B, int R, int NS, int NT, Part PT>
__device__ __forceinline__ void put_part(typename LdsPart<PT>::T* lds, int tid,
                                         const float2 (&v)[StageShape<B, R, NT>::PER][R]) {
  using SS = StageShape<B, R, NT>;
  using LP = LdsPart<PT>;
  if constexpr (bit_fields<B, NT>()) {
    typename LP::T* own = lds + padded<LP::SH>(out_index<B, R, NS>(tid, 0));
#pragma unroll
    for (int p = 0; p < SS::PER; ++p)
#pragma unroll
      for (int r = 0; r < R; ++r)
        own[padded<LP::SH>(out_index<B, R, NS>(p * NT, r))] = LP::of(v[p][r]);
  } else {
#pragma unroll
    for (int p = 0; p < SS::PER; ++p) {
      const int b = tid + p * NT;
      if (SS::GUARD && b >= SS::TOT) continue;
      const int base = out_index<B, R, NS>(b, 0), pbase = padded<LP::SH>(base);
#pragma unroll
      for (int r = 0; r < R; ++r)
        lds[padded_step<LP::SH, NS * B::ESTR, R, B::L>(pbase, base, r)] = LP::of(v[p][r]);
    }
  }
}
template <class B, int R, int NT, Part PT>
__device__ __forceinline__ void get_part(const typename LdsPart<PT>::T* lds, int tid,
                                         float2 (&v)[StageShape<B, R, NT>::PER][R]) {
  using SS = StageShape<B, R, NT>;
  using LP = LdsPart<PT>;
  if constexpr (bit_fields<B, NT>()) {
    const typename LP::T* own = lds + padded<LP::SH>(in_index<B, R>(tid, 0));
#pragma unroll
    for (int p = 0; p < SS::PER; ++p)
#pragma unroll
      for (int r = 0; r < R; ++r)
        LP::to(v[p][r], own[padded<LP::SH>(in_index<B, R>(p * NT, r))]);
  } else {
#pragma unroll
    for (int p = 0; p < SS::PER; ++p) {
      const int b = tid + p * NT;
      if (SS::GUARD && b >= SS::TOT) continue;
      const int base = in_index<B, R>(b, 0), pbase = padded<LP::SH>(base);
#pragma unroll
      for (int r = 0; r < R; ++r)
        LP::to(v[p][r], lds[padded_step<LP::SH, SS::NB * B::ESTR, R, B::L>(pbase, base, r)]);
    }
  }
}

template <int W, bool WHOLE>
struct WinFft {
  static constexpr int NT = wd_nt(W);
  using Lds = LdsPart<WHOLE ? Part::kWhole : Part::kRe>;
  using T = typename Lds::T;
  static constexpr int SIZE = padded<Lds::SH>(W * W);
  using Rows = RowBatch<W, W>;
  using Cols = Batch<W, W, W, 0, 1, W, true>;

  // xb of a stage's butterflies past the first NT: set where the stage's
  // twiddles repeat every NT butterflies.
  template <class B, int R, int NS>
  __device__ __forceinline__ static constexpr bool round_xb() {
    constexpr int NB = B::L / R;
    return B::SEQ_FAST ? (W & (W - 1)) == 0 && (NT / W) % NS == 0
                       : (NB & (NB - 1)) == 0 && NT % NB == 0;
  }

  // From the inputs v of the stage (B, NS) (twiddles applied) through the
  // rest of the 2D transform; fin(v) gets the outputs of the last column
  // stage (radix next_radix(W / span), see last_span).
  template <class B, int NS, bool ROWS, class F>
  __device__ __forceinline__ static void run(
      T* lds, const float2* tw, int tid,
      float2 (&v)[StageShape<B, next_radix(W / NS), NT>::PER][next_radix(W / NS)], const F& fin) {
    constexpr int R = next_radix(W / NS);
    using SS = StageShape<B, R, NT>;
#pragma unroll
    for (int p = 0; p < SS::PER; ++p)
      if (!SS::GUARD || tid + p * NT < SS::TOT) dft_fma<R>(v[p]);
    if constexpr (NS * R < W) {
      pass<B, R, NS, B, NS * R, ROWS>(lds, tw, tid, v, fin);
    } else if constexpr (ROWS) {
      pass<B, R, NS, Cols, 1, false>(lds, tw, tid, v, fin);
    } else {
      fin(v);
    }
  }

  template <class BO, int RO, int NSO, class BI, int NSI, bool ROWS, class F>
  __device__ __forceinline__ static void pass(T* lds, const float2* tw, int tid,
                                              float2 (&v)[StageShape<BO, RO, NT>::PER][RO],
                                              const F& fin) {
    constexpr int RI = next_radix(W / NSI);
    using SI = StageShape<BI, RI, NT>;
    float2 u[SI::PER][RI];
    if constexpr (WHOLE) {
      put_part<BO, RO, NSO, NT, Part::kWhole>(lds, tid, v);
      __syncthreads();
      get_part<BI, RI, NT, Part::kWhole>(lds, tid, u);
    } else {
      put_part<BO, RO, NSO, NT, Part::kRe>(lds, tid, v);
      __syncthreads();
      get_part<BI, RI, NT, Part::kRe>(lds, tid, u);
      __syncthreads();
      put_part<BO, RO, NSO, NT, Part::kIm>(lds, tid, v);
      __syncthreads();
      get_part<BI, RI, NT, Part::kIm>(lds, tid, u);
    }
    if constexpr (NSI > 1) {
#pragma unroll
      for (int p = 0; p < SI::PER; ++p) {
        const int b = tid + p * NT;
        if (SI::GUARD && b >= SI::TOT) continue;
        int s, j;
        stage_coords<BI, SI::NB>(b, s, j);
        stage_twiddle<BI, RI, NSI>(tw, j % NSI, p > 0 && round_xb<BI, RI, NSI>(), u[p]);
        // one butterfly's twiddles at a time: no registers for all of them
        if constexpr (SI::PER * RI >= 24) __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();  // LDS free for the next exchange
    run<BI, NSI, ROWS>(lds, tw, tid, u, fin);
  }
};

// Span of the last stage of a length-w transform (product of the radices
// before it).
__host__ __device__ constexpr int last_span(int w, int ns = 1) {
  return ns * next_radix(w / ns) == w ? ns : last_span(w, ns * next_radix(w / ns));
}

// 2D FFT of each W x W window, then either I(kw) = |Psi(kw)|^2 / W^2 summed
// over each bin's pixel list in FP64 (the lists encode the angle test at
// full-grid frequency f kw), or (CBED) I written out in full. One workgroup
// per window; window p belongs to the segment whose range holds it (its own
// outputs and, for the sums, its own pixel lists).
//
// Bin sums: |Psi|^2 (where the window passes through LDS by components: the
// squares of the real parts, then of the imaginary parts) is summed over the
// lists. The lists are cut into chunks of kWdListChunk = 64 entries (one per
// lane, kNoPix padding at the end of each bin); chunk k belongs to the bin j
// with off[j] <= k < off[j + 1]. Wave w takes the contiguous chunks [K w / NW,
// K (w + 1) / NW) of the K in all, so it meets only a few bins: each lane sums
// its entry of the wave's chunks of a bin in order, one wave sum per bin met
// and walk is added to red[j][w] (zero for the bins a wave does not meet), and
// the bin total adds red[j][0 .. NW) in order. The pixel indices of kWdChunks
// chunks are loaded together, so the load latency is paid once per group of
// chunks. Bound: the exchanges and these sums, whose VALU work alone is 8 us
// per window of W = 128 and compute unit where the loads take 6.
template <int W, bool CBED>
__global__ __launch_bounds__(wd_nt(W)) __attribute__((amdgpu_waves_per_eu(wd_wpe(W))))
void k_window_detect(const float2* __restrict__ window,
                                                            const float2* __restrict__ twW,
                                                            const WindowSegs segs) {
  constexpr bool WHOLE = wd_whole(W, CBED);
  using WF = WinFft<W, WHOLE>;
  using Rows = typename WF::Rows;
  using Cols = typename WF::Cols;
  constexpr int NT = WF::NT;
  constexpr int NW = NT / 64;
  constexpr int R0 = next_radix(W), NSL = last_span(W), RL = W / NSL;
  using S0 = StageShape<Rows, R0, NT>;
  using SL = StageShape<Cols, RL, NT>;
  __shared__ typename WF::T lds[WF::SIZE];
  __shared__ float2 tw[W];
  __shared__ double red[CBED ? 1 : kMaxDet][NW];
  const int tid = threadIdx.x;
  load_twiddles<W, NT>(tw, twW, tid);
  const double inv_w2 = 1.0 / ((double)W * (double)W);
  const int p = blockIdx.x;
  int k = 0;  // segment of window p (uniform)
  while (k + 1 < segs.n && p >= segs.s[k + 1].begin) ++k;
  const WindowSeg& sg = segs.s[k];
  const int q = p - sg.begin;  // probe within the segment
  float2 v[S0::PER][R0];
  {
    const float2* src = window + (size_t)p * W * W;
#pragma unroll
    for (int c = 0; c < S0::PER; ++c) {
      const int b = tid + c * NT;
      if (!S0::GUARD || b < S0::TOT) {
        int row, j;
        stage_coords<Rows, S0::NB>(b, row, j);
#pragma unroll
        for (int r = 0; r < R0; ++r) v[c][r] = src[row * W + j + r * (W / R0)];
      }
    }
  }
  WF::template run<Rows, 1, true>(lds, tw, tid, v, [&](float2(&z)[SL::PER][RL]) {
    if constexpr (CBED) {
      float* dst = sg.cbed + (size_t)q * W * W;
#pragma unroll
      for (int c = 0; c < SL::PER; ++c) {
        const int b = tid + c * NT;
        if (SL::GUARD && b >= SL::TOT) continue;
        int s, j;
        stage_coords<Cols, SL::NB>(b, s, j);
#pragma unroll
        for (int r = 0; r < RL; ++r)
          put_out(dst + (j + r * NSL) * W + s,
                  ((double)z[c][r].x * z[c][r].x + (double)z[c][r].y * z[c][r].y) * inv_w2,
                  sg.oa);
      }
    } else {
      const uint16_t* __restrict__ pix = sg.pix;
      const BinLists* __restrict__ lists = sg.lists;  // uniform: scalar loads
      const int nb = lists->n;
      const int* off = lists->off;
      const int K = off[nb];  // chunks of kWdListChunk entries
      const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
      const int c0 = (int)((long long)K * wv / NW), c1 = (int)((long long)K * (wv + 1) / NW);
      for (int i = tid; i < nb * NW; i += NT) red[i / NW][i % NW] = 0.0;
      auto sum_part = [&]() {
        int j = 0;  // bin of the current chunk (uniform in the wave)
        while (j < nb && c0 >= off[j + 1]) ++j;
        double acc = 0.0;
        for (int k0 = c0; k0 < c1; k0 += kWdChunks) {
          int px[kWdChunks];
#pragma unroll
          for (int c = 0; c < kWdChunks; ++c)
            px[c] = k0 + c < c1 ? (int)pix[(size_t)(k0 + c) * kWdListChunk + lane] : (int)kNoPix;
#pragma unroll
          for (int c = 0; c < kWdChunks; ++c) {
            const int kk = k0 + c;
            if (kk < c1) {
              if (kk >= off[j + 1]) {  // bin j ends: its wave sum, then the bin of chunk kk
                const double sm = wave_sum(acc);
                if (lane == 0) red[j][wv] += sm;
                acc = 0.0;
                do ++j;
                while (kk >= off[j + 1]);
              }
              const bool ok = px[c] != (int)kNoPix;
              const auto z = lds[padded<WF::Lds::SH>(ok ? px[c] : 0)];
              double I;
              if constexpr (WHOLE) I = (double)z.x * z.x + (double)z.y * z.y;
              else I = (double)z * z;
              acc += ok ? I : 0.0;
            }
          }
        }
        if (c1 > c0) {
          const double sm = wave_sum(acc);
          if (lane == 0) red[j][wv] += sm;
        }
      };
      if constexpr (WHOLE) {
        put_part<Cols, RL, NSL, NT, Part::kWhole>(lds, tid, z);
        __syncthreads();
        sum_part();
      } else {
        put_part<Cols, RL, NSL, NT, Part::kRe>(lds, tid, z);
        __syncthreads();
        sum_part();
        __syncthreads();
        put_part<Cols, RL, NSL, NT, Part::kIm>(lds, tid, z);
        __syncthreads();
        sum_part();
      }
      __syncthreads();
      if (tid < nb) {
        double sm = 0.0;
        for (int w = 0; w < NW; ++w) sm += red[tid][w];
        put_out(sg.out + (size_t)q * nb + tid, sm * inv_w2, sg.oa);
      }
    }
  });
}

inline unsigned blocks_for(size_t n, unsigned bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

// A group shares one union window, so a larger one reads fewer S-matrix pixels
// per probe and pays for the union's pixels that a member does not have. FP32
// is bound by its products, which a union wastes: 64 only where windows are
// large against the scan step. 16-bit operands are bound by what they read:
// 64 as soon as a window is three tiles wide. Measured (window sum, groups of
// 16 / 32 / 64, 12800 raster probes): FP32 W = 64 722 / 660 / 770 us, W = 96
// 2767 / 2628 / 2943 us, W = 144 13.8 / 13.1 / 11.8 ms; BF16 W = 48 94 / 85 /
// 78 us, W = 64 205 / 176 / 156 us, W = 128 2569 / 1666 / 1236 us. Below W = 48
// that many probes would do a little better in larger groups (FP32 W = 32 83 / 79
// / 98, BF16 W = 32 39 / 35 / 33, W = 16 24 / 21 / 22 us), fewer or scattered
// ones worse (1200 scattered probes, FP32 W = 16 17 / 26 / 47, BF16 W = 32 24 /
// 28 / 39 us on 768^2; 30 probes, FP32 W = 32 9 / 12 / 13 us): 16 for them all.
int contract_group(int w, Prec pr) {
  if (pr != Prec::kF32) return w >= 48 ? 64 : 16;
  return w >= 128 ? kCG128 : (w >= 64 ? 32 : 16);
}

// A launch has at least kCFill workgroups, so that groups of unequal unions even
// out: with own / 4 slots one group of 15 probes of W = 128 ran on 32 workgroups
// (164 us, on 256 39) and the 38 groups of 1200 scattered probes of W = 64 on 304
// (193 us, on 2280 110). FP32 groups of 16 and 32 probes leave registers and LDS
// for three workgroups per compute unit, and their launches have three whole
// rounds of those 768. Rounds that end part full, and slots in powers of two,
// which put the tiles beyond a whole number per slot on the same compute units
// in every group, cost aligned scans up to a quarter (W = 64: 2048 probes 166 us
// with 2048 workgroups, 127 with 2304; 1024 probes 98 and 69; a ragged scan of
// 5673 probes 403 and 392; over 108 scans 0.5 % on average, the worst 8 % longer).
// 16-bit sums and groups of 64 are on average as fast or faster with 2048, a
// multiple of which keeps one tile of neighbouring groups on one XCD. More than
// the tiles of two windows per group are never needed by windows that overlap.
constexpr int kCFill = 2048, kCFill32 = 3 * 768;

int contract_tile_slots(int w, int window_tile_div, int groups, int group, Prec pr) {
  const int own = (w * w + kCTile - 1) / kCTile;  // tiles of one window
  const int want = std::max(1, own / std::max(1, window_tile_div));
  const int fill = pr == Prec::kF32 && group < 64 ? kCFill32 / groups
                                                  : (kCFill + groups - 1) / groups;
  return std::max(want, std::min(2 * own, fill));
}

int window_big_tiles(int w) { return w / 16; }

// Accumulator slots of the per-element binning kernels for n bins: the
// smallest of 4, 8, 16 and kMaxDet that holds them (the kernels test each
// element against every slot below n, so fewer slots mean less work per
// element; the sums are the same).
static int bin_slots(int n) { return n <= 4 ? 4 : (n <= 8 ? 8 : (n <= 16 ? 16 : kMaxDet)); }

hipError_t launch_window_big(float2* window, int np, int w, const float2* twW, int f,
                             const DetBins& bins, double* partial, float* cbed, OutAcc acc,
                             hipStream_t st) {
  const bool want_cbed = cbed != nullptr;
  if (w == kW4) {
    hipLaunchKernelGGL(k_window_rows256, dim3((unsigned)((size_t)np * kW4 / kR4)), dim3(256), 0,
                       st, window, twW);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)((size_t)np * window_big_tiles(w)));
    if (want_cbed) {
      hipLaunchKernelGGL((k_window_cols256_detect<true, 1>), grid, dim3(256), 0, st, window, twW,
                         f, bins, (double*)nullptr, cbed, acc);
      return hipGetLastError();
    }
#define C256(NBB)                                                                          \
  hipLaunchKernelGGL((k_window_cols256_detect<false, NBB>), grid, dim3(256), 0, st, window, \
                     twW, f, bins, partial, (float*)nullptr, OutAcc{})
    switch (bin_slots(bins.n)) {
      case 4: C256(4); break;
      case 8: C256(8); break;
      case 16: C256(16); break;
      default: C256(kMaxDet); break;
    }
#undef C256
    return hipGetLastError();
  }
#define WCOLS(WW, NBB)                                                                     \
  hipLaunchKernelGGL((k_window_cols_lds<WW, false, NBB>), grid, dim3(kBigNT), 0, st, window, \
                     twW, f, bins, partial, (float*)nullptr, OutAcc{})
#define WBIG(WW)                                                                           \
  case WW: {                                                                               \
    hipLaunchKernelGGL(k_window_rows_lds<WW>, dim3((unsigned)((size_t)np * WW / kBigRows)), \
                       dim3(kBigNT), 0, st, window, twW);                                  \
    hipError_t e = hipGetLastError();                                                      \
    if (e != hipSuccess) return e;                                                         \
    const dim3 grid((unsigned)((size_t)np * (WW / kBigTC)));                               \
    if (want_cbed) {                                                                       \
      hipLaunchKernelGGL((k_window_cols_lds<WW, true, 1>), grid, dim3(kBigNT), 0, st,      \
                         window, twW, f, bins, (double*)nullptr, cbed, acc);               \
      break;                                                                               \
    }                                                                                      \
    switch (bin_slots(bins.n)) {                                                           \
      case 4: WCOLS(WW, 4); break;                                                         \
      case 8: WCOLS(WW, 8); break;                                                         \
      case 16: WCOLS(WW, 16); break;                                                       \
      default: WCOLS(WW, kMaxDet); break;                                                  \
    }                                                                                      \
    break;                                                                                 \
  }
  switch (w) {
    WBIG(144)
    WBIG(192)
    default:
      return hipErrorInvalidValue;
  }
#undef WBIG
#undef WCOLS
  return hipGetLastError();
}

hipError_t launch_window_detect(const float2* window, const WindowSegs& segs, int w,
                                const float2* twW, hipStream_t st) {
  if (segs.total <= 0) return hipSuccess;
  if (segs.n < 1 || segs.n > kMaxSeg) return hipErrorInvalidValue;
#define WD(WW)                                                                          \
  case WW:                                                                              \
    hipLaunchKernelGGL((k_window_detect<WW, false>), dim3((unsigned)segs.total),     \
                       dim3(wd_nt(WW)), 0, st, window, twW, segs);                      \
    break;
  switch (w) {
    WD(8)
    WD(16)
    WD(32)
    WD(64)
    WD(128)
    WD(24)
    WD(48)
    WD(72)
    WD(96)
    WD(12)
    WD(18)
    WD(36)
    default:
      return hipErrorInvalidValue;
  }
#undef WD
  return hipGetLastError();
}

hipError_t launch_window_cbed(const float2* window, const WindowSegs& segs, int w,
                              const float2* twW, hipStream_t st) {
  if (segs.total <= 0) return hipSuccess;
  if (segs.n < 1 || segs.n > kMaxSeg) return hipErrorInvalidValue;
#define WC(WW)                                                                          \
  case WW:                                                                              \
    hipLaunchKernelGGL((k_window_detect<WW, true>), dim3((unsigned)segs.total),      \
                       dim3(wd_nt(WW)), 0, st, window, twW, segs);                      \
    break;
  switch (w) {
    WC(8)
    WC(16)
    WC(32)
    WC(64)
    WC(128)
    WC(24)
    WC(48)
    WC(72)
    WC(96)
    WC(12)
    WC(18)
    WC(36)
    default:
      return hipErrorInvalidValue;
  }
#undef WC
  return hipGetLastError();
}

}  // namespace prism
