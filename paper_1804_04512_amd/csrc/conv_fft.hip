// Full convolution through the Fourier transform (Section II-A names this route for the backward
// pass: image and filter padded to the output size, transformed, multiplied point by point,
// transformed back; an image's transform is computed once and serves every filter).
//
//   dx[n,c] = crop_pad( sum_k  dz[n,k] (*) w[k,c] ),   (*) = true (filter-flipping) full convolution
//
// which is exactly the backward-data sum  dx[n,c,i,j] = sum_{k,r,s} dz[n,k,i+pad-r,j+pad-s] w[k,c,r,s].
// Here the padded size is the next power of two (at most 64 x 64, so a whole complex image fits in
// LDS): no wrap-around reaches the part that is kept.
//
//   fft2_forward_kernel    one workgroup per real image (a dz map, formed on the fly from the pooled
//                          gradient, the pooling bytes and the layer output exactly as the other
//                          backward kernels do, or a filter slice): rows, then columns, decimation
//                          in frequency, natural order in, bit-reversed order out;
//   fft2_product_kernel    per frequency the sum over k of the products of the two spectra, tiles of
//                          image pairs x channels in registers, frequencies across the lanes;
//   fft2_inverse_kernel    columns and rows back by decimation in time (bit-reversed in, natural
//                          out, so no reordering pass exists anywhere), scaled, cropped;
//   fft2_product_inverse_kernel   both in one, for callers whose workspace holds no product spectra.
// The filters are real, so convolving is linear over the complex numbers with real coefficients:
// two images n, n+1 of the batch ride through all three stages as ONE complex signal
// dz[n] + i dz[n+1], and the real and imaginary parts of the result are dx[n] and dx[n+1].  That
// halves the image transforms, the products and the inverse transforms.
// All arithmetic is fp32; the result differs from the direct sum by rounding only (a few 1e-7 of
// the largest output).
#include "dll_internal.h"

namespace dllk {
namespace {

constexpr int kFftThreads = 256;
constexpr int kMaxLog = 6;                 // padded sides up to 64
constexpr int kTw = 1 << kMaxLog;          // twiddles exp(-2 pi i t / 64), t < 64

__device__ __forceinline__ float2 cmul(float2 a, float2 b) { return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }

__device__ __forceinline__ void make_twiddles(float2 *tw) {
  if (threadIdx.x < kTw) {
    float s, c;
    sincospif(-(float)threadIdx.x / (float)(kTw / 2), &s, &c);
    tw[threadIdx.x] = make_float2(c, s);
  }
}

// A transform of 2^l points runs in at most two passes, radix 2^a then 2^b with a = min(l, 3), a + b = l:
// a pass takes its 2, 4 or 8 points into registers, so a 64 x 64 image crosses LDS four times instead of
// the twelve of radix-2 passes, with three barriers instead of twelve.
__device__ __forceinline__ int first_log(int l) { return l < 3 ? l : 3; }

// v times exp(-+ 2 pi i m / 8)
template <bool INVERSE>
__device__ __forceinline__ float2 times_w8(float2 v, int m) {
  constexpr float h = 0.70710678118654752f;
  const float s = INVERSE ? -1.0f : 1.0f;
  switch (m) {
  case 1: return make_float2(h * (v.x + s * v.y), h * (v.y - s * v.x));
  case 2: return make_float2(s * v.y, -s * v.x);
  case 3: return make_float2(h * (s * v.y - v.x), -h * (s * v.x + v.y));
  default: return v;
  }
}
// The 2^RL-point transform in registers.  Forward: natural order in, v[p] = X[bit-reversed p] out.
// Inverse: the same stages backwards.
template <bool INVERSE, int RL>
__device__ __forceinline__ void small_dft(float2 (&v)[1 << RL]) {
  constexpr int R = 1 << RL;
#pragma unroll
  for (int t = 0; t < RL; ++t) {
    const int half = INVERSE ? 1 << t : R >> (t + 1);
#pragma unroll
    for (int p = 0; p < R / 2; ++p) {
      const int m = p & (half - 1), i0 = 2 * (p - m) + m, i1 = i0 + half;
      const float2 a = v[i0];
      if (INVERSE) {
        const float2 b = times_w8<true>(v[i1], m * (4 / half));
        v[i0] = cadd(a, b);
        v[i1] = csub(a, b);
      } else {
        const float2 b = v[i1];
        v[i0] = cadd(a, b);
        v[i1] = times_w8<false>(csub(a, b), m * (4 / half));
      }
    }
  }
}
template <int RL>
__device__ __forceinline__ constexpr int reversed(int p) {
  int r = 0;
  for (int b = 0; b < RL; ++b) r |= ((p >> b) & 1) << (RL - 1 - b);
  return r;
}
// twiddles between the passes of a line of 2^len_log points: v[p] *= exp(-+ 2 pi i j reversed(p) / 2^len_log)
template <bool INVERSE, int RL>
__device__ __forceinline__ void twiddle(float2 (&v)[1 << RL], const float2 *tw, int j, int len_log) {
#pragma unroll
  for (int p = 1; p < 1 << RL; ++p) {
    float2 w = tw[(j * reversed<RL>(p)) << (kMaxLog - len_log)];
    if (INVERSE) w.y = -w.y;
    v[p] = cmul(v[p], w);
  }
}

// The image in LDS: row i, column c at (i << lpw) + (c ^ row_swizzle(i)).  A wavefront works 64 columns
// of one row, 8 columns of 8 neighbouring rows, or one column of 32 or 64 rows at a time: all three fall into
// different banks.
__device__ __forceinline__ int row_swizzle(int i, int lpw) { return (((i & 3) << 3) | ((i >> 2) & 7)) & ((1 << lpw) - 1); }
__device__ __forceinline__ int at(int i, int c, int lpw) { return (i << lpw) + (c ^ row_swizzle(i, lpw)); }

// One pass along the rows (ROWS) or down the columns.  FIRST: the pass of radix 2^a over points 2^b apart, with
// the twiddles; else the pass of radix 2^b over neighbouring points.  `load` and `store` move one element by
// (row, column); only rows in [r0, r1) are worked (row passes).
template <bool INVERSE, bool ROWS, bool FIRST, int RL, class Load, class Store>
__device__ __forceinline__ void fft_pass_r(const float2 *tw, int lph, int lpw, int r0, int r1, Load load, Store store) {
  const int len = ROWS ? lpw : lph;
  const int rest = len - RL;                    // log2 of the line's positions per point of the radix
  const int ulog = FIRST ? rest : 0;            // log2 of the distance between a butterfly's points
  int lines, line_log = 0;
  if (ROWS) { lines = r1 - r0; while ((1 << line_log) < lines) ++line_log; } else { lines = 1 << lpw; line_log = lpw; }
  const int items = 1 << (line_log + rest);
  // lanes take neighbouring columns (column passes), neighbouring points (first row pass: what comes from or goes
  // to memory) or neighbouring rows (second row pass)
  for (int it = threadIdx.x; it < items; it += kFftThreads) {
    int line, q;
    if (ROWS && FIRST) { q = it & ((1 << rest) - 1); line = it >> rest; } else { line = it & ((1 << line_log) - 1); q = it >> line_log; }
    if (line >= lines) continue;
    if (ROWS) line += r0;
    const int base = FIRST ? q : q << RL;
    float2 v[1 << RL];
#pragma unroll
    for (int m = 0; m < 1 << RL; ++m) { const int x = base + (m << ulog); v[m] = ROWS ? load(line, x) : load(x, line); }
    if (INVERSE && FIRST) twiddle<true, RL>(v, tw, q, len);
    small_dft<INVERSE, RL>(v);
    if (!INVERSE && FIRST) twiddle<false, RL>(v, tw, q, len);
#pragma unroll
    for (int m = 0; m < 1 << RL; ++m) { const int x = base + (m << ulog); if (ROWS) store(line, x, v[m]); else store(x, line, v[m]); }
  }
}
template <bool INVERSE, bool ROWS, bool FIRST, class Load, class Store>
__device__ __forceinline__ void fft_pass(const float2 *tw, int lph, int lpw, int r0, int r1, Load load, Store store) {
  const int len = ROWS ? lpw : lph, rl = FIRST ? first_log(len) : len - first_log(len);   // uniform
  if (rl == 3) fft_pass_r<INVERSE, ROWS, FIRST, 3>(tw, lph, lpw, r0, r1, load, store);
  else if (rl == 2) fft_pass_r<INVERSE, ROWS, FIRST, 2>(tw, lph, lpw, r0, r1, load, store);
  else fft_pass_r<INVERSE, ROWS, FIRST, 1>(tw, lph, lpw, r0, r1, load, store);
}

struct FftFwdArgs {
  const float *src;            // plain images [count][H][W], or dy of a layer
  const float *src_y;          // layer output (same shape as dy) where act' needs it
  const unsigned char *src_idx;
  int src_dz, src_act, src_pool;
  int count, H, W;             // real image size before padding (a dz map: pre-pool size)
  int pair_stride;             // > 0: workgroup g packs images g' and g' + pair_stride (the same filter map of
                               // two neighbouring batch images) as real and imaginary part; count = images given,
                               // planes = maps per batch image
  int planes;
  int lph, lpw;                // log2 of the padded sides
  float2 *out;                 // [count][PH * PW], bit-reversed order
};

__device__ __forceinline__ float act_deriv(int act, float out) {
  if (act == ACT_SIGMOID) return out * (1.0f - out);
  if (act == ACT_RELU) return out > 0.0f ? 1.0f : 0.0f;
  return 1.0f;
}

// dz = unpool(dy) * act'(y) at pre-pool position (i, j) of image `img`
__device__ __forceinline__ float fft_src_value(const FftFwdArgs &a, int img, int i, int j) {
  if (!a.src_dz) return a.src[((long)img * a.H + i) * a.W + j];
  long o;
  if (a.src_pool == 2) {
    o = ((long)img * (a.H >> 1) + (i >> 1)) * (a.W >> 1) + (j >> 1);
    const unsigned char f = a.src_idx[o];
    if ((f & kIdxPosMask) != (unsigned char)(((i & 1) << 1) | (j & 1))) return 0.0f;
    if (a.src_act == ACT_RELU_FLAGGED) return (f & kIdxInactive) ? 0.0f : a.src[o];
  } else {
    o = ((long)img * a.H + i) * a.W + j;
  }
  float g = a.src[o];
  if (a.src_act == ACT_SIGMOID || a.src_act == ACT_RELU) g *= act_deriv(a.src_act, a.src_y[o]);
  return g;
}

// Both operands' transforms in one launch: the first `split` workgroups take `x`, the others `w`.
__global__ __launch_bounds__(kFftThreads) void fft2_forward_kernel(const FftFwdArgs x, const FftFwdArgs w, int split) {
  const bool second = (int)blockIdx.x >= split;
  const FftFwdArgs &a = second ? w : x;
  const int block = second ? (int)blockIdx.x - split : (int)blockIdx.x;
  extern __shared__ float2 fbuf[];   // [PH * PW] + twiddles
  const int F = 1 << (a.lph + a.lpw);
  float2 *tw = fbuf + F;
  // packed: workgroup (pair p, plane k) takes images (2p, k) and (2p + 1, k) of [N][planes]
  int img = block, img2 = -1;
  if (a.pair_stride > 0) {
    const int p = block / a.planes, k = block - p * a.planes;
    img = 2 * p * a.planes + k;
    img2 = img + a.pair_stride < a.count ? img + a.pair_stride : -1;
  }
  make_twiddles(tw);
  const int lph = a.lph, lpw = a.lpw;
  float2 *dst = a.out + (long)block * F;
  auto from_image = [&](int i, int c) {
    const bool in = c < a.W;
    return make_float2(in ? fft_src_value(a, img, i, c) : 0.0f, in && img2 >= 0 ? fft_src_value(a, img2, i, c) : 0.0f);
  };
  auto get = [&](int i, int c) { return fbuf[at(i, c, lpw)]; };
  auto get_padded = [&](int i, int c) { return i < a.H ? fbuf[at(i, c, lpw)] : make_float2(0.0f, 0.0f); };
  auto put = [&](int i, int c, float2 v) { fbuf[at(i, c, lpw)] = v; };
  auto to_spectrum = [&](int i, int c, float2 v) { dst[(i << lpw) + c] = v; };
  __syncthreads();   // the twiddles
  // the rows below the image are zero and stay zero under the row transform: they are never touched
  fft_pass<false, true, true>(tw, lph, lpw, 0, a.H, from_image, put);
  __syncthreads();
  if (lpw > 3) {
    fft_pass<false, true, false>(tw, lph, lpw, 0, a.H, get, put);
    __syncthreads();
  }
  if (lph > 3) {
    fft_pass<false, false, true>(tw, lph, lpw, 0, 0, get_padded, put);
    __syncthreads();
    fft_pass<false, false, false>(tw, lph, lpw, 0, 0, get, to_spectrum);
  } else {
    fft_pass<false, false, true>(tw, lph, lpw, 0, 0, get_padded, to_spectrum);
  }
}

struct FftInvArgs {
  const float2 *xf;   // [ceil(N/2)][K][F]: batch images 2p (real part) and 2p + 1 (imaginary part)
  const float2 *wf;   // [K][C][F]
  int N, K, C;
  int lph, lpw;
  int H, W, off;      // output size and the crop offset (the layer's padding)
  float *out;         // [N][C][H][W]
  float2 *yf;         // [ceil(N/2)][C][F]: the products' sums over k
};

// Back from a spectrum (`load` by row and column) to the kept part of image pair (2 pr, 2 pr + 1), channel c.
// Ends without a barrier.
template <class Load>
__device__ __forceinline__ void inverse_image(const FftInvArgs &a, float2 *fbuf, const float2 *tw, int pr, int c, Load load) {
  const int lph = a.lph, lpw = a.lpw, n = 2 * pr;
  const int r0 = a.off, r1 = a.off + a.H;   // rows that are kept
  const float scale = 1.0f / (float)(1 << (lph + lpw));
  float *dst = a.out + ((long)n * a.C + c) * a.H * a.W;
  const long next = (long)a.C * a.H * a.W;   // the pair's second image
  const bool two = n + 1 < a.N;
  auto get = [&](int i, int x) { return fbuf[at(i, x, lpw)]; };
  auto put = [&](int i, int x, float2 v) { fbuf[at(i, x, lpw)] = v; };
  auto put_kept = [&](int i, int x, float2 v) { if (i >= r0 && i < r1) fbuf[at(i, x, lpw)] = v; };
  auto to_image = [&](int i, int x, float2 v) {
    x -= a.off;
    if (x < 0 || x >= a.W) return;
    const int o = (i - r0) * a.W + x;
    dst[o] = v.x * scale;
    if (two) dst[o + next] = v.y * scale;
  };
  if (lph > 3) {
    fft_pass<true, false, false>(tw, lph, lpw, 0, 0, load, put);
    __syncthreads();
    fft_pass<true, false, true>(tw, lph, lpw, 0, 0, get, put_kept);
  } else {
    fft_pass<true, false, true>(tw, lph, lpw, 0, 0, load, put_kept);
  }
  __syncthreads();
  if (lpw > 3) {
    fft_pass<true, true, false>(tw, lph, lpw, r0, r1, get, put);
    __syncthreads();
  }
  fft_pass<true, true, true>(tw, lph, lpw, r0, r1, get, to_image);
}

// Sums over k of the products of the spectra.  A wavefront owns PT image pairs x CT channels at 64 neighbouring
// frequencies, one per lane: every value loaded serves CT (an image's) or PT (a filter's) complex products, and
// every load is 512 contiguous bytes.  The four wavefronts of a workgroup take neighbouring channel tiles of the same
// pairs and meet in the L1 cache.  Inside the inverse kernel, with a whole spectrum per workgroup, registers
// allowed tiles of 2 x 2 and the stage was bound by re-reading spectra from L2 (1 GB for 32 pairs x 32
// channels x 32 maps at 64 x 64; 4 x 8 tiles read a third of that).  Product and inverse 128 -> 35 + 16 us.
template <int PT, int CT>
__global__ __launch_bounds__(kFftThreads) void fft2_product_kernel(const FftInvArgs a, int ctiles, int tiles) {
  const int F = 1 << (a.lph + a.lpw), lane = threadIdx.x & 63;
  const int tile = __builtin_amdgcn_readfirstlane(blockIdx.y * 4 + (threadIdx.x >> 6));
  if (tile >= tiles) return;
  const int pairs = (a.N + 1) / 2;
  const int pr0 = tile / ctiles * PT, c0 = tile % ctiles * CT;
  const int f = blockIdx.x * 64 + lane, fc = f < F ? f : 0;
  float2 acc[PT][CT];
#pragma unroll
  for (int i = 0; i < PT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[i][j] = make_float2(0.0f, 0.0f);
  // surplus rows and columns of the last tiles re-read the last pair / channel and are never stored
  const float2 *xp[PT], *wp[CT];
#pragma unroll
  for (int i = 0; i < PT; ++i) xp[i] = a.xf + (long)min(pr0 + i, pairs - 1) * a.K * F;
#pragma unroll
  for (int j = 0; j < CT; ++j) wp[j] = a.wf + (long)min(c0 + j, a.C - 1) * F;
  float2 xv[2][PT], wv[2][CT];
  auto load = [&](int b, int k) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PT; ++i) xv[b][i] = xp[i][(long)k * F + fc];
#pragma unroll
    for (int j = 0; j < CT; ++j) wv[b][j] = wp[j][(long)k * a.C * F + fc];
  };
  auto multiply = [&](int b) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) {
        const float2 p = cmul(xv[b][i], wv[b][j]);
        acc[i][j].x += p.x;
        acc[i][j].y += p.y;
      }
  };
  // the next k's values are on their way while one k is multiplied; the last k is re-read, not multiplied
  load(0, 0);
  for (int k = 0; k < a.K; k += 2) {
    load(1, min(k + 1, a.K - 1));
    __builtin_amdgcn_sched_barrier(0);
    multiply(0);
    __builtin_amdgcn_sched_barrier(0);
    load(0, min(k + 2, a.K - 1));
    __builtin_amdgcn_sched_barrier(0);
    if (k + 1 < a.K) multiply(1);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (f >= F) return;
#pragma unroll
  for (int i = 0; i < PT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j)
      if (pr0 + i < pairs && c0 + j < a.C) a.yf[((long)(pr0 + i) * a.C + c0 + j) * F + f] = acc[i][j];
}

__global__ __launch_bounds__(kFftThreads) void fft2_inverse_kernel(const FftInvArgs a) {
  extern __shared__ float2 fbuf[];
  float2 *tw = fbuf + (1 << (a.lph + a.lpw));
  make_twiddles(tw);
  __syncthreads();
  const int pr = blockIdx.x / a.C, c = blockIdx.x - pr * a.C;
  const float2 *src = a.yf + ((long)blockIdx.x << (a.lph + a.lpw));
  inverse_image(a, fbuf, tw, pr, c, [&](int i, int x) { return src[(i << a.lpw) + x]; });
}

// PT pairs of batch images x CT channels per workgroup: every spectrum entry that is loaded serves
// PT (a filter's) or CT (an image's) products, which is what the product stage is bound by.
template <int PT, int CT>
__global__ __launch_bounds__(kFftThreads) void fft2_product_inverse_kernel(const FftInvArgs a) {
  extern __shared__ float2 fbuf[];
  const int PW = 1 << a.lpw, F = PW << a.lph;
  float2 *tw = fbuf + F;
  const int c0 = blockIdx.x * CT, pr0 = blockIdx.y * PT;
  const int pairs = (a.N + 1) / 2;
  make_twiddles(tw);
  constexpr int kSlots = (1 << (2 * kMaxLog)) / kFftThreads;   // 16 spectrum entries per thread at 64 x 64
  constexpr int kBatch = PT * CT > 1 ? kSlots / 2 : kSlots;    // entries whose loads are in flight together
  float2 acc[PT][CT][kSlots];
#pragma unroll
  for (int i = 0; i < PT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
      for (int q = 0; q < kSlots; ++q) acc[i][j][q] = make_float2(0.0f, 0.0f);
  // surplus rows and columns of the last tiles re-read the last pair / channel and are never stored
  const float2 *xp[PT], *wp[CT];
#pragma unroll
  for (int i = 0; i < PT; ++i) xp[i] = a.xf + (long)min(pr0 + i, pairs - 1) * a.K * F;
#pragma unroll
  for (int j = 0; j < CT; ++j) wp[j] = a.wf + (long)min(c0 + j, a.C - 1) * F;
  for (int k = 0; k < a.K; ++k) {
#pragma unroll
    for (int h = 0; h < kSlots / kBatch; ++h) {
      // loads first, products after: entries past F re-read entry 0 and are never stored
      float2 xv[PT][kBatch], wv[CT][kBatch];
#pragma unroll
      for (int q = 0; q < kBatch; ++q) {
        const int e = threadIdx.x + (h * kBatch + q) * kFftThreads;
        const int ec = e < F ? e : 0;
#pragma unroll
        for (int i = 0; i < PT; ++i) xv[i][q] = xp[i][(long)k * F + ec];
#pragma unroll
        for (int j = 0; j < CT; ++j) wv[j][q] = wp[j][(long)k * a.C * F + ec];
      }
#pragma unroll
      for (int q = 0; q < kBatch; ++q)
#pragma unroll
        for (int i = 0; i < PT; ++i)
#pragma unroll
          for (int j = 0; j < CT; ++j) {
            const float2 p = cmul(xv[i][q], wv[j][q]);
            acc[i][j][h * kBatch + q].x += p.x;
            acc[i][j][h * kBatch + q].y += p.y;
          }
    }
  }
#pragma unroll
  for (int i = 0; i < PT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j) {
      const int pr = pr0 + i, c = c0 + j;
      if (pr >= pairs || c >= a.C) continue;   // uniform over the workgroup
      __syncthreads();   // the previous image has been read out
#pragma unroll
      for (int q = 0; q < kSlots; ++q) {
        const int e = threadIdx.x + q * kFftThreads;
        if (e < F) fbuf[at(e >> a.lpw, e & (PW - 1), a.lpw)] = acc[i][j][q];
      }
      __syncthreads();
      inverse_image(a, fbuf, tw, pr, c, [&](int r, int x) { return fbuf[at(r, x, a.lpw)]; });
    }
}

int log2_ceil(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}

}  // namespace

bool conv_fft_plan(int Ho, int Wo, int R, int S, int *lph, int *lpw) {
  const int fh = Ho + R - 1, fw = Wo + S - 1;   // size of the full convolution
  if (fh < 1 || fw < 1 || fh > (1 << kMaxLog) || fw > (1 << kMaxLog)) return false;
  int a = log2_ceil(fh), b = log2_ceil(fw);
  if (a < 1) a = 1;
  if (b < 1) b = 1;
  *lph = a; *lpw = b;
  return true;
}

hipError_t launch_conv_full_fft(const ConvFftArgs &g, hipStream_t stream) {
  int lph, lpw;
  if (!conv_fft_plan(g.Ho, g.Wo, g.R, g.S, &lph, &lpw)) return hipErrorInvalidValue;
  const int F = 1 << (lph + lpw);
  const size_t lds = (size_t)(F + kTw) * sizeof(float2);
  FftFwdArgs x;
  x.src = g.dy; x.src_y = g.y; x.src_idx = g.idx;
  x.src_dz = 1; x.src_act = g.act; x.src_pool = g.pool;
  x.count = g.N * g.K; x.H = g.Ho; x.W = g.Wo; x.lph = lph; x.lpw = lpw;
  x.pair_stride = g.K; x.planes = g.K;
  x.out = g.xf;
  const int pairs = (g.N + 1) / 2;
  FftFwdArgs f;
  f.src = g.w; f.src_y = nullptr; f.src_idx = nullptr;
  f.src_dz = 0; f.src_act = ACT_IDENTITY; f.src_pool = 1;
  f.count = g.K * g.C; f.H = g.R; f.W = g.S; f.lph = lph; f.lpw = lpw;
  f.pair_stride = 0; f.planes = 1;
  f.out = g.wf;
  const long nx = (long)pairs * g.K, nw = f.count;
  if (nx + nw <= kMaxGrid) {
    hipLaunchKernelGGL(fft2_forward_kernel, dim3((unsigned)(nx + nw)), dim3(kFftThreads), lds, stream, x, f, (int)nx);
  } else {   // more transforms than a grid holds: one operand after the other
    hipLaunchKernelGGL(fft2_forward_kernel, dim3((unsigned)nx), dim3(kFftThreads), lds, stream, x, f, (int)nx);
    hipLaunchKernelGGL(fft2_forward_kernel, dim3((unsigned)nw), dim3(kFftThreads), lds, stream, x, f, 0);
  }
  FftInvArgs v;
  v.xf = g.xf; v.wf = g.wf; v.N = g.N; v.K = g.K; v.C = g.C; v.lph = lph; v.lpw = lpw;
  v.H = g.H; v.W = g.W; v.off = g.pad; v.out = g.dx;
  v.yf = g.yf;
  if (g.yf && (long)pairs * g.C <= kMaxGrid) {
    // 4 x 8 tiles once they give every SIMD of the chip two wavefronts (one wavefront of 8 x 8 tiles moves
    // less but waits out every k's loads: 38 against 35 us at 32 x 32 x 32 maps), 4 x 4 ones below
    const int chunks = (F + 63) / 64, prows = (pairs + 3) / 4;
    const int c8 = (g.C + 7) / 8, c4 = (g.C + 3) / 4;
    if ((long)c8 * prows * chunks >= 8L * chip().cus)
      hipLaunchKernelGGL((fft2_product_kernel<4, 8>), dim3(chunks, (c8 * prows + 3) / 4), dim3(kFftThreads), 0, stream, v, c8, c8 * prows);
    else
      hipLaunchKernelGGL((fft2_product_kernel<4, 4>), dim3(chunks, (c4 * prows + 3) / 4), dim3(kFftThreads), 0, stream, v, c4, c4 * prows);
    hipLaunchKernelGGL(fft2_inverse_kernel, dim3(pairs * g.C), dim3(kFftThreads), lds, stream, v);
    return hipGetLastError();
  }
  // 2 x 2 tiles once there is enough work to fill the chip with them
  if ((long)pairs * g.C >= 4L * chip().cus)
    hipLaunchKernelGGL((fft2_product_inverse_kernel<2, 2>), dim3((g.C + 1) / 2, (pairs + 1) / 2), dim3(kFftThreads), lds, stream, v);
  else
    hipLaunchKernelGGL((fft2_product_inverse_kernel<1, 1>), dim3(g.C, pairs), dim3(kFftThreads), lds, stream, v);
  return hipGetLastError();
}

}  // namespace dllk
