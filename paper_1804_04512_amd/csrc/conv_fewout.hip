// Forward-form convolution with very few output channels (Kout <= 3) on fp32 MFMA.
//
// The case: the CRBM's visible reconstruction (Section II: the full convolution of the hidden
// states with the filters, K hidden maps -> one or three visible maps) and the backward-data pass
// into a grey-scale or RGB input (Section II-A).  With output channels on the MFMA N axis, as in
// the general engine, 15 of 16 columns would multiply zeros.  Here the N axis carries 16
// neighbouring output COLUMNS instead, and the filter enters as a banded (Toeplitz) operand:
//   out[i, j0+jj] = sum_{c,r,t} win[c][i+r][t] * B[(c,r,t)][jj],   B[(c,r,t)][jj] = wgt[c][r][t-jj] (0 <= t-jj < S)
// with win the source window of the tile (16+R-1 rows, 16+S-1 columns, zero outside the image).
// M = 16 output rows, N = 16 output columns, K = (channel, filter row, window column): S of every
// 16+S-1 products are real, e.g. 9/24 for 9x9 filters instead of 1/16.  B fragments are read from
// the compact filter rows in LDS (each row padded with zeros on both sides), so the banded matrix
// is never stored.
//
// One workgroup = one 16x16 output tile of one image, all (<= 3) output channels.  The wavefronts split the
// source channels: each stages one channel's window and filter rows in LDS of its own, so nothing in the loop
// waits for a workgroup, and has the next channel's values on their way while it multiplies.  The
// partial tiles are added in wavefront order at the end.  Which element of a plane a lane moves, and to where, is
// the same for every channel and worked out once.  (The form before staged eight channels at a time for
// the whole workgroup, three divisions by run-time sizes per element and nothing in flight during the
// products: 64 x 40 maps of 20 x 20 back through 9 x 9 filters 45 -> 20 us, of which the products are 7.)
#include "dll_internal.h"

namespace dllk {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kRsx = 34;           // LDS row stride of the window: 2 mod 32 -> conflict-free A reads
constexpr int kSteps = 8;          // MFMA steps a window row can have (window <= 32 columns: S <= 17)
constexpr int kRoww = 15 + 4 * kSteps + 1;   // filter row: 15 zeros, the taps, zeros up to the last column a lane reads
constexpr int kTapSlots = 7;       // filter values per lane and channel: at most 3 x 144
constexpr int kPlaneSlots = 32;    // window values per lane and channel at most
constexpr unsigned kOob = 0x80000000u;   // byte offset past any plane: the range check returns zero

struct FewoutParams {
  ConvEngineArgs a;
  int tiles_x, tiles_y;
  int rows;        // window rows = 16 + R - 1
  int winp;        // window columns staged = 4 * wsteps >= 16 + S - 1
  int wsteps;
  int inv_winp;    // ceil(65536 / winp): exact division of a plane's element numbers
};

__device__ __forceinline__ float act_apply(int act, float z) {
  if (act == ACT_SIGMOID) return 1.0f / (1.0f + expf(-z));
  if (act == ACT_RELU) return z > 0.0f ? z : 0.0f;
  return z;
}

// The same sums tap by tap, straight from memory: the zeros beside the band carry an infinity or NaN of the source into
// all 16 columns, so a wavefront with finite sums and others takes its channels again here, and it reaches the
// outputs whose windows hold it and no others (a filter of more than 16 rows can leave no sum of a tile finite).  It reads the kernel's arguments again: kept in scalar registers for it,
// they cost the loop above 2 to 8 %.
template <int KO, int WAVES, bool POOL>
__device__ __forceinline__ void tap_by_tap(floatx4 (&acc)[KO]) {
  unsigned long args = (unsigned long)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(args));
  const auto &p = *(const __attribute__((address_space(4))) FewoutParams *)args;
  const auto &a = p.a;
  const int bid = blockIdx.x, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = bid / (p.tiles_x * p.tiles_y), ty = (bid / p.tiles_x) % p.tiles_y;
  const int i = ty * 16 + 4 * (lane >> 4), j = bid % p.tiles_x * 16 + (lane & 15);
  const int RSf = a.R * a.S, Ws = POOL ? a.Win >> 1 : a.Win, Hs = POOL ? a.Hin >> 1 : a.Hin;
#pragma unroll
  for (int c = 0; c < KO; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int ci = wave; ci < a.Cin; ci += WAVES)
    for (int rs = 0; rs < RSf; ++rs) {
      const int gj = j - a.pad_w + rs % a.S;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int gi = i + v - a.pad_h + rs / a.S;
        if (gi < 0 || gi >= a.Hin || gj < 0 || gj >= a.Win) continue;
        const long o = ((long)(n * a.Cin + ci) * Hs + (POOL ? gi >> 1 : gi)) * Ws + (POOL ? gj >> 1 : gj);
        float x = a.src[o];
        if (a.src_dz && a.src_act == ACT_SIGMOID) x *= a.src_y[o] * (1.0f - a.src_y[o]);
        if (a.src_dz && a.src_act == ACT_RELU) x = a.src_y[o] > 0.0f ? x : 0.0f;
        if constexpr (POOL) {
          const unsigned char f = a.src_idx[o];
          if ((f & kIdxPosMask) != (((gi & 1) << 1) | (gj & 1)) || (a.src_act == ACT_RELU_FLAGGED && (f & kIdxInactive))) x = 0.0f;
        }
#pragma unroll
        for (int c = 0; c < KO; ++c)
          acc[c][v] = fmaf(x, a.w[a.w_flip ? (long)(ci * KO + c) * RSf + (RSf - 1 - rs) : (long)(c * a.Cin + ci) * RSf + rs], acc[c][v]);
      }
    }
}

// NS: window values per lane and channel; POOL: the source is dz behind 2x2 pooling
template <int KO, int NS, int WAVES, bool POOL>
__global__ __launch_bounds__(WAVES * 64) void conv_fewout_kernel(const FewoutParams p) {
  extern __shared__ float lds[];
  const ConvEngineArgs &a = p.a;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, kq = lane >> 4;
  const int psx = p.rows * kRsx, wrows = KO * a.R * kRoww;
  float *xs = lds + wave * (psx + wrows);   // [rows][kRsx], this wavefront's
  float *wf = xs + psx;                     // [KO][R][kRoww]
  const int bid = blockIdx.x;
  const int tx = bid % p.tiles_x, ty = (bid / p.tiles_x) % p.tiles_y, n = bid / (p.tiles_x * p.tiles_y);
  const int i0 = ty * 16, j0 = tx * 16;
  const int RSf = a.R * a.S;
  const int Wsrc = POOL ? a.Win >> 1 : a.Win, HW = (POOL ? a.Hin >> 1 : a.Hin) * Wsrc;   // of a plane as it is stored
  const bool need_y = a.src_dz && (a.src_act == ACT_SIGMOID || a.src_act == ACT_RELU);

  // the lane's window elements: byte offset inside a source plane (out of range: padding), LDS offset
  const int plane = p.rows * p.winp;
  int voff[NS], dst[NS];
  unsigned char want[POOL ? NS : 1], fv[POOL ? NS : 1];   // position inside the pooling window; the window's byte
#pragma unroll
  for (int u = 0; u < NS; ++u) {
    const int e = lane + 64 * u;
    const int y = (e * p.inv_winp) >> 16, x = e - y * p.winp;
    const int gi = i0 - a.pad_h + y, gj = j0 - a.pad_w + x;
    voff[u] = (e < plane && gi >= 0 && gi < a.Hin && gj >= 0 && gj < a.Win) ? (POOL ? 4 * ((gi >> 1) * Wsrc + (gj >> 1)) : 4 * (gi * a.Win + gj)) : (int)kOob;
    dst[u] = e < plane ? y * kRsx + x : -1;
    if (POOL) want[u] = ((gi & 1) << 1) | (gj & 1);
  }
  // the lane's filter taps: byte offset from the channel's first, LDS offset
  int woff[kTapSlots], wdst[kTapSlots];
  const int taps = KO * RSf;
  for (int e = lane; e < wrows; e += 64) wf[e] = 0.0f;   // the zero borders stay, the taps are rewritten
#pragma unroll
  for (int u = 0; u < kTapSlots; ++u) {
    const int e = lane + 64 * u;
    woff[u] = (int)kOob;
    wdst[u] = -1;
    if (64 * u >= taps || e >= taps) continue;
    const int c = e / RSf, rs = e - c * RSf, r = rs / a.S, s = rs - r * a.S;
    woff[u] = 4 * (a.w_flip ? c * RSf + (a.R - 1 - r) * a.S + (a.S - 1 - s) : c * a.Cin * RSf + rs);
    wdst[u] = (c * a.R + r) * kRoww + 15 + s;
  }

  float gv[NS], yv[NS], tv[kTapSlots];
  auto load_channel = [&](int ci) __attribute__((always_inline)) {
    const long base = (long)(n * a.Cin + ci) * HW;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.src + base), 0, 4 * HW, 0x00020000);
#pragma unroll
    for (int u = 0; u < NS; ++u) gv[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, voff[u], 0, 0));
    if (need_y) {
      const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.src_y + base), 0, 4 * HW, 0x00020000);
#pragma unroll
      for (int u = 0; u < NS; ++u) yv[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ry, voff[u], 0, 0));
    }
    if constexpr (POOL) {
      const __amdgpu_buffer_rsrc_t ri = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(a.src_idx + base), 0, HW, 0x00020000);
#pragma unroll
      for (int u = 0; u < NS; ++u) fv[u] = __builtin_amdgcn_raw_buffer_load_b8(ri, (int)((unsigned)voff[u] >> 2), 0, 0);
    }
    const float *w0 = a.w + (long)ci * (a.w_flip ? KO * RSf : RSf);
    const int wbytes = a.w_flip ? 4 * taps : 4 * (((KO - 1) * a.Cin + 1) * RSf);   // to the end of the channel's last filter
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(w0), 0, wbytes, 0x00020000);
#pragma unroll
    for (int u = 0; u < kTapSlots; ++u)
      if (64 * u < taps) tv[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rw, woff[u], 0, 0));
  };
  auto store_channel = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      float v = gv[u];
      if (need_y) {   // dz = dy * act'(y), from the layer output
        if (a.src_act == ACT_SIGMOID) v *= yv[u] * (1.0f - yv[u]);
        else v = yv[u] > 0.0f ? v : 0.0f;
      }
      if constexpr (POOL) {   // the gradient sits at the recorded position
        const bool off = (fv[u] & kIdxPosMask) != want[u] || (a.src_act == ACT_RELU_FLAGGED && (fv[u] & kIdxInactive));
        v = off ? 0.0f : v;
      }
      if (dst[u] >= 0) xs[dst[u]] = v;
    }
#pragma unroll
    for (int u = 0; u < kTapSlots; ++u)
      if (64 * u < taps && wdst[u] >= 0) wf[wdst[u]] = tv[u];
  };

  floatx4 acc[KO];
#pragma unroll
  for (int c = 0; c < KO; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};

  if (wave < a.Cin) load_channel(wave);
  for (int ci = wave; ci < a.Cin; ci += WAVES) {
    store_channel();
    if (ci + WAVES < a.Cin) load_channel(ci + WAVES);   // in flight during the products
    // LDS of one wavefront: its accesses are served in order, only the compiler must keep them so
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // ---- MFMA over the channel's filter rows; the fragments of the next row are read from LDS while the
    // current one is multiplied.  A: lane (row i16, k = kq) reads window column 4*step + kq of row
    // i16 + r; B: lane (column i16, k = kq) reads tap 4*step + kq - i16 of the padded filter row (zero
    // outside the S taps).
    {
      float afA[kSteps], afB[kSteps], bfA[KO][kSteps], bfB[KO][kSteps];
      auto load_row = [&](int r, float (&af)[kSteps], float (&bf)[KO][kSteps]) __attribute__((always_inline)) {
        const float *ap = xs + (i16 + r) * kRsx + kq;
#pragma unroll
        for (int st = 0; st < kSteps; ++st) af[st] = ap[4 * st];
#pragma unroll
        for (int c = 0; c < KO; ++c) {
          const float *bp = wf + (c * a.R + r) * kRoww + 15 + kq - i16;
#pragma unroll
          for (int st = 0; st < kSteps; ++st) bf[c][st] = bp[4 * st];
        }
      };
      auto mfma_row = [&](const float (&af)[kSteps], const float (&bf)[KO][kSteps]) __attribute__((always_inline)) {
#pragma unroll
        for (int st = 0; st < kSteps; ++st) {
          if (st < p.wsteps) {
#pragma unroll
            for (int c = 0; c < KO; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[st], bf[c][st], acc[c], 0, 0, 0);
          }
        }
      };
      load_row(0, afA, bfA);
      for (int r = 0; r < a.R; r += 2) {   // a row past the last re-reads it and is not multiplied
        load_row(min(r + 1, a.R - 1), afB, bfB);
        __builtin_amdgcn_sched_barrier(0);
        mfma_row(afA, bfA);
        __builtin_amdgcn_sched_barrier(0);
        load_row(min(r + 2, a.R - 1), afA, bfA);
        __builtin_amdgcn_sched_barrier(0);
        if (r + 1 < a.R) mfma_row(afB, bfB);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }

  // (a tile with no finite output, as all are once a training run has diverged, has nothing to set apart)
  bool some = false, all = true;
#pragma unroll
  for (int c = 0; c < KO; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const bool stored = i0 + 4 * kq + v < a.Hout && j0 + i16 < a.Wout, finite = __builtin_isfinite(acc[c][v]);
      some = some || (stored && finite);
      all = all && (!stored || finite);
    }
  if (!__all(all) && __any(some)) tap_by_tap<KO, WAVES, POOL>(acc);

  // ---- the wavefronts' partial tiles, added in wavefront order, then bias, activation, store.
  // Lane holds D[row 4*kq + v][column i16].
  __syncthreads();
  float *red = lds;   // [wave][KO][lane][4]
#pragma unroll
  for (int c = 0; c < KO; ++c)
    *reinterpret_cast<float4 *>(red + ((wave * KO + c) * 64 + lane) * 4) = make_float4(acc[c][0], acc[c][1], acc[c][2], acc[c][3]);
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int c = 0; c < KO; ++c) {
      float4 s = *reinterpret_cast<const float4 *>(red + ((0 * KO + c) * 64 + lane) * 4);
#pragma unroll
      for (int w = 1; w < WAVES; ++w) {
        const float4 t = *reinterpret_cast<const float4 *>(red + ((w * KO + c) * 64 + lane) * 4);
        s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
      }
      const float bv = a.bias ? a.bias[c] : 0.0f;
      const float sv[4] = {s.x, s.y, s.z, s.w};
      const int oj = j0 + i16;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int oi = i0 + 4 * kq + v;
        if (oi < a.Hout && oj < a.Wout) a.out[((n * a.Kout + c) * a.Hout + oi) * a.Wout + oj] = act_apply(a.act, sv[v] + bv);
      }
    }
  }
}

size_t fewout_lds_bytes(const ConvEngineArgs &a, int waves) {
  const size_t stage = sizeof(float) * waves * ((size_t)(16 + a.R - 1) * kRsx + (size_t)a.Kout * a.R * kRoww);
  const size_t red = sizeof(float) * waves * (size_t)a.Kout * 64 * 4;
  return stage > red ? stage : red;
}
inline int fewout_winp(const ConvEngineArgs &a) { return 4 * ((16 + a.S - 1 + 3) / 4); }

template <int KO, int NS>
hipError_t launch_fewout_t(const FewoutParams &p, unsigned blocks, int waves, hipStream_t stream) {
  const size_t lds = fewout_lds_bytes(p.a, waves);
  auto launch = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * waves), lds, stream, p);
    return hipGetLastError();
  };
  // (the largest window's pooled form needs more registers than eight wavefronts leave: the launcher asks for four)
  if constexpr (NS == kPlaneSlots) {
    if (p.a.src_dz && p.a.src_pool == 2) return launch(conv_fewout_kernel<KO, NS, 4, true>);
  } else {
    if (p.a.src_dz && p.a.src_pool == 2) return waves == 8 ? launch(conv_fewout_kernel<KO, NS, 8, true>) : launch(conv_fewout_kernel<KO, NS, 4, true>);
  }
  return waves == 8 ? launch(conv_fewout_kernel<KO, NS, 8, false>) : launch(conv_fewout_kernel<KO, NS, 4, false>);
}
template <int KO>
hipError_t launch_fewout_k(const FewoutParams &p, unsigned blocks, int waves, hipStream_t stream) {
  const int slots = (p.rows * p.winp + 63) / 64;
  if (slots <= 7) return launch_fewout_t<KO, 7>(p, blocks, waves, stream);    // 5x5 filters and smaller
  if (slots <= 12) return launch_fewout_t<KO, 12>(p, blocks, waves, stream);
  return launch_fewout_t<KO, kPlaneSlots>(p, blocks, waves, stream);
}

}  // namespace

bool conv_fewout_applies(const ConvEngineArgs &a) {
  if (a.Kout > 3 || a.pool != 1 || a.sample || a.out_pool) return false;
  if (a.act != ACT_IDENTITY && a.act != ACT_SIGMOID && a.act != ACT_RELU) return false;
  if (a.src_dz && a.src_pool != 2 && a.src_act != ACT_IDENTITY && a.src_act != ACT_SIGMOID && a.src_act != ACT_RELU) return false;
  if (16 + a.S - 1 > 4 * kSteps || (16 + a.R - 1) * fewout_winp(a) > 64 * kPlaneSlots || a.Kout * a.R * a.S > 64 * kTapSlots) return false;
  if ((long)a.N * ((a.Hout + 15) / 16) * ((a.Wout + 15) / 16) > kMaxGrid) return false;   // the engine's tiles are wider
  // 32-bit byte offsets inside a plane and a channel's filters
  if (4L * a.Hin * a.Win >= (long)kOob || 4L * a.Kout * a.Cin * a.R * a.S >= (long)kOob) return false;
  return fewout_lds_bytes(a, 4) <= 64 * 1024;
}

hipError_t launch_conv_fewout(const ConvEngineArgs &a, hipStream_t stream) {
  FewoutParams p;
  p.a = a;
  p.tiles_x = (a.Wout + 15) / 16;
  p.tiles_y = (a.Hout + 15) / 16;
  p.rows = 16 + a.R - 1;
  p.winp = fewout_winp(a);
  p.wsteps = p.winp / 4;
  p.inv_winp = (65536 + p.winp - 1) / p.winp;
  const long blocks = (long)a.N * p.tiles_x * p.tiles_y;
  if (blocks <= 0 || blocks > kMaxGrid) return hipErrorInvalidValue;
  // eight wavefronts a tile halve the chain of channels each walks, as long as the tiles alone leave SIMDs idle
  const bool huge = a.src_dz && a.src_pool == 2 && p.rows * p.winp > 64 * 12;
  const int waves = !huge && a.Cin > 4 && blocks < 4L * chip().cus && fewout_lds_bytes(a, 8) <= 64 * 1024 ? 8 : 4;
  switch (a.Kout) {
    case 1: return launch_fewout_k<1>(p, (unsigned)blocks, waves, stream);
    case 2: return launch_fewout_k<2>(p, (unsigned)blocks, waves, stream);
    case 3: return launch_fewout_k<3>(p, (unsigned)blocks, waves, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace dllk
