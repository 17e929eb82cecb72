// One output tile of the small fp32 MFMA product, shared by its own launch (gemm_small.hip) and by the
// training step's closing launch (conv_wgrad.hip), where products that nothing later waits for run as jobs.
#pragma once

#include "dll_internal.h"

namespace dllk {
namespace small_gemm {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int KT = 32;    // k-tile

__device__ __forceinline__ float act_apply(int act, float z) {
  if (act == ACT_SIGMOID) return 1.0f / (1.0f + expf(-z));
  if (act == ACT_RELU) return z > 0.0f ? z : 0.0f;
  return z;
}
__device__ __forceinline__ float act_deriv(int act, float out) {
  if (act == ACT_SIGMOID) return out * (1.0f - out);
  if (act == ACT_RELU) return out > 0.0f ? 1.0f : 0.0f;
  return 1.0f;
}

struct SmallParams {
  GemmArgs a;
  unsigned a_bytes, b_bytes;   // extents of the operands (below 2 GiB)
  int whole;                   // aligned rows of whole 16-byte groups: of every k-contiguous operand; weight-gradient form: of the result
};

constexpr unsigned kOob = 0x80000000u;   // byte offset beyond any operand: reads as zero

// One operand's fragments of a k-tile: frag[t][s] = X(x0 + 16 t + i16, k0 + 8 kq + s), X(x, k) = src[x * sx + k * sk];
// `row[t]`: byte offset of the lane's row, kOob past the operand's last one.  Range-checked buffer
// loads: a k past the end gets the out-of-range offset and reads zero.  Nothing here depends on a loaded
// value.
// A k-contiguous operand is read 16 bytes at a time, which needs no more than 4-byte alignment; unless
// its rows are whole groups, `clear_tail` takes off what a row's last group holds of the next row.
template <bool KC, int Q>
__device__ __forceinline__ void load_frags(float (&frag)[Q][8], const __amdgpu_buffer_rsrc_t &src, const unsigned (&row)[Q],
                                           unsigned sk_bytes, int k, int Kdim) {
#pragma unroll
  for (int t = 0; t < Q; ++t) {
    if constexpr (KC) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int kk = k + 4 * h;
        const floatx4 v = __builtin_bit_cast(
            floatx4, __builtin_amdgcn_raw_buffer_load_b128(src, (int)(kk < Kdim ? row[t] + 4u * (unsigned)kk : kOob), 0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) frag[t][4 * h + e] = v[e];
      }
    } else {
#pragma unroll
      for (int s = 0; s < 8; ++s)
        frag[t][s] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                   src, (int)(k + s < Kdim ? row[t] + (unsigned)(k + s) * sk_bytes : kOob), 0, 0));
    }
  }
}
template <int Q>
__device__ __forceinline__ void clear_tail(float (&frag)[Q][8], int k, int Kdim) {
#pragma unroll
  for (int t = 0; t < Q; ++t)
#pragma unroll
    for (int s = 0; s < 8; ++s) frag[t][s] = k + s < Kdim ? frag[t][s] : 0.0f;
}

// Floats of LDS a tile needs: [wavefront][quarter][lane][4].
template <int WAVES, int Q> constexpr int kRedFloats = WAVES * Q * Q * 64 * 4;

// Q = 2: 32 x 32 tile (four 16 x 16 quarters); Q = 1: 16 x 16 tile, for products whose 32 x 32 tiles
// would occupy a small part of the chip with long k loops.  A is contiguous along k.
// EXTRAS: the RBM's epilogues (states, squared differences) exist.  (mt, nt): the tile; tile: its number.
template <bool B_KC, bool WHOLE, int WAVES, int Q, bool EXTRAS>
__device__ __forceinline__ void tile_product(const SmallParams &p, int mt, int nt, int tile, float *lds) {
  constexpr int TS = 16 * Q;
  float (*red)[Q * Q][64][4] = reinterpret_cast<float (*)[Q * Q][64][4]>(lds);
  const GemmArgs &a = p.a;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i16 = lane & 15, kq = lane >> 4;
  const int m0 = mt * TS, n0 = nt * TS;
  const int nkt = (a.Kdim + KT - 1) / KT;

  floatx4 acc[Q][Q];   // [m quarter][n quarter]; lane holds C(m = i16, n = 4 kq + v)
#pragma unroll
  for (int i = 0; i < Q; ++i)
#pragma unroll
    for (int j = 0; j < Q; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  float afA[Q][8], bfA[Q][8], afB[Q][8], bfB[Q][8], afC[Q][8], bfC[Q][8], afD[Q][8], bfD[Q][8];
  const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.A), 0, (int)p.a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.B), 0, (int)p.b_bytes, 0x00020000);
  unsigned rowA[Q], rowB[Q];
#pragma unroll
  for (int t = 0; t < Q; ++t) {
    const int m = m0 + 16 * t + i16, n = n0 + 16 * t + i16;
    rowA[t] = m < a.M ? 4u * (unsigned)m * (unsigned)a.a_m : kOob;
    rowB[t] = n < a.N ? 4u * (unsigned)n * (unsigned)a.b_n : kOob;
  }
  const unsigned skB = 4u * (unsigned)a.b_k;
  // (a row past the end plus a k stays past the end: the operands are below 2 GiB)
  // Two k-contiguous operands: a k-tile is four load instructions, issued whether it exists or not (past the
  // last one they read zeros without touching memory), so that the compiler can wait for one k-tile and
  // leave the later ones in flight (100 x 64 x 1536: 11.3 -> 8.2 us).  An operand read across k takes 8 per
  // 16 rows: there a k-tile that does not exist is not asked for.
  auto load_tile = [&](int kt, float (&af)[Q][8], float (&bf)[Q][8]) __attribute__((always_inline)) {
    if (!B_KC && kt >= nkt) return;
    const int k = kt * KT + 8 * kq;
    load_frags<true, Q>(af, rsA, rowA, 4u, k, a.Kdim);
    load_frags<B_KC, Q>(bf, rsB, rowB, skB, k, a.Kdim);
  };
  auto multiply = [&](int kt, float (&af)[Q][8], float (&bf)[Q][8]) __attribute__((always_inline)) {
    if constexpr (!WHOLE) {   // both operands: a neighbour row's infinity must not meet the other's zero
      clear_tail<Q>(af, kt * KT + 8 * kq, a.Kdim);
      if constexpr (B_KC) clear_tail<Q>(bf, kt * KT + 8 * kq, a.Kdim);
    }
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
      for (int i = 0; i < Q; ++i)
#pragma unroll
        for (int j = 0; j < Q; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf[j][s], af[i][s], acc[i][j], 0, 0, 0);
  };
  // this wavefront's k-tiles: wave, wave + WAVES, ...; four register sets, so that three k-tiles'
  // loads are in flight while one is multiplied: with a handful of workgroups on the whole chip
  // (a batch-by-64 product over a long k) the loop runs at memory latency divided by that depth
  if (wave < nkt) {
    load_tile(wave, afA, bfA);
    load_tile(wave + WAVES, afB, bfB);
    load_tile(wave + 2 * WAVES, afC, bfC);
    for (int kt = wave; kt < nkt; kt += 4 * WAVES) {
      load_tile(kt + 3 * WAVES, afD, bfD);
      __builtin_amdgcn_sched_barrier(0);
      multiply(kt, afA, bfA);
      __builtin_amdgcn_sched_barrier(0);
      load_tile(kt + 4 * WAVES, afA, bfA);
      __builtin_amdgcn_sched_barrier(0);
      if (kt + WAVES < nkt) multiply(kt + WAVES, afB, bfB);
      __builtin_amdgcn_sched_barrier(0);
      load_tile(kt + 5 * WAVES, afB, bfB);
      __builtin_amdgcn_sched_barrier(0);
      if (kt + 2 * WAVES < nkt) multiply(kt + 2 * WAVES, afC, bfC);
      __builtin_amdgcn_sched_barrier(0);
      load_tile(kt + 6 * WAVES, afC, bfC);
      __builtin_amdgcn_sched_barrier(0);
      if (kt + 3 * WAVES < nkt) multiply(kt + 3 * WAVES, afD, bfD);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- the partial tiles meet in LDS
#pragma unroll
  for (int i = 0; i < Q; ++i)
#pragma unroll
    for (int j = 0; j < Q; ++j)
      *reinterpret_cast<float4 *>(&red[wave][Q * i + j][lane][0]) = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
  __syncthreads();
  if (wave >= Q * Q) return;
  // ---- wavefront w < Q * Q finishes quarter w: rows m0 + 16 (w / Q) .., columns n0 + 16 (w % Q) ..
  const int m = m0 + 16 * (wave / Q) + i16, n = n0 + 16 * (wave % Q) + 4 * kq;
  float c[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {   // wavefront order, whatever finished first
    const float4 t = *reinterpret_cast<const float4 *>(&red[w][wave][lane][0]);
    c[0] += t.x; c[1] += t.y; c[2] += t.z; c[3] += t.w;
  }
  // everything the epilogue reads, in one batch of clamped loads
  const bool min_ = m < a.M;
  bool ok[4];
  long o[4];
  float bv[4], rv[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    ok[v] = min_ && n + v < a.N;
    o[v] = ok[v] ? (long)m * a.c_m + (long)(n + v) * a.c_n : 0;
    bv[v] = a.bias ? a.bias[n + v < a.N ? n + v : 0] : 0.0f;
    rv[v] = a.C_ref ? a.C_ref[o[v]] : 0.0f;
  }
  float un[4] = {0.0f, 0.0f, 0.0f, 0.0f}, sq[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if constexpr (EXTRAS) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      un[v] = a.uniform ? a.uniform[o[v]] : 0.0f;
      sq[v] = a.sq_ref ? a.sq_ref[o[v]] : 0.0f;
    }
  }
  if (Q == 1 && (a.sm_labels || a.sm_prob)) {
    // Softmax (+ cross-entropy where there are labels) on the finished logits: a row's 16 columns sit in the four
    // lanes i16, i16 + 16, i16 + 32, i16 + 48 (four columns each), so two exchanges complete a row.
    // Columns past N count as -inf / 0; rows past M compute on clamped data and store nothing.
    const int label = a.sm_labels ? a.sm_labels[min(m, a.M - 1)] : -1;
    float z[4], mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      z[v] = c[v] + bv[v];
      if (n + v < a.N) mx = fmaxf(mx, z[v]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    float e[4], sum = 0.0f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      e[v] = n + v < a.N ? expf(z[v] - mx) : 0.0f;
      sum += e[v];
    }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    const float inv = 1.0f / sum;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (!ok[v]) continue;
      if (a.Cout) a.Cout[o[v]] = z[v];
      if (a.sm_prob) { a.sm_prob[o[v]] = e[v] * inv; continue; }
      a.sm_dz[o[v]] = (e[v] * inv - (n + v == label ? 1.0f : 0.0f)) * a.sm_scale;
      if (n + v == label) a.sm_rowloss[m] = -(z[v] - mx - logf(sum));
    }
    return;
  }
  float sum_sq = 0.0f;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    c[v] = act_apply(a.act, c[v] + bv[v]);
    if constexpr (EXTRAS) {
      if (ok[v] && a.sample) a.sample[o[v]] = un[v] < c[v] ? 1.0f : 0.0f;
      const float d = sq[v] - c[v];
      sum_sq += ok[v] ? d * d : 0.0f;
    }
    if (a.C_ref) c[v] *= act_deriv(a.c_ref_act, rv[v]);
    if (!ok[v]) continue;
    if (a.Cout) a.Cout[o[v]] = c[v];
  }
  if constexpr (EXTRAS) {
    if (a.sq_ref) {   // one number per finished quarter, added up later in a fixed order
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) sum_sq += __shfl_xor(sum_sq, off, 64);
      if (lane == 0) a.sq_partial[tile * (Q * Q) + wave] = sum_sq;
    }
  }
}

// The weight-gradient form: both operands contiguous across k (A along m, B along n), the contraction as
// short as a batch, many outputs.  Read with the k-wise tiles above it costs sixteen 4-byte loads per lane
// and eight MFMAs; here a lane's 16 bytes of A at one k are its rows m0 + 4 i16 + i of four MFMA
// row tiles and its 8 bytes of B columns n0 + 2 i16 + j of two column tiles (which row of the tile a lane
// stands for is free as long as the stores know it), so two loads feed eight MFMAs.  64 x 32 outputs per workgroup,
// the four wavefronts split k in batches of 16; PHASES = 2: the batches of A2 B2, taken off, follow.
// 784 x 500 over 2 x 100 rows: 15.6 -> 10.4 us, with the step's column sums beside it.  Bound by the latency of its
// two or three dependent round trips (operands, parameters, store), not by the matrix pipe.
constexpr int kOuterM = 64, kOuterN = 32;
constexpr int kOuterRedFloats = 4 * 8 * 64 * 4;
template <int PHASES>
__device__ __forceinline__ void outer_product(const SmallParams &p, int mt, int nt, float *lds) {
  typedef float floatx2 __attribute__((ext_vector_type(2)));
  constexpr int MQ = 4, NQ = 2, KB = 4;
  float (*red)[MQ * NQ][64][4] = reinterpret_cast<float (*)[MQ * NQ][64][4]>(lds);
  const GemmArgs &a = p.a;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i16 = lane & 15, kq = lane >> 4;
  const int m0 = mt * kOuterM, n0 = nt * kOuterN;
  const int nb1 = (a.Kdim + 4 * KB - 1) / (4 * KB), nb = PHASES * nb1;
  const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.A), 0, (int)p.a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.B), 0, (int)p.b_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsA2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(PHASES == 2 ? a.A2 : a.A), 0, (int)p.a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsB2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(PHASES == 2 ? a.B2 : a.B), 0, (int)p.b_bytes, 0x00020000);
  // byte offsets of the lane's columns; past the last one nothing is read.  A group that starts inside and ends
  // past the end holds the next row's first elements: they only feed outputs that are never stored.
  const unsigned colA = m0 + MQ * i16 < a.M ? 4u * (unsigned)(m0 + MQ * i16) : kOob;
  const unsigned colB = n0 + NQ * i16 < a.N ? 4u * (unsigned)(n0 + NQ * i16) : kOob;
  const unsigned skA = 4u * (unsigned)a.a_k, skB = 4u * (unsigned)a.b_k;
  floatx4 acc[MQ][NQ];
#pragma unroll
  for (int i = 0; i < MQ; ++i)
#pragma unroll
    for (int j = 0; j < NQ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  floatx4 fa[2][KB];
  floatx2 fb[2][KB];
  auto load_from = [&](const __amdgpu_buffer_rsrc_t &ra, const __amdgpu_buffer_rsrc_t &rb, int b, floatx4 (&va)[KB], floatx2 (&vb)[KB]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < KB; ++s) {
      const int k = (b * KB + s) * 4 + kq;
      const bool in = k < a.Kdim;
      va[s] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(ra, (int)(in ? colA + (unsigned)k * skA : kOob), 0, 0));
      vb[s] = __builtin_bit_cast(floatx2, __builtin_amdgcn_raw_buffer_load_b64(rb, (int)(in ? colB + (unsigned)k * skB : kOob), 0, 0));
    }
  };
  auto load = [&](int b, floatx4 (&va)[KB], floatx2 (&vb)[KB]) __attribute__((always_inline)) {
    if (PHASES == 2 && b >= nb1) load_from(rsA2, rsB2, b - nb1, va, vb);   // a batch past the last one reads zeros
    else load_from(rsA, rsB, b, va, vb);
  };
  auto multiply = [&](int b, const floatx4 (&va)[KB], const floatx2 (&vb)[KB]) __attribute__((always_inline)) {
    const float sign = PHASES == 2 && b >= nb1 ? -1.0f : 1.0f;
#pragma unroll
    for (int s = 0; s < KB; ++s)
#pragma unroll
      for (int j = 0; j < NQ; ++j) {
        const float bj = PHASES == 2 ? vb[s][j] * sign : vb[s][j];
#pragma unroll
        for (int i = 0; i < MQ; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bj, va[s][i], acc[i][j], 0, 0, 0);
      }
  };
  load(wave, fa[0], fb[0]);
  load(wave + 4, fa[1], fb[1]);
  for (int b = wave; b < nb; b += 8) {
    multiply(b, fa[0], fb[0]);
    __builtin_amdgcn_sched_barrier(0);
    load(b + 8, fa[0], fb[0]);
    __builtin_amdgcn_sched_barrier(0);
    if (b + 4 < nb) multiply(b + 4, fa[1], fb[1]);
    __builtin_amdgcn_sched_barrier(0);
    load(b + 12, fa[1], fb[1]);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int i = 0; i < MQ; ++i)
#pragma unroll
    for (int j = 0; j < NQ; ++j) *reinterpret_cast<floatx4 *>(&red[wave][i * NQ + j][lane][0]) = acc[i][j];
  __syncthreads();
  // wavefront w finishes rows m0 + 4 i16 + w: 8 neighbouring columns per lane, summed in wavefront order
  const int m = m0 + MQ * i16 + wave, n = n0 + NQ * 4 * kq;
  float c[8];
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    floatx4 t = *reinterpret_cast<const floatx4 *>(&red[0][wave * NQ + j][lane][0]);
#pragma unroll
    for (int w = 1; w < 4; ++w) t += *reinterpret_cast<const floatx4 *>(&red[w][wave * NQ + j][lane][0]);
#pragma unroll
    for (int v = 0; v < 4; ++v) c[NQ * v + j] = PHASES == 2 ? t[v] * a.alpha : t[v];
  }
  if (m >= a.M) return;
  const long o = (long)m * a.c_m + n;
  // everything the epilogue reads, in one batch: 16 bytes at a time where result rows are whole aligned
  // groups, else from clamped addresses
  float u[8] = {}, v[8] = {};
  if (p.whole) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const long oh = n + 4 * h < a.N ? o + 4 * h : 0;
      const floatx4 uq = a.update ? *reinterpret_cast<const floatx4 *>(a.update + oh) : floatx4{0.f, 0.f, 0.f, 0.f};
      const floatx4 vq = a.vel ? *reinterpret_cast<const floatx4 *>(a.vel + oh) : floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < 4; ++e) { u[4 * h + e] = uq[e]; v[4 * h + e] = vq[e]; }
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const long oe = n + e < a.N ? o + e : 0;
      u[e] = a.update ? a.update[oe] : 0.0f;
      v[e] = a.vel ? a.vel[oe] : 0.0f;
    }
  }
  if (a.vel) {
#pragma unroll
    for (int e = 0; e < 8; ++e) update_param(&u[e], &v[e], c[e], a.step, a.mu, a.decay);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) update_param(&u[e], nullptr, c[e], a.step, a.mu, a.decay);
  }
  if (p.whole) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (n + 4 * h >= a.N) continue;
      if (a.Cout) *reinterpret_cast<floatx4 *>(a.Cout + o + 4 * h) = floatx4{c[4 * h], c[4 * h + 1], c[4 * h + 2], c[4 * h + 3]};
      if (a.update) *reinterpret_cast<floatx4 *>(a.update + o + 4 * h) = floatx4{u[4 * h], u[4 * h + 1], u[4 * h + 2], u[4 * h + 3]};
      if (a.vel) *reinterpret_cast<floatx4 *>(a.vel + o + 4 * h) = floatx4{v[4 * h], v[4 * h + 1], v[4 * h + 2], v[4 * h + 3]};
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (n + e >= a.N) continue;
      if (a.Cout) a.Cout[o + e] = c[e];
      if (a.update) a.update[o + e] = u[e];
      if (a.vel) a.vel[o + e] = v[e];
    }
  }
}

// Host: the operands as the kernels see them.  False: an operand of 2 GiB or more.
inline bool make_params(const GemmArgs &a, SmallParams *p) {
  p->a = a;
  p->a.split_k = 1;
  auto al16 = [](const void *q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; };
  if (a.a_k == 1)
    p->whole = a.Kdim % 4 == 0 && al16(a.A) && a.a_m % 4 == 0 && (a.b_k != 1 || (al16(a.B) && a.b_n % 4 == 0));
  else
    p->whole = a.N % 4 == 0 && a.c_m % 4 == 0 && al16(a.Cout) && al16(a.update) && al16(a.vel);
  const long ab = 4 * ((long)(a.M - 1) * a.a_m + (long)(a.Kdim - 1) * a.a_k + 1), bb = 4 * ((long)(a.N - 1) * a.b_n + (long)(a.Kdim - 1) * a.b_k + 1);
  p->a_bytes = (unsigned)ab;
  p->b_bytes = (unsigned)bb;
  return ab < (long)kOob && bb < (long)kOob;
}
// 16 x 16 tiles while 32 x 32 ones would number at most two per CU: four times the workgroups, a
// quarter of the multiplications per wavefront (measured faster for every product of the small
// workloads, whatever its k)
inline int tile_quarters(int M, int N) { return (long)((N + 31) / 32) * ((M + 31) / 32) <= 512 ? 1 : 2; }

}  // namespace small_gemm
}  // namespace dllk
