// fp32 MFMA matrix product for SMALL problems: the dense layers of the paper's MNIST and CIFAR
// networks and of the fully-connected RBM (Sections II-A, IV, V: a few hundred units, batch 100).
//
// Such a product cannot fill the chip; what it costs is a chain of latencies (launch, first
// loads, one LDS round trip and one barrier per k-tile, a split-K reduction launch).  This kernel
// shortens the chain instead of raising the rate:
//   * 32 x 32 or, for the smallest products, 16 x 16 output tile per workgroup (many more workgroups
//     than the 128 x 64 tiles of the big kernel, far fewer products with padding);
//   * the four wavefronts split the k range BETWEEN them and each multiplies the whole tile, so
//     there is no LDS staging and no barrier inside the k loop at all: every lane loads its
//     MFMA fragments straight from global memory, the next three k-tiles' loads in flight while
//     the current one is multiplied.  Inside a k-tile of 32, the lane with k-quarter kq owns the 8
//     consecutive k values 8*kq .. 8*kq+7 of both operands (any assignment works as long as both
//     operands use the same one), which makes a k-contiguous operand two 16-byte loads per row;
//   * the partial tiles meet in LDS once, are added in wavefront order (results do not depend
//     on timing), and one wavefront per 16 x 16 quarter of the tile finishes it: bias, activation,
//     act' of a reference tensor, store.  No split-K partials in global memory, no reduction launch.
// Every global load is a range-checked buffer load: what lies past an operand's end reads as zero, so nothing
// is masked but the rows that are no whole 16-byte groups, and that at the multiplication.
#include "dll_internal.h"
#include "gemm_small_body.h"

namespace dllk {
namespace {

using small_gemm::SmallParams;

template <bool B_KC, bool WHOLE, int WAVES, int Q, bool EXTRAS>
__global__ __launch_bounds__(WAVES * 64) void gemm_small_kernel(const SmallParams p) {
  __shared__ __attribute__((aligned(16))) float red[small_gemm::kRedFloats<WAVES, Q>];
  small_gemm::tile_product<B_KC, WHOLE, WAVES, Q, EXTRAS>(p, blockIdx.y, blockIdx.x, blockIdx.y * gridDim.x + blockIdx.x, red);
}

}  // namespace

// Where a product runs here rather than on the persistent kernel (128 x 64 tiles, split-K partials and a
// reduction launch for products of few tiles).  Up to 1.5 x 2^27 multiply-adds in any case (129 x 1024 x
// 1024 RBM step: 87 us there, 55 here; but the 128 x 1000 x 2048 logits: 15 + 7 us with the loss behind
// them there, 27 here).  Up to 2^28 where the shortest extent leaves the persistent kernel's tiles half
// empty (large-image step at batch 16: 274 against 259 us).  Up to 2^29 where all three are at least 256, i.e.
// where several rows of its tiles re-read operands (512 x 1000 x 1000 RBM step 184 against 117; but with the
// 128 x 2048 x 2000 products of a large-image step 370 against 379 in all).  Up to 2^30 where rows of the operands
// or the result are no multiples of four, which the persistent kernel's 16-byte accesses need (500 x 1600 x 1001 RBM step 267
// against 192).  Where only the batch is none and the product is a gradient, as far from 128 on (RBM steps of
// 903 x 2148 x 136 242 against 102, 867 x 1036 x 680 265 against 132) and up to 2^29 below (127 x 3012 x 2392 184
// against 240); a forward product does not mind its batch (255 x 1912 x 1696: 47 there against 64 here).
// And only while every operand and result lies below 2 GiB, where the kernel's buffers end (one row through a
// weight matrix of 2^29 floats is not many multiply-adds), and no extent is past 2^26, so that the jobs of a closing
// launch, column sums of 16 columns a workgroup among them, fit a grid.
bool gemm_is_small(GemmForm form, int M, int N, int Kdim) {
  const long macs = (long)M * N * Kdim, limit = 1L << 29;
  if ((long)M * N >= limit || (long)M * Kdim >= limit || (long)N * Kdim >= limit) return false;
  if (M > (1 << 26) || N > (1 << 26) || Kdim > (1 << 26)) return false;
  const int rows = (form == GemmForm::kWeightGrad ? M : Kdim) | N;
  if ((rows & 3) != 0) return macs <= (1L << 30);
  const int batch = form == GemmForm::kDataGrad ? M : (form == GemmForm::kWeightGrad ? Kdim : 0);
  const int least = M < N ? (M < Kdim ? M : Kdim) : (N < Kdim ? N : Kdim);
  if ((batch & 3) != 0) return macs <= (least >= 128 ? 1L << 30 : 1L << 29);
  if (least >= 256) return macs <= (1L << 29);
  return macs <= (least <= 64 ? 1L << 28 : 3L << 26);
}

bool gemm_prefers_small(const GemmArgs &a) {
  if (gemm_is_small(a.b_k == 1 ? GemmForm::kForward : GemmForm::kDataGrad, a.M, a.N, a.Kdim)) return true;
  return a.a_k == 1 && a.b_n == 1 && !a.update && !a.sm_labels && (long)a.M * a.N * a.Kdim <= (1L << 28);
}

// Tiles of 16 x 16 (the launcher's choice below for this size) hold whole rows of up to 16 logits.
bool gemm_fuses_softmax(int M, int N, int Kdim) { return gemm_is_small(GemmForm::kForward, M, N, Kdim) && N <= 16 && (M + 31) / 32 <= 512; }

hipError_t launch_gemm_small(const GemmArgs &a, hipStream_t stream) {
  if (a.sm_prob && (a.sm_labels || !gemm_fuses_softmax(a.M, a.N, a.Kdim) || a.act != ACT_IDENTITY || a.C_ref)) return hipErrorInvalidValue;
  if (a.sm_labels && (!gemm_fuses_softmax(a.M, a.N, a.Kdim) || !a.sm_dz || !a.sm_rowloss || a.act != ACT_IDENTITY || a.C_ref))
    return hipErrorInvalidValue;
  SmallParams p;
  // A across k, updates: the weight-gradient form, a job of the closing launch
  if (a.a_k != 1 || a.update || a.A2 || a.B2 || !small_gemm::make_params(a, &p)) return hipErrorInvalidValue;
  const bool b_kc = a.b_k == 1;
  const bool fine = small_gemm::tile_quarters(a.M, a.N) == 1;
  const int TS = fine ? 16 : 32;
  const dim3 grid((a.N + TS - 1) / TS, (a.M + TS - 1) / TS);
  // (eight wavefronts per workgroup, sharing the k range in eighths, measured slower at every size tried)
  auto launch = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, stream, p);
    return hipGetLastError();
  };
#define DLL_SMALL(BK_, WH, EX) (fine ? launch(gemm_small_kernel<BK_, WH, 4, 1, EX>) : launch(gemm_small_kernel<BK_, WH, 4, 2, EX>))
#define DLL_SMALL_B(WH, EX) (b_kc ? DLL_SMALL(true, WH, EX) : DLL_SMALL(false, WH, EX))
  if (a.uniform || a.sq_ref) {
    if (a.sm_labels || a.sm_prob || (a.uniform && !a.sample) || (a.sq_ref && !a.sq_partial)) return hipErrorInvalidValue;
    return p.whole ? DLL_SMALL_B(true, true) : DLL_SMALL_B(false, true);
  }
  return p.whole ? DLL_SMALL_B(true, false) : DLL_SMALL_B(false, false);
#undef DLL_SMALL_B
#undef DLL_SMALL
}

size_t gemm_small_tiles(int M, int N) {
  const int q = small_gemm::tile_quarters(M, N), TS = 16 * q;
  return (size_t)((N + TS - 1) / TS) * ((M + TS - 1) / TS) * q * q;
}

}  // namespace dllk
