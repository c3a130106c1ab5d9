// Step a2 as a stand-alone kernel: Inv_t = (I + A_t)^{-1} for every frame
// of every head (Eq. 5), one workgroup per matrix.  The algorithm is
// described in vda_inverse_body.h.  The result is written by rows, or as the
// operand tiles of the bf16 or the fp32 state scan (InvLayout).
#include "vda_common.h"
#include "vda_inverse_body.h"
#include "vda_launch.h"

namespace vda {
namespace {

// Three waves per SIMD, so that three matrices of d_k = 128 share a compute
// unit (576 frames are one round of 256 compute units; at two, 186 registers,
// they took 53 us instead of 36).
// (OUT: an InvLayout.)
template <int DK, int OUT>
__global__ __launch_bounds__(inv::inverse_threads(DK)) __attribute__((amdgpu_waves_per_eu(3)))
void inverse_kernel(const float* A_part, unsigned first_split, int plan_splits, unsigned extra,
                    size_t part_stride,
                    float* Inv,  // may alias A_part (in place)
                    float* B_part, size_t b_mat, size_t b_stride) {
  constexpr int kT = inv::inverse_threads(DK);
  __shared__ __align__(16) float lds[inv::inverse_lds_floats(DK)];

  const int tid = threadIdx.x;
  if (blockIdx.x >= gridDim.x - extra) {
    // One of the workgroups past the matrices: fold the token-range partials
    // of B_t of split frame first_split + (its index) / 4, quarter (its
    // index) % 4 of the matrix, into the first partial (in place), alongside
    // the inversions.
    const unsigned e = blockIdx.x - (gridDim.x - extra);
    const size_t f = first_split + e / 4;
    const size_t quarter = b_mat / 4;
    inv::fold_b_partials(B_part + f * b_mat, plan_splits, (e % 4) * quarter,
                         (e % 4 + 1) * quarter, b_stride, tid, kT);
    return;
  }
  const size_t base = (size_t)blockIdx.x * (DK * DK);
  // Frames from first_split on were split into plan_splits token ranges.
  const int splits = blockIdx.x >= first_split ? plan_splits : 1;
  inv::invert_matrix<DK, static_cast<InvLayout>(OUT)>(A_part, splits, part_stride, base, Inv, lds, tid);
}

}  // namespace

hipError_t launch_frame_inverse(const float* A_part, float* B_part, SplitPlan plan,
                                long long count, int d_k, int d_v, InvLayout out, float* Inv,
                                hipStream_t stream) {
  const int splits = plan.splits > 1 && plan.tail > 0 ? plan.splits : 1;
  const unsigned first_split = splits > 1 ? (unsigned)(count - plan.tail) : (unsigned)count;
  // Partial p of frame f is matrix f + p * tail.
  const size_t part_stride = (size_t)plan.tail * d_k * d_k;
  const size_t b_mat = (size_t)d_v * d_k;
  const size_t b_stride = (size_t)plan.tail * b_mat;
  // One workgroup per matrix, then four per split frame to fold its B
  // partials (a quarter of the matrix each, one memory round trip).
  const unsigned extra = splits > 1 ? 4u * (unsigned)plan.tail : 0u;
  const dim3 grid((unsigned)count + extra);
#define VDA_INVERSE(DK, OUT)                                                                 \
  hipLaunchKernelGGL((inverse_kernel<DK, (int)InvLayout::OUT>), grid,                        \
                     dim3(inv::inverse_threads(DK)), 0, stream, A_part, first_split, splits, \
                     extra, part_stride, Inv, B_part, b_mat, b_stride)
#define VDA_INVERSE_DK(DK)                                                  \
  if (out == InvLayout::kBf16Tiles)                                         \
    VDA_INVERSE(DK, kBf16Tiles);                                            \
  else if (out == InvLayout::kF32Tiles)                                     \
    VDA_INVERSE(DK, kF32Tiles);                                             \
  else                                                                      \
    VDA_INVERSE(DK, kRows);
  switch (d_k) {
    case 32: VDA_INVERSE_DK(32) break;
    case 64: VDA_INVERSE_DK(64) break;
    case 128: VDA_INVERSE_DK(128) break;
    default: return hipErrorInvalidValue;
  }
#undef VDA_INVERSE_DK
#undef VDA_INVERSE
  return hipGetLastError();
}

}  // namespace vda
