// The prompt state S_T (Sec. 2.2, Eq. 1b): the prompt enters as a leading
// frame updated from the zero state (Sec. 4), so after the statistics and
// the inverse of that one frame per head, S_T = B_T (I + A_T)^{-1} for the
// joint rule (Eq. 5) or B_T / sqrt(L) for the frozen rule (Eq. 3c, U = L).
// This last step is one small d_v x d_k x d_k product per head, run once
// per prompt: exact fp32 products on v_mfma_f32_16x16x4_f32, one workgroup
// per head and 16 rows of S, its waves sharing the column slices.  Latency
// bounds it (one round trip for all operands, 32 products in a chain per
// slice): 4 us for 16 heads of 128 x 128, 32 us as one dependent
// multiply-add loop per element.  From 2^16 row blocks on a workgroup takes
// several in turn: one each would pass the 2^32 threads of a launch at 2^21
// heads of 128 value channels, which the other steps still take.
#include "vda_common.h"
#include "vda_launch.h"

namespace vda {
namespace {

// S[h] = B[h] Inv[h], the first d_v rows and d_k columns.  B is [H][pv][PK]
// and Inv [H][PK][PK], symmetric (PK >= d_k, pv >= d_v: zero-padded heads);
// S is [H][d_v][d_k].  nblocks: H * pv / 16 row blocks.
constexpr unsigned kTextStateGrid = 1u << 16;

template <int PK>
__global__ __launch_bounds__(kThreads)
void text_state_kernel(const float* __restrict__ B, const float* __restrict__ Inv, int pv, int d_k,
                       int d_v, unsigned nblocks, float* __restrict__ S) {
  constexpr int NB = PK / 16, KC = PK / 16;
  constexpr int NBW = (NB + 3) / 4;  // column slices per wave
  const unsigned nrb = (unsigned)pv / 16;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lg = lane >> 4;
  if (wave >= NB) return;
  for (unsigned i = blockIdx.x; i < nblocks; i += gridDim.x) {
    const int rb = (int)(i % nrb);
    const size_t h = i / nrb;
    // Lane group lg supplies k = 16 c + 4 lg + s of chunk c: row li of B's block,
    // and of Inv's slice its row by symmetry, both 16 bytes at a time.
    const float* b = B + (h * pv + rb * 16 + li) * PK + 4 * lg;
    const float* m = Inv + (h * PK + wave * 16 + li) * PK + 4 * lg;
    floatx4 bv[KC], mv[NBW][KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      bv[c] = *reinterpret_cast<const floatx4*>(b + 16 * c);
#pragma unroll
      for (int q = 0; q < NBW; ++q)
        mv[q][c] = *reinterpret_cast<const floatx4*>(m + (size_t)q * 64 * PK + 16 * c);
    }
    floatx4 acc[NBW];
#pragma unroll
    for (int q = 0; q < NBW; ++q) acc[q] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int q = 0; q < NBW; ++q)
          acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[c][s], mv[q][c][s], acc[q], 0, 0, 0);
#pragma unroll
    for (int q = 0; q < NBW; ++q) {
      const int col = (wave + 4 * q) * 16 + li;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = rb * 16 + 4 * lg + e;
        if (row < d_v && col < d_k) S[(h * d_v + row) * d_k + col] = acc[q][e];
      }
    }
  }
}

// The frozen rule: S[h][r][c] = B[h][r][c] * scale.
__global__ __launch_bounds__(kThreads)
void text_scale_kernel(const float* __restrict__ B, int H, int pk, int pv, int d_k, int d_v,
                       float scale, float* __restrict__ S) {
  const long long total = (long long)H * d_v * d_k;
  for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < total;
       i += (long long)gridDim.x * kThreads) {
    const int c = (int)(i % d_k);
    const long long hr = i / d_k;
    S[i] = B[((size_t)(hr / d_v) * pv + hr % d_v) * pk + c] * scale;
  }
}

}  // namespace

hipError_t launch_text_state(const float* B, const float* Inv, int H, int pk, int pv, int d_k,
                             int d_v, float scale, float* S, hipStream_t stream) {
  if (Inv != nullptr) {
    const unsigned nblocks = (unsigned)H * (unsigned)(pv / 16);
    const dim3 grid(nblocks < kTextStateGrid ? nblocks : kTextStateGrid);
#define VDA_TEXT_STATE(PK)                                                                      \
  hipLaunchKernelGGL(text_state_kernel<PK>, grid, dim3(kThreads), 0, stream, B, Inv, pv, d_k, d_v, \
                     nblocks, S)
    switch (pk) {
      case 32: VDA_TEXT_STATE(32); break;
      case 64: VDA_TEXT_STATE(64); break;
      case 128: VDA_TEXT_STATE(128); break;
      default: return hipErrorInvalidValue;
    }
#undef VDA_TEXT_STATE
    return hipGetLastError();
  }
  long long g = ((long long)H * d_v * d_k + kThreads - 1) / kThreads;
  if (g > 8192) g = 8192;
  hipLaunchKernelGGL(text_scale_kernel, dim3((unsigned)g), dim3(kThreads), 0, stream, B, H, pk, pv,
                     d_k, d_v, scale, S);
  return hipGetLastError();
}

}  // namespace vda
