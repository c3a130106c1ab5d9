// Steps a5-a7: gather, readout, RMSNorm and gate.
//   S~_t = P_{t-1} + R_{t+1}            (Eq. A.4 with the window [t, t], alpha = 1)
//   o_{t,u} = S~_t q_{t,u}               (Eq. 1a)
//   y_{t,u} = G * o / sqrt(mean(o^2) + eps)      (Eq. 1c)
// G is the per-head gate, or (TOKGATE) the output gate G^L per token and
// channel, read beside the queries.
//
// bf16 path: a workgroup owns one frame of one head and every `chunks`-th
// 64-token super-group of it (the frame's workgroups sweep it together).
// It sums the two fp32 states, rounds S~ to bf16 once into LDS, and
// each wavefront keeps all of S~ as MFMA A-operands in registers.  It then
// streams 16-token groups: the group's queries are the B-operand (16-byte
// loads straight from HBM, two groups in flight per wave), O^T = S~ Q^T is
// accumulated in fp32 by v_mfma_f32_16x16x32_bf16, and the RMSNorm over the
// d_v outputs of a token is a lane-local sum plus two cross-lane exchanges.
// The normalised, gated values are rounded to bf16 into a per-wave LDS tile
// of the group's 16 token rows, from which each 16-byte-per-lane streaming
// store writes consecutive whole token rows (one contiguous run of up to
// 1 KB when the output is frame-major per head; with the token-major output
// of the epilogue's layout conversion, a head's rows sit out_heads * d_v
// apart and each is one run of d_v values).
#include "vda_common.h"
#include "vda_launch.h"

namespace vda {
namespace {

// Local window [lo, hi] of frame f (0-based, clipped to [0, F)): the frame's
// chunk of `chunk` frames (counted from `offset` positions before frame 0)
// and `radius` chunks on each side (Eq. A.4's [l_t, h_t]).
struct Window {
  int lo, hi;
};

__device__ __forceinline__ Window local_window(int f, int F, int chunk, int radius, int offset) {
  const int c = (f + offset) / chunk;
  const int lo = (c - radius) * chunk - offset;
  const int hi = (c + radius + 1) * chunk - offset - 1;
  return Window{max(0, lo), min(F - 1, hi)};
}

// Decay bridge factors of Eq. A.4 for key channels j .. j + W - 1 of head h:
// df = prod_{r = lo..f} alpha_r, dr = prod_{r = f..hi} alpha_r.
template <int W>
__device__ __forceinline__ void bridge_decay(const float* alpha, int h, int F, int DKr, int j,
                                             int f, Window w, float (&df)[W], float (&dr)[W]) {
#pragma unroll
  for (int c = 0; c < W; ++c) df[c] = dr[c] = 1.0f;
  if (alpha == nullptr) return;
  const float* a = alpha + (size_t)h * F * DKr + j;
  for (int r = w.lo; r <= w.hi; ++r) {
#pragma unroll
    for (int c = 0; c < W; ++c) {
      const float x = a[(size_t)r * DKr + c];
      if (r <= f) df[c] *= x;
      if (r >= f) dr[c] *= x;
    }
  }
}

// GENOUT: the general layouts (the token-major output, a padded narrow
// head: row stride and stored channels at run time; a token-major raw query,
// qh heads per clip, L2-normalised here when ql2); otherwise frame-major rows
// of DK and DV channels.
template <int DK, int DV, bool TOKGATE, bool GENOUT>
__global__ __launch_bounds__(kThreads, 2)
void readout_bf16_kernel(const uint16_t* __restrict__ Q, const float* __restrict__ S_fwd,
                         const float* __restrict__ S_rev, const float* __restrict__ gate,
                         int F, int N, int chunks, unsigned nwg,
                         int dvo, int oh, int qh, int ql2, const float* __restrict__ alpha,
                         int wchunk, int wradius, int woffset, const uint16_t* __restrict__ gtok,
                         uint16_t* __restrict__ out) {
  constexpr int SLD = DK + 8;  // bf16 row stride of S~ in LDS
  constexpr int MB = DV / 16;  // 16-row blocks of S~ (output channels)
  constexpr int KB = DK / 32;  // 32-wide k steps
  constexpr int OLD = DV + 8;  // bf16 row stride of the output staging tiles
  __shared__ __align__(16) uint16_t st[DV * SLD];
  // One 16-token output tile per wave: bf16, or with an output gate per token
  // fp32, so that the gate is applied where whole rows are stored and its own
  // rows are read in the stores' layout.
  constexpr int GLD = DV + 4;  // fp32 row stride
  __shared__ __align__(16) uint16_t otile[TOKGATE ? 4 * 16 * GLD * 2 : 4 * 16 * OLD];

  // The chunks of one frame read the same two states: keep them on one XCD.
  const unsigned L = xcd_grouped_id(blockIdx.x, nwg);
  const unsigned fh = L / chunks;
  const int chunk = L % chunks;
  const float g = TOKGATE ? 1.0f : gate[fh / F];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform (scalar)
  const int li = lane & 15;
  const int lg = lane >> 4;

  {
    // Gather (Eq. A.4): the forward state entering the frame's local window
    // and the reverse state leaving it, each decayed across the skipped
    // frames (the own frame only, with alpha = 1, in the core operator).
    const int h = (int)(fh / F), f = (int)(fh % F);
    const Window w = local_window(f, F, wchunk, wradius, woffset);
    const float* sf = S_fwd + ((size_t)h * F + w.lo) * (DV * DK);
    const float* sr = S_rev + ((size_t)h * F + w.hi) * (DV * DK);
    // This thread's columns are the same in every iteration below.
    static_assert((kThreads * 4) % DK == 0, "fixed columns per thread");
    float df[4], dr[4];
    bridge_decay<4>(alpha, h, F, DK, (tid * 4) % DK, f, w, df, dr);
    // Fully unrolled (a compile-time trip count; DV * DK is a multiple of
    // kThreads * 4), so all of a thread's loads are in flight together.
    static_assert((DV * DK) % (kThreads * 4) == 0, "state size");
#pragma unroll
    for (int it = 0; it < (DV * DK) / (kThreads * 4); ++it) {
      const int idx = tid * 4 + it * (kThreads * 4);
      const float4 a = *reinterpret_cast<const float4*>(sf + idx);
      const float4 b = *reinterpret_cast<const float4*>(sr + idx);
      const int i = idx / DK, j = idx % DK;
      *reinterpret_cast<uint2*>(&st[i * SLD + j]) =
          make_uint2(pack_bf16x2(a.x * df[0] + b.x * dr[0], a.y * df[1] + b.y * dr[1]),
                     pack_bf16x2(a.z * df[2] + b.z * dr[2], a.w * df[3] + b.w * dr[3]));
    }
  }
  lds_barrier();

  // S~ as MFMA A-operands: held in registers on the plain frame-major path;
  // the gated and general-layout variants read them from LDS at each group
  // instead, which leaves them the registers for two query groups in flight.
  constexpr bool kSopRegs = !GENOUT && !TOKGATE;
  bf16x8 sop[kSopRegs ? MB : 1][kSopRegs ? KB : 1];
  if constexpr (kSopRegs) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
        sop[mb][kb] = *reinterpret_cast<const bf16x8*>(&st[(mb * 16 + li) * SLD + kb * 32 + lg * 8]);
  }
  const uint16_t* sop_lds = &st[li * SLD + lg * 8];

  // This frame's query rows: DK channels at row stride qh * DK, from head
  // h % qh of clip h / qh (frame-major per head when qh = 1).
  const unsigned qhu = GENOUT ? (unsigned)qh : 1u, hp = fh / F, fr = fh % F;
  const uint32_t qrs = qhu * (uint32_t)DK;
  const uint16_t* qbase = Q + (((size_t)(hp / qhu) * F + fr) * N * qhu + hp % qhu) * DK;
  // This frame's output rows: dvo channels at row stride oh * dvo, likewise.
  const unsigned ohu = GENOUT ? (unsigned)oh : 1u;
  const int dvw = GENOUT ? dvo : DV;
  const uint32_t ors = ohu * (uint32_t)dvw;
  uint16_t* obase = out + (((size_t)(hp / ohu) * F + fr) * N * ohu + hp % ohu) * dvw;
  const float inv_norm = 1.0f / (float)dvw;

  // The frame's tokens go in 64-token super-groups, dealt out to its
  // `chunks` workgroups in turn (super-group c, c + chunks, ...), so the
  // workgroups of one frame sweep it together and the device streams a
  // compact address window; within a super-group wave w takes the 16-token
  // group at 16 w.  The queries of a wave's next kQ groups are in flight in
  // a register ring (slot d: group n0 + S*d, S = 64 * chunks tokens apart).
  // Rows past the frame are clamped onto its last row (always valid
  // memory); their outputs are dropped by the range-checked stores, so
  // loads and stores need no branches.
  constexpr int kQ = 2;
  const int S = 64 * chunks;
  uint4 qr[kQ][KB];
  auto load_q = [&](int nq, uint4 (&qv)[KB]) {
    const int row = min(nq + li, N - 1);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
      qv[kb] = *reinterpret_cast<const uint4*>(qbase + (size_t)row * qrs + kb * 32 + lg * 8);
  };
  // TOKGATE: the output gate of the same groups, whole rows of the true dvw
  // channels in the stores' layout (rows past the frame and a padded head's
  // channels read as zero); read once, so streamed (nt), whatever its size: a
  // gate still in the cache costs a little more so, one from memory less (us a
  // pass, default -> nt, same buffers again / after a 400 MB fill: 8 MB of
  // gates, 4 heads x 21 x 1560 x 32, 33.3 -> 34.4 and 43.8 -> 42.4; 34 MB, 8 x
  // 16 x 1024 x 128, 82 -> 83 and 105 -> 98; 75 MB, 16 x 36 x 512 x 128, 101 ->
  // 105 and 136 -> 121; 201 MB, 24 x 21 x 1560 x 128, 274 -> 268 and 318 ->
  // 304).  (From a copy padded to 32 channels, as the other inputs of
  // 16-channel heads are, those heads took 100 us a pass at 12 heads x 40
  // frames x 1000 tokens, 81 so.)
  constexpr int CPR = DV / 8;     // 16-byte chunks per token row
  constexpr int RPI = 64 / CPR;   // token rows per store instruction
  const __amdgpu_buffer_rsrc_t grsrc =
      make_rsrc(TOKGATE ? gtok + (size_t)fh * N * dvw : Q, TOKGATE ? (uint32_t)N * dvw * 2u : 0u);
  u32x4 gr[TOKGATE ? kQ : 1][TOKGATE ? 16 / RPI : 1];
  auto load_gate = [&](int ng, u32x4 (&gv)[TOKGATE ? 16 / RPI : 1]) {
    if constexpr (TOKGATE) {
#pragma unroll
      for (int r = 0; r < 16 / RPI; ++r) {
        const uint32_t off = ((uint32_t)(ng + r * RPI + lane / CPR) * dvw + lane % CPR * 8) * 2u;
        gv[r] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                       grsrc, (int)(!GENOUT || lane % CPR * 8 < dvw ? off : kOutOfRange), 0, 2));
      }
    }
  };
  const __amdgpu_buffer_rsrc_t orsrc =
      make_rsrc(obase, ((uint32_t)(N - 1) * ors + (uint32_t)dvw) * 2u);

  const int n_first = chunk * 64 + wave * 16;
  if (n_first >= N) return;
  // Issue the ring in slot order (the scheduler must not reorder it), so on
  // loop entry slot 0 is the oldest load and waits stay partial.
#pragma unroll
  for (int d = 0; d < kQ; ++d) {
    load_q(n_first + S * d, qr[d]);
    if constexpr (TOKGATE) load_gate(n_first + S * d, gr[d]);
    __builtin_amdgcn_sched_barrier(0);
  }
  for (int n0 = n_first; n0 < N; n0 += S * kQ) {
#pragma unroll
    for (int d = 0; d < kQ; ++d) {
      // Groups past the frame (at most kQ-1 per wave) run on clamped rows;
      // their stores fall outside the buffer range and are dropped.
      const int ng = n0 + S * d;
      floatx4 acc[MB];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) acc[mb] = floatx4{0.f, 0.f, 0.f, 0.f};
      // (An opaque zero offset keeps the compiler from hoisting the LDS
      // operand reads out of the loop into registers.)
      int zero_off = 0;
      if constexpr (!kSopRegs) asm volatile("v_mov_b32 %0, 0" : "=v"(zero_off));
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const bf16x8 qop = __builtin_bit_cast(bf16x8, qr[d][kb]);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          bf16x8 aop;
          if constexpr (kSopRegs)
            aop = sop[mb][kb];
          else
            aop = *reinterpret_cast<const bf16x8*>(sop_lds + zero_off + mb * 16 * SLD + kb * 32);
          acc[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, qop, acc[mb], 0, 0, 0);
        }
      }
      // A raw query: |q|^2 of the lane's token from the operand registers
      // (the token's DK channels are spread over lanes li + 16 lg), so that
      // the L2-normalised query's output is this one divided by
      // sqrt(|q|^2 + eps), which the RMSNorm below takes in.
      float qn2 = 1.0f;
      if constexpr (GENOUT) {
        if (ql2) {
          float s = 0.f;
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) {
            const uint32_t w4[4] = {qr[d][kb].x, qr[d][kb].y, qr[d][kb].z, qr[d][kb].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              s = fmaf(bf16_lo(w4[e]), bf16_lo(w4[e]), s);
              s = fmaf(bf16_hi(w4[e]), bf16_hi(w4[e]), s);
            }
          }
          s += __shfl_xor(s, 16);
          s += __shfl_xor(s, 32);
          qn2 = s + kL2Eps;
        }
      }
      load_q(ng + S * kQ, qr[d]);
      // lane holds o[token ng + li][mb*16 + 4*lg + i]
      float ss = 0.f;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i) ss = fmaf(acc[mb][i], acc[mb][i], ss);
      ss += __shfl_xor(ss, 16);
      ss += __shfl_xor(ss, 32);
      // With q / n (n^2 = qn2) in place of q: g (o / n) / sqrt(mean((o / n)^2)
      // + eps) = g o / sqrt(mean(o^2) + eps n^2).
      const float scale = g / sqrtf(ss * inv_norm + kRmsEps * qn2);
      // Stores of whole token rows: the group's outputs (16 tokens x DV,
      // bf16) go through this wave's LDS tile, then each store instruction
      // writes 64 / (DV / 8) consecutive token rows, one contiguous run of
      // up to 1 KB.
      if constexpr (TOKGATE) {
        float* tile = reinterpret_cast<float*>(otile) + wave * (16 * GLD);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          *reinterpret_cast<floatx4*>(&tile[li * GLD + mb * 16 + 4 * lg]) = acc[mb] * scale;
#pragma unroll
        for (int r = 0; r < 16 / RPI; ++r) {
          const int tok = r * RPI + lane / CPR, ch = lane % CPR;
          const floatx4 y0 = *reinterpret_cast<const floatx4*>(&tile[tok * GLD + ch * 8]);
          const floatx4 y1 = *reinterpret_cast<const floatx4*>(&tile[tok * GLD + ch * 8 + 4]);
          const u32x4 gw = gr[d][r];
          const u32x4 v = {pack_bf16x2(y0[0] * bf16_lo(gw[0]), y0[1] * bf16_hi(gw[0])),
                           pack_bf16x2(y0[2] * bf16_lo(gw[1]), y0[3] * bf16_hi(gw[1])),
                           pack_bf16x2(y1[0] * bf16_lo(gw[2]), y1[1] * bf16_hi(gw[2])),
                           pack_bf16x2(y1[2] * bf16_lo(gw[3]), y1[3] * bf16_hi(gw[3]))};
          store_b128_stream(orsrc, !GENOUT || ch * 8 < dvw ? ((uint32_t)(ng + tok) * ors + ch * 8) * 2u
                                                          : kOutOfRange, v);
        }
        load_gate(ng + S * kQ, gr[d]);
      } else {
        uint16_t* tile = otile + wave * (16 * OLD);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          *reinterpret_cast<uint2*>(&tile[li * OLD + mb * 16 + 4 * lg]) =
              make_uint2(pack_bf16x2(acc[mb][0] * scale, acc[mb][1] * scale),
                         pack_bf16x2(acc[mb][2] * scale, acc[mb][3] * scale));
#pragma unroll
        for (int r0 = 0; r0 < 16; r0 += RPI) {
          const int tok = r0 + lane / CPR, ch = lane % CPR;
          const u32x4 v = *reinterpret_cast<const u32x4*>(&tile[tok * OLD + ch * 8]);
          // Channels past dvo (zero padding of a narrow head) are not stored.
          store_b128_stream(orsrc, !GENOUT || ch * 8 < dvw ? ((uint32_t)(ng + tok) * ors + ch * 8) * 2u
                                                          : kOutOfRange, v);
        }
      }
    }
  }
}

// fp32 storage: exact fp32 products (v_mfma_f32_16x16x4_f32) and sums, laid
// out as the bf16 path: O^T = S~ Q^T with S~ as the A-operand and the
// queries of one 16-token group per wave as the B-operand.  Lane group lg of
// k chunk c supplies the channels 16 c + 4 lg + s (s = 0..3, one product
// each), so both operands are 16-byte pieces: the queries straight from
// memory (one step's loads in flight during the previous one's products),
// S~ from its fp32 image in LDS (row stride DK + 4 floats: the 16 rows of
// a lane group start on different banks).
// What bounds it: the fp32 matrix rate (2 d_k d_v flop per token, 32 cycles
// per product); the LDS reads of S~ take a quarter of the LDS rate meanwhile.
// 57 us at 4 heads x 21 frames x 1560 tokens x 128 channels (33 us of
// products on the busiest compute unit; 344 us on the vector ALUs with an LDS
// read per multiply-add); two 16-token groups per wave and step 71 us (a
// coarser split of the frames).
template <int DK, int DV, bool TOKGATE>
__global__ __launch_bounds__(kThreads, 2)
void readout_f32_kernel(const float* __restrict__ Q, const float* __restrict__ S_fwd,
                        const float* __restrict__ S_rev, const float* __restrict__ gate,
                        int F, int N, int chunks, unsigned nwg, int dvo, int oh, int qh,
                        int ql2, const float* __restrict__ alpha, int wchunk, int wradius,
                        int woffset, const float* __restrict__ gtok, float* __restrict__ out) {
  constexpr int SLD = DK + 4;  // fp32 row stride of S~ in LDS
  constexpr int MB = DV / 16;  // 16-row blocks of S~ (output channels)
  constexpr int KC = DK / 16;  // 16-channel k chunks
  __shared__ __align__(16) float st[DV * SLD];

  // The workgroups of one frame read the same two states: keep them on one XCD.
  const unsigned L = xcd_grouped_id(blockIdx.x, nwg);
  const unsigned fh = L / (unsigned)chunks;
  const int chunk = (int)(L % (unsigned)chunks);
  const float g = TOKGATE ? 1.0f : gate[fh / F];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform (scalar)
  const int li = lane & 15;
  const int lg = lane >> 4;
  const float inv_norm = 1.0f / (float)dvo;
  // Query and output rows as in readout_bf16_kernel.
  const unsigned hp = fh / F, fr = fh % F;
  const uint32_t qrs = (uint32_t)qh * DK;
  const float* qbase = Q + (((size_t)(hp / (unsigned)qh) * F + fr) * N * qh + hp % (unsigned)qh) * DK;
  const uint32_t ors = (uint32_t)oh * (uint32_t)dvo;
  float* obase = out + (((size_t)(hp / (unsigned)oh) * F + fr) * N * oh + hp % (unsigned)oh) * dvo;

  // The frame's 64-token super-groups are dealt out to its workgroups in
  // turn, as in readout_bf16_kernel; rows past the frame are clamped onto its
  // last row, and their outputs dropped by the range-checked stores.
  const int n_first = chunk * 64 + wave * 16;
  const int S = 64 * chunks;
  floatx4 qn[KC];
  auto load_q = [&](int n0) {
    const int row = min(n0 + li, N - 1);
#pragma unroll
    for (int c = 0; c < KC; ++c)
      qn[c] = *reinterpret_cast<const floatx4*>(qbase + (size_t)row * qrs + 16 * c + 4 * lg);
  };
  load_q(n_first);

  {
    // Gather (Eq. A.4), as in readout_bf16_kernel.
    const int h = (int)hp, f = (int)fr;
    const Window w = local_window(f, F, wchunk, wradius, woffset);
    const float* sf = S_fwd + ((size_t)h * F + w.lo) * (DV * DK);
    const float* sr = S_rev + ((size_t)h * F + w.hi) * (DV * DK);
    float df[4], dr[4];
    bridge_decay<4>(alpha, h, F, DK, (tid * 4) % DK, f, w, df, dr);
#pragma unroll
    for (int it = 0; it < (DV * DK) / (kThreads * 4); ++it) {
      const int idx = tid * 4 + it * (kThreads * 4);
      const float4 a = *reinterpret_cast<const float4*>(sf + idx);
      const float4 b = *reinterpret_cast<const float4*>(sr + idx);
      reinterpret_cast<floatx4*>(st)[((idx / DK) * SLD + idx % DK) / 4] =
          floatx4{a.x * df[0] + b.x * dr[0], a.y * df[1] + b.y * dr[1], a.z * df[2] + b.z * dr[2],
                  a.w * df[3] + b.w * dr[3]};
    }
  }
  lds_barrier();

  const __amdgpu_buffer_rsrc_t grsrc =
      make_rsrc(TOKGATE ? gtok + (size_t)fh * N * dvo : Q, TOKGATE ? (uint32_t)N * dvo * 4u : 0u);
  const __amdgpu_buffer_rsrc_t orsrc =
      make_rsrc(obase, ((uint32_t)(N - 1) * ors + (uint32_t)dvo) * 4u);
  const floatx4* st4 = reinterpret_cast<const floatx4*>(st) + (li * SLD + 4 * lg) / 4;

  for (int n0 = n_first; n0 < N; n0 += S) {
    floatx4 qv[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) qv[c] = qn[c];
    load_q(n0 + S);
    // (An opaque zero offset keeps the compiler from hoisting the LDS operand
    // reads out of the loop into registers.)
    int zero_off;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero_off));
    floatx4 acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[mb] = floatx4{0.f, 0.f, 0.f, 0.f};
    // The next chunk's S~ is read during the current one's products.
    floatx4 a[2][MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) a[0][mb] = st4[zero_off + mb * 4 * SLD];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      if (c + 1 < KC) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) a[(c + 1) & 1][mb] = st4[zero_off + mb * 4 * SLD + 4 * (c + 1)];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          acc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c & 1][mb][s], qv[c][s], acc[mb], 0, 0, 0);
    }
    // lane holds o[token n][mb*16 + 4*lg + i]
    const int n = n0 + li;
    float ss = 0.f;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 4; ++i) ss = fmaf(acc[mb][i], acc[mb][i], ss);
    ss += __shfl_xor(ss, 16);
    ss += __shfl_xor(ss, 32);
    // A raw query, as in readout_bf16_kernel: |q|^2 over the token's row.
    float qn2 = 1.0f;
    if (ql2) {
      float s = 0.f;
#pragma unroll
      for (int c = 0; c < KC; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) s = fmaf(qv[c][i], qv[c][i], s);
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      qn2 = s + kL2Eps;
    }
    const float scale = g / sqrtf(ss * inv_norm + kRmsEps * qn2);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      floatx4 y = acc[mb] * scale;
      const uint32_t ch = mb * 16 + 4 * lg;
      if constexpr (TOKGATE)
        y *= __builtin_bit_cast(
            floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                         grsrc, (int)((int)ch < dvo ? ((uint32_t)n * dvo + ch) * 4u : kOutOfRange), 0, 0));
      // Channels past dvo (zero padding of a narrow head) are not stored.
      store_b128(orsrc, (int)ch < dvo ? ((uint32_t)n * ors + ch) * 4u : kOutOfRange,
                 __builtin_bit_cast(u32x4, y));
    }
  }
}

inline int readout_chunks(long long fh_count, int N) {
  // Enough workgroups to cover the chip a few times, each with >= 512 tokens.
  const long long target = 2048;
  long long c = (target + fh_count - 1) / fh_count;
  const long long cap = (N + 511) / 512;
  if (c > cap) c = cap;
  return c < 1 ? 1 : (int)c;
}

// fp32 storage: workgroups per frame.  The kernel is bound by the matrix
// rate, which the workgroups of a compute unit share, so what matters is an
// even load over the compute units: a launch takes about as many 64-token
// steps as the busiest one has, and something like one more per workgroup
// for the state prologue.  The smallest count that minimises it is used (84
// frames of 1560 tokens on 256 compute units: 3 workgroups, 252 in all).
inline int readout_f32_chunks(long long fh_count, int N, int cus) {
  const int steps = (N + 63) / 64;
  int best = 1;
  long long best_cost = -1;
  for (int c = 1; c <= steps && c <= 32; ++c) {
    const long long cost = ((fh_count * c + cus - 1) / cus) * ((steps + c - 1) / c + 1);
    if (best_cost < 0 || cost < best_cost) best = c, best_cost = cost;
  }
  return best;
}

template <int DK, int DV>
hipError_t launch_readout_t(bool is_f32, const void* q, const float* S_fwd, const float* S_rev,
                            const float* gate, int F, int N, int H, int d_v_norm,
                            const GatherOptions& go, int cus, void* out, hipStream_t stream) {
  const long long fh_count = (long long)H * F;
  const bool genout = go.out_heads > 1 || d_v_norm != DV || go.q_heads > 1 || go.q_l2;
  const int ql2 = go.q_l2 ? 1 : 0;
  if (is_f32) {
    const int chunks = readout_f32_chunks(fh_count, N, cus);
    const dim3 grid((unsigned)(fh_count * chunks));
#define VDA_READOUT_F32(TG)                                                                      \
  hipLaunchKernelGGL((readout_f32_kernel<DK, DV, TG>), grid, dim3(kThreads), 0, stream,          \
                     static_cast<const float*>(q), S_fwd, S_rev, gate, F, N, chunks, grid.x,     \
                     d_v_norm, go.out_heads, go.q_heads, ql2, go.alpha, go.chunk, go.radius,     \
                     go.offset, static_cast<const float*>(go.gate_tokens),                       \
                     static_cast<float*>(out))
    if (go.gate_tokens != nullptr)
      VDA_READOUT_F32(true);
    else
      VDA_READOUT_F32(false);
#undef VDA_READOUT_F32
    return hipGetLastError();
  }
  const int chunks = readout_chunks(fh_count, N);
  const dim3 grid((unsigned)(fh_count * chunks));
#define VDA_READOUT_LAUNCH(TG, GO)                                                               \
  hipLaunchKernelGGL((readout_bf16_kernel<DK, DV, TG, GO>), grid, dim3(kThreads), 0, stream,     \
                     static_cast<const uint16_t*>(q), S_fwd, S_rev, gate, F, N, chunks, grid.x,  \
                     d_v_norm, go.out_heads, go.q_heads, ql2, go.alpha, go.chunk, go.radius,     \
                     go.offset, static_cast<const uint16_t*>(go.gate_tokens),                    \
                     static_cast<uint16_t*>(out))
  if (go.gate_tokens != nullptr) {
    if (genout) {
      VDA_READOUT_LAUNCH(true, true);
    } else {
      VDA_READOUT_LAUNCH(true, false);
    }
  } else if (genout) {
    VDA_READOUT_LAUNCH(false, true);
  } else {
    VDA_READOUT_LAUNCH(false, false);
  }
#undef VDA_READOUT_LAUNCH
  return hipGetLastError();
}

}  // namespace

hipError_t launch_readout(bool is_f32, const void* q, const float* S_fwd, const float* S_rev,
                          const float* gate, int F, int N, int H, int d_k, int d_v, int d_v_norm,
                          const GatherOptions& go, int cus, void* out, hipStream_t stream) {
#define VDA_READOUT_CASE(DKV, DVV)                                                             \
  if (d_k == DKV && d_v == DVV)                                                                \
    return launch_readout_t<DKV, DVV>(is_f32, q, S_fwd, S_rev, gate, F, N, H, d_v_norm, go, cus, \
                                      out, stream);
  VDA_READOUT_CASE(32, 32) VDA_READOUT_CASE(32, 64) VDA_READOUT_CASE(32, 128)
  VDA_READOUT_CASE(64, 32) VDA_READOUT_CASE(64, 64) VDA_READOUT_CASE(64, 128)
  VDA_READOUT_CASE(128, 32) VDA_READOUT_CASE(128, 64) VDA_READOUT_CASE(128, 128)
#undef VDA_READOUT_CASE
  return hipErrorInvalidValue;
}

}  // namespace vda
