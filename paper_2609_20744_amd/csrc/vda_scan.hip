// Steps a3/a4: the forward and reverse state scans of Eq. A.1 (alpha = 1),
// Algorithm 1 step 5, from a zero initial state:
//     P_t = (P_{t-1} + B_t) Inv_t,    R_t = (R_{t+1} + B_t) Inv_t.
// The entering state of every frame (P_{t-1} forward, R_{t+1} reverse) is
// stored for the readout.
//
// The rows of the d_v x d_k state evolve independently (each is a row vector
// times Inv_t), so a chain (head, direction) is split into 16-row blocks,
// one workgroup each, and the frame loop runs inside the workgroup with the
// 16 x d_k block of the state on chip, in fp32.  Per frame the wavefronts
// multiply the block by Inv_t, each producing some 16-column slices.  The
// matrices and B_t of the next two frames are in flight in a register ring,
// so memory latency stays off the serial path, which holds only the matrix
// product and its barriers.  Workgroups of one chain are placed on one XCD so
// they share Inv_t in its L2.
//
// Products: with fp32 storage (scan_f32_kernel), v_mfma_f32_16x16x4_f32
// (exact fp32 products).  With bf16 products (scan_bf16_kernel, which also
// stages Inv_t through LDS, see there), each fp32 operand x is split into
// bf16 hi = bf16(x) and lo = bf16(x - hi), and the product is hi*hi + hi*lo +
// lo*hi on v_mfma_f32_16x16x32_bf16 with fp32 accumulation (about 16
// mantissa bits per operand, relative error ~1e-5), several times the fp32
// matrix rate.
#include "vda_common.h"
#include "vda_launch.h"

namespace vda {
namespace {

__device__ __forceinline__ void split_bf16x8(const float (&x)[8], bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const __bf16 h = (__bf16)x[e];
    hi[e] = h;
    lo[e] = (__bf16)(x[e] - (float)h);
  }
}

// The exact fp32 scan (fp32 storage path).  Options of the full operator
// (template switches, so the core path carries none of their work):
//   DECAY  - the entering state is decayed, Sbar = S Diag(alpha_t), before
//            the frame's write (Eq. 5 / A.1 with alpha);
//   FROZEN - the frozen-state additive rule with 1/sqrt(U) key scaling,
//            S_t = Sbar_t (I - A_t / U) + B_t / sqrt(U) (Eq. 3c): the product
//            takes I - A_t / U, formed from A_t, and the write B_t / sqrt(U)
//            is added after it, that is at the start of the next step (B is
//            loaded one frame late).
// It may start from a text state, S_T / 2 (Eq. 1b).
// As in the tiled scan of the bf16 path the product
// is formed transposed, Inv_t x^T: its result leaves a lane four
// consecutive columns of one state row, which are its B-operand of the next
// product (v_mfma_f32_16x16x4_f32, lane group lg of k chunk c supplying k =
// 16 c + 4 lg + s in product s).  So each of NB / NBW waves keeps its NBW
// 16-column blocks of the 16 rows in registers and hands them to the others
// through LDS, double buffered, one barrier per step; B_t and the entering
// states pass through the wave's own LDS, so that memory sees whole runs of
// a row.  Inv_t comes as fp32 operand tiles (TILES, from the inverse in
// vda_forward's fp32 path) or by rows (the stage entry point; A_t of the
// frozen rule), of which it is symmetric; two steps ahead, each chunk
// refilled as its products are issued.  By rows a load takes 16 bytes of a
// different row per lane, and those loads bound the step: 52 us for
// 4 heads x 21 frames of 128 x 128 (51 before the state stayed in registers),
// and 37 from tiles, of which the products' issue is 19.
template <int DK, bool FROZEN, bool DECAY, bool TILES>
__global__ __launch_bounds__(DK == 32 ? 128 : 256) __attribute__((amdgpu_waves_per_eu(2)))
void scan_f32_kernel(const float* __restrict__ Mat, const float* __restrict__ Bm,
                     const float* __restrict__ alpha, const float* __restrict__ text_state,
                     int F, int DV, unsigned nwg, float inv_u, float inv_sqrt_u,
                     float* __restrict__ S_fwd, float* __restrict__ S_rev) {
  constexpr int NB = DK / 16;                 // 16-column blocks, and k chunks
  constexpr int NBW = DK == 128 ? 2 : 1;      // blocks per wave
  constexpr int W = NB / NBW;                 // waves
  constexpr int kRow = 16 * NBW + 4;          // floats per row of a wave's blocks in LDS
  constexpr int LPR = 4 * NBW;                // lanes per row in memory order
  constexpr int RPI = 64 / LPR;               // rows per access in memory order
  static_assert(16 / RPI == NBW, "as many accesses in either order");
  __shared__ floatx4 xop[2][NB][64];          // the state's operand: [step parity][chunk][lane]
  __shared__ __align__(16) float xb[W][16 * kRow], xs[W][16 * kRow];

  const int nrb = DV / 16;
  const unsigned L = xcd_grouped_id(blockIdx.x, nwg);
  const int rb = L % nrb;
  const unsigned chain = L / nrb;
  const int dir = chain & 1;
  const unsigned hb = chain >> 1;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform (scalar)
  const int li = lane & 15;
  const int lg = lane >> 4;

  const size_t mat_b = (size_t)DV * DK;  // one B / state matrix
  // This lane's state: row rb * 16 + li, columns col + 16 j + r (j < NBW, r < 4).
  const int col = 16 * NBW * wave + 4 * lg;
  // In memory order: row mrow + RPI j, columns mcol .. mcol + 3 of the wave's.
  const int mrow = lane / LPR, mcol = (lane % LPR) * 4;
  const uint32_t mem_off = (uint32_t)((rb * 16 + mrow) * DK + 16 * NBW * wave + mcol) * 4u;
  float* const bm = &xb[wave][mrow * kRow + mcol];
  const float* const bx = &xb[wave][li * kRow + 4 * lg];
  float* const sx = &xs[wave][li * kRow + 4 * lg];
  const float* const sm = &xs[wave][mrow * kRow + mcol];
  floatx4 x[NBW];
#pragma unroll
  for (int j = 0; j < NBW; ++j)
    x[j] = text_state != nullptr
               ? 0.5f * *reinterpret_cast<const floatx4*>(text_state + (size_t)hb * mat_b +
                                                          (size_t)(rb * 16 + li) * DK + col + 16 * j)
               : floatx4{0.f, 0.f, 0.f, 0.f};

  float* Sout = dir == 0 ? S_fwd : S_rev;
  const __amdgpu_buffer_rsrc_t srsrc =
      make_rsrc(Sout + (size_t)hb * F * mat_b, (uint32_t)(F * mat_b * sizeof(float)));
  const __amdgpu_buffer_rsrc_t brsrc =
      make_rsrc(Bm + (size_t)hb * F * mat_b, (uint32_t)(F * mat_b * sizeof(float)));
  const __amdgpu_buffer_rsrc_t arsrc =
      make_rsrc(DECAY ? alpha + (size_t)hb * F * DK : Bm, DECAY ? (uint32_t)(F * DK * 4) : 0u);
  const __amdgpu_buffer_rsrc_t mrsrc =
      make_rsrc(Mat + (size_t)hb * F * (DK * DK), (uint32_t)F * (uint32_t)(DK * DK * 4));

  auto frame_of = [&](int step) { return dir == 0 ? step : F - 1 - step; };

  // Two-slot register ring, as separately named arrays: step s uses slot
  // s % 2, whose registers take step s + 2 (past the end: a clamped, unused
  // step, so no branch hides the loads from the wait-count bookkeeping).
  struct Slot {
    floatx4 m[NBW][NB];  // rows 16 (NBW wave + j) + li of the matrix, by chunk
    floatx4 b[NBW];      // B_t (frozen: of the frame before), memory order
    floatx4 al[NBW];     // alpha_t
  };
  Slot s0, s1;
  auto load_add = [&](int step, Slot& s) {
    const int bframe = FROZEN ? frame_of(step - 1) : frame_of(step);
    const uint32_t off = (uint32_t)bframe * (uint32_t)(mat_b * 4u) + mem_off;
#pragma unroll
    for (int j = 0; j < NBW; ++j)
      s.b[j] = __builtin_bit_cast(
          floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                       brsrc, (int)((unsigned)bframe < (unsigned)F ? off + (uint32_t)(RPI * DK * 4 * j)
                                                                   : kOutOfRange),
                       0, 0));
    if constexpr (DECAY) {
#pragma unroll
      for (int j = 0; j < NBW; ++j)
        s.al[j] = __builtin_bit_cast(
            floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                         arsrc, (int)((uint32_t)(frame_of(step) * DK + col + 16 * j) * 4u), 0, 0));
    }
  };
  const uint32_t moff = TILES ? (uint32_t)(NBW * wave * NB * 1024 + lane * 16)
                              : (uint32_t)((16 * NBW * wave + li) * DK + 4 * lg) * 4u;
  auto load_chunk = [&](int step, Slot& s, int c) {
    const uint32_t base = (uint32_t)frame_of(step) * (uint32_t)(DK * DK * 4);
#pragma unroll
    for (int j = 0; j < NBW; ++j)
      s.m[j][c] = __builtin_bit_cast(
          floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                       mrsrc, (int)(moff + (TILES ? (uint32_t)((j * NB + c) * 1024)
                                                 : (uint32_t)((16 * j * DK + 16 * c) * 4))),
                       (int)base, 0));
  };

  // B of the coming step in the products' order (a wave's LDS operations run
  // in order).
  floatx4 bn[NBW];
  auto turn_b = [&](const Slot& s) {
#pragma unroll
    for (int j = 0; j < NBW; ++j) *reinterpret_cast<floatx4*>(bm + RPI * kRow * j) = s.b[j];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < NBW; ++j) bn[j] = *reinterpret_cast<const floatx4*>(bx + 16 * j);
    __builtin_amdgcn_wave_barrier();
  };

  // Step `step` on slot s; o is the other slot, the coming step's.
  auto step_body = [&](int step, int par, Slot& s, const Slot& o) {
#pragma unroll
    for (int j = 0; j < NBW; ++j) {
      floatx4 u;
      if constexpr (FROZEN) {
        x[j] += bn[j] * inv_sqrt_u;  // the previous frame's write
        u = DECAY ? x[j] * s.al[j] : x[j];
      } else {
        u = DECAY ? x[j] * s.al[j] + bn[j] : x[j] + bn[j];
      }
      xop[par][NBW * wave + j][lane] = u;
      *reinterpret_cast<floatx4*>(sx + 16 * j) = x[j];  // the entering state, on its way to memory
    }
    lds_barrier();  // the state's operand is complete
    floatx4 y[NBW];
#pragma unroll
    for (int j = 0; j < NBW; ++j) y[j] = *reinterpret_cast<const floatx4*>(sm + RPI * kRow * j);
    const int refill = min(step + 2, F - 1);
    load_add(refill, s);
    turn_b(o);
    const uint32_t soff = (uint32_t)frame_of(step) * (uint32_t)(mat_b * 4u) + mem_off;
#pragma unroll
    for (int j = 0; j < NBW; ++j)
      store_b128(srsrc, step < F ? soff + (uint32_t)(RPI * DK * 4 * j) : kOutOfRange,
                 __builtin_bit_cast(u32x4, y[j]));
    // Even and odd products in separate accumulators.
    floatx4 acc[NBW][2];
#pragma unroll
    for (int j = 0; j < NBW; ++j) acc[j][0] = acc[j][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      const floatx4 xv = xop[par][c][lane];
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < NBW; ++j) {
          float m = s.m[j][c][e];
          if constexpr (FROZEN)  // I - A / U
            m = (16 * c + 4 * lg + e == 16 * (NBW * wave + j) + li ? 1.0f : 0.0f) - m * inv_u;
          acc[j][e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(m, xv[e], acc[j][e & 1], 0, 0, 0);
        }
      load_chunk(refill, s, c);
    }
#pragma unroll
    for (int j = 0; j < NBW; ++j) x[j] = acc[j][0] + acc[j][1];
  };

  auto fill = [&](int step, Slot& s) {
    load_add(step, s);
#pragma unroll
    for (int c = 0; c < NB; ++c) load_chunk(step, s, c);
    __builtin_amdgcn_sched_barrier(0);
  };
  fill(0, s0);
  fill(min(1, F - 1), s1);
  turn_b(s0);
  // A padded step (step >= F) reads a clamped matrix and stores nothing.
  for (int step = 0; step < F; step += 2) {
    step_body(step, 0, s0, s1);
    step_body(step + 1, 1, s1, s0);
  }
}

// 16-byte chunks of the blocks on and above the diagonal of a DK x DK fp32
// matrix (row-major): block row i holds 16 rows of (DK - 16 i) / 4 chunks,
// starting at column 16 i.
template <int DK>
struct UpperChunks {
  static constexpr int NB = DK / 16;
  static constexpr int total = 16 * (NB * DK / 4 - 2 * NB * (NB - 1));
  static constexpr int per_thread = (total + kThreads - 1) / kThreads;
};

// Row and first column of upper-triangle chunk f (f < UpperChunks<DK>::total).
template <int DK>
__device__ __forceinline__ void upper_chunk(int f, int& row, int& col) {
  int start = 0;
  row = 0;
  col = 0;
#pragma unroll
  for (int i = 0; i < DK / 16; ++i) {
    const int cw = (DK - 16 * i) / 4;  // chunks per row in block row i
    if (f >= start && f < start + 16 * cw) {
      const int loc = f - start;
      row = 16 * i + loc / cw;
      col = 16 * i + 4 * (loc % cw);
    }
    start += 16 * cw;
  }
}

// Matrix-core phase of one scan step for wave W (a template, so that which
// operand halves are read along rows and which down columns is fixed at
// compile time and no branch separates the LDS reads): out = x Inv_t for
// this wave's 16-column slices.  x, the 16 x d_k block, comes already split
// into bf16 hi and lo planes (row stride PLD); Inv_t is the upper-triangle
// image (row stride XLD).  Even and odd k steps accumulate separately, which
// halves the chain of dependent matrix products.
template <int DK, int W>
__device__ __forceinline__ void scan_mfma_phase(const uint16_t* __restrict__ xhi,
                                                const uint16_t* __restrict__ xlo,
                                                float* __restrict__ xs_next,
                                                const float* __restrict__ ivs, int li, int lg) {
  constexpr int XLD = DK + 4;
  constexpr int PLD = DK + 8;
  constexpr int NB = DK / 16;
  constexpr int NBW = (NB + 3) / 4;
  constexpr int KB = DK / 32;
  if constexpr (W >= NB) {
    return;  // d_k = 32: two slices, waves 2 and 3 idle
  } else {
    // A-operand: row li of the block at k = 32 ks + 4 lg + e, 32 ks + 16 + 4 lg + e.
    bf16x8 ahi[KB], alo[KB];
#pragma unroll
    for (int ks = 0; ks < KB; ++ks) {
      const int o = li * PLD + 32 * ks + 4 * lg;
      const u32x2 h0 = *reinterpret_cast<const u32x2*>(&xhi[o]);
      const u32x2 h1 = *reinterpret_cast<const u32x2*>(&xhi[o + 16]);
      const u32x2 l0 = *reinterpret_cast<const u32x2*>(&xlo[o]);
      const u32x2 l1 = *reinterpret_cast<const u32x2*>(&xlo[o + 16]);
      ahi[ks] = __builtin_bit_cast(bf16x8, u32x4{h0[0], h0[1], h1[0], h1[1]});
      alo[ks] = __builtin_bit_cast(bf16x8, u32x4{l0[0], l0[1], l1[0], l1[1]});
    }
#pragma unroll
    for (int m = 0; m < NBW; ++m) {
      const int nb = W + 4 * m;
      if (nb < NB) {
        floatx4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < KB; ++ks) {
          // B-operand: Inv[k][16 nb + li] at this lane's k values, in two
          // halves of four, each inside k block kb = 2 ks + h.
          float t[8];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int k0 = 32 * ks + 16 * h + 4 * lg;
            if (2 * ks + h > nb) {  // row 16 nb + li of the stored block (nb, kb)
              const floatx4 v = reinterpret_cast<const floatx4*>(ivs)[((nb * 16 + li) * XLD + k0) / 4];
#pragma unroll
              for (int c = 0; c < 4; ++c) t[4 * h + c] = v[c];
            } else {  // column 16 nb + li of the stored block (kb, nb)
              const float* q = &ivs[k0 * XLD + nb * 16 + li];
#pragma unroll
              for (int c = 0; c < 4; ++c) t[4 * h + c] = q[c * XLD];
            }
          }
          bf16x8 bhi, blo;
          split_bf16x8(t, bhi, blo);
          floatx4& a = acc[ks & 1];
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo[ks], bhi, a, 0, 0, 0);
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi[ks], blo, a, 0, 0, 0);
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi[ks], bhi, a, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
          xs_next[(lg * 4 + i) * XLD + nb * 16 + li] = acc[0][i] + acc[1][i];
      }
    }
  }
}

// The split-bf16 scan from Inv_t by rows.  The recurrence, the work split
// (one 16-row block of one chain per workgroup) and the products are those
// of scan_f32_kernel; the difference is how Inv_t reaches the matrix cores.
// Per frame the workgroup copies only the blocks of Inv_t on and above the
// diagonal (36 of 64 at d_k = 128; the others are their transposes, as
// Inv_t is symmetric) with consecutive lanes on consecutive 16-byte chunks
// into an LDS image, and each wave reads its operands from there.  Scattered
// per-lane reads of whole rows of Inv_t from memory are limited by the
// address units, not by bandwidth; the coalesced half-size copy is what
// makes this scan faster.  Inv_t and B_t of the next two frames are in
// flight in a register ring.
//
// Matrix-core k order: in each 32-wide k step, lane group g holds
// k = 4g + e and 16 + 4g + e (e < 4), in both operands.  So each 4-value
// half of an operand lies in one 16 x 16 block of Inv_t: block (kb, nb) with
// kb = 2 ks or 2 ks + 1 for output column block nb, the same for every lane.
// When kb > nb the half is read along row 16 nb + li of the stored block
// (nb, kb) (one 16-byte read), otherwise down column 16 nb + li of the stored
// block (kb, nb) (four 4-byte reads).  With a row stride of 132 floats the
// two lane groups of each 32-lane LDS pass then fall on distinct banks in
// both kinds of read.
//
// It serves the stage entry point, which takes Inv_t by rows and none of the
// full operator's options: with bf16 storage the whole passes run on the tiled
// scan.
template <int DK>
__global__ __launch_bounds__(kThreads)
void scan_bf16_kernel(const float* __restrict__ Mat, const float* __restrict__ Bm,
                      int F, int DV, unsigned nwg, float* __restrict__ S_fwd,
                      float* __restrict__ S_rev) {
  constexpr int XLD = DK + 4;        // LDS row stride (floats)
  constexpr int VW = DK >= 64 ? 4 : 2;  // floats per access in the row-wise phase
  constexpr int NG = DK / (16 * VW);    // accesses per thread in the row-wise phase
  using U = UpperChunks<DK>;
  constexpr int CPT = U::per_thread;
  constexpr int PLD = DK + 8;        // bf16 row stride of the split planes
  __shared__ __align__(16) float ivs[(DK + 1) * XLD];  // matrix image, plus a dummy row
  __shared__ __align__(16) float xs[2][16 * XLD];
  __shared__ __align__(16) uint16_t xsp[2][16 * PLD];   // bf16 hi / lo planes of the block

  const int nrb = DV / 16;
  const unsigned L = xcd_grouped_id(blockIdx.x, nwg);
  const int rb = L % nrb;
  const unsigned chain = L / nrb;
  const int dir = chain & 1;
  const unsigned hb = chain >> 1;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform (scalar)
  const int li = lane & 15;
  const int lg = lane >> 4;

  // Row-wise phase role: row pr of the block; access g covers columns
  // pc + g * 16 * VW .. + VW - 1 (16 consecutive lanes on one contiguous run).
  const int pr = tid >> 4;
  const int pc = (tid & 15) * VW;

  const size_t mat_b = (size_t)DV * DK;  // one B / state matrix
  for (int i = tid; i < 16 * XLD; i += kThreads) xs[0][i] = 0.f;  // the initial state

  float* Sout = dir == 0 ? S_fwd : S_rev;
  const size_t row_off = (size_t)(rb * 16 + pr) * DK + pc;
  // Entering states of this head, [F][d_v][d_k]: a range-checked buffer, so
  // the padded steps past the last frame store nothing.
  const __amdgpu_buffer_rsrc_t srsrc =
      make_rsrc(Sout + (size_t)hb * F * mat_b, (uint32_t)(F * mat_b * sizeof(float)));
  // B of this head, range-checked (frames outside [0, F) read as zero).
  const __amdgpu_buffer_rsrc_t brsrc =
      make_rsrc(Bm + (size_t)hb * F * mat_b, (uint32_t)(F * mat_b * sizeof(float)));

  auto frame_of = [&](int step) { return dir == 0 ? step : F - 1 - step; };

  // This thread's upper-triangle chunks: byte offsets within a matrix and
  // LDS positions in 16-byte units (chunks past the end: out of range, and
  // the dummy row).
  uint32_t goff[CPT];
  int loff[CPT];
#pragma unroll
  for (int e = 0; e < CPT; ++e) {
    const int f = e * kThreads + tid;
    int row, col;
    upper_chunk<DK>(f, row, col);
    const bool in = f < U::total;
    goff[e] = in ? (uint32_t)(row * DK + col) * 4u : kOutOfRange;
    loff[e] = (in ? row * XLD + col : DK * XLD) / 4;
  }

  // Two-frame register ring, as separately named arrays (compile-time
  // indices only).
  u32x4 ir0[CPT], ir1[CPT];
  float bs0[NG][VW], bs1[NG][VW];
  auto load_step = [&](int step, u32x4 (&ir)[CPT], float (&bb)[NG][VW]) {
    const int frame = frame_of(step);
    // B rows first (they are needed earlier in the step than the matrix),
    // and everything through buffer loads, which the compiler keeps in
    // program order.
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const uint32_t off = (uint32_t)(((size_t)frame * mat_b + row_off + g * 16 * VW) * 4u);
      if constexpr (VW == 4) {
        const u32x4 x =
            __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(brsrc, (int)off, 0, 0));
#pragma unroll
        for (int v = 0; v < 4; ++v) bb[g][v] = __uint_as_float(x[v]);
      } else {
        const u32x2 x =
            __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(brsrc, (int)off, 0, 0));
        bb[g][0] = __uint_as_float(x[0]);
        bb[g][1] = __uint_as_float(x[1]);
      }
    }
    const size_t fh = (size_t)hb * F + frame;
    const __amdgpu_buffer_rsrc_t irsrc = make_rsrc(Mat + fh * (DK * DK), DK * DK * 4u);
#pragma unroll
    for (int e = 0; e < CPT; ++e)
      ir[e] = __builtin_bit_cast(
          u32x4, __builtin_amdgcn_raw_buffer_load_b128(irsrc, (int)goff[e], 0, 0));
  };

  auto stage = [&](const u32x4 (&ir)[CPT]) {
#pragma unroll
    for (int e = 0; e < CPT; ++e) reinterpret_cast<u32x4*>(ivs)[loff[e]] = ir[e];
  };

  int cur = 0;
  auto step_body = [&](int step, u32x4 (&ir)[CPT], float (&bb)[NG][VW]) {
    // Frame index within the head; past the end it is out of the buffer
    // range (>= F forward, negative and so huge as unsigned in reverse).
    const int frame = dir == 0 ? step : F - 1 - step;
    lds_barrier();  // xs[cur] holds the entering state; the last matrix image is consumed
    stage(ir);
    {
      const uint32_t off = (uint32_t)((size_t)(unsigned)frame * mat_b + row_off) * 4u;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        float* x = &xs[cur][pr * XLD + pc + g * 16 * VW];
        float v[VW];
        if constexpr (VW == 4) {
          const floatx4 xv = reinterpret_cast<const floatx4*>(xs[cur])[(pr * XLD + pc + g * 16 * VW) / 4];
#pragma unroll
          for (int c = 0; c < 4; ++c) v[c] = xv[c];
        } else {
          const float2 xv = *reinterpret_cast<const float2*>(x);
          v[0] = xv.x;
          v[1] = xv.y;
        }
        if constexpr (VW == 4)
          store_b128(srsrc, off + g * 64u * VW,
                     u32x4{__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]),
                           __float_as_uint(v[3])});
        else
          store_b64(srsrc, off + g * 64u * VW, make_uint2(__float_as_uint(v[0]), __float_as_uint(v[1])));
#pragma unroll
        for (int c = 0; c < VW; ++c) v[c] += bb[g][c];
        // The product's A-operand, split once here into bf16 hi and lo
        // (instead of by each of the four waves).
        uint32_t hw[VW / 2], lw[VW / 2];
#pragma unroll
        for (int c = 0; c < VW; c += 2) {
          const uint32_t h = pack_bf16x2(v[c], v[c + 1]);
          hw[c / 2] = h;
          lw[c / 2] = pack_bf16x2(v[c] - bf16_lo(h), v[c + 1] - bf16_hi(h));
        }
        const int po = pr * PLD + pc + g * 16 * VW;
        if constexpr (VW == 4) {
          *reinterpret_cast<u32x2*>(&xsp[0][po]) = u32x2{hw[0], hw[1]};
          *reinterpret_cast<u32x2*>(&xsp[1][po]) = u32x2{lw[0], lw[1]};
        } else {
          *reinterpret_cast<uint32_t*>(&xsp[0][po]) = hw[0];
          *reinterpret_cast<uint32_t*>(&xsp[1][po]) = lw[0];
        }
        (void)x;
      }
    }
    lds_barrier();
    // Always refill (past the end: a clamped, unused frame) so no branch
    // hides the loads from the wait-count bookkeeping.
    load_step(min(step + 2, F - 1), ir, bb);
    switch (wave) {  // wave-uniform
      case 0: scan_mfma_phase<DK, 0>(xsp[0], xsp[1], xs[cur ^ 1], ivs, li, lg); break;
      case 1: scan_mfma_phase<DK, 1>(xsp[0], xsp[1], xs[cur ^ 1], ivs, li, lg); break;
      case 2: scan_mfma_phase<DK, 2>(xsp[0], xsp[1], xs[cur ^ 1], ivs, li, lg); break;
      default: scan_mfma_phase<DK, 3>(xsp[0], xsp[1], xs[cur ^ 1], ivs, li, lg); break;
    }
    cur ^= 1;
  };

  // Issue the ring in slot order (pinned against rescheduling) so slot 0 is
  // the oldest load on loop entry.
  load_step(0, ir0, bs0);
  __builtin_amdgcn_sched_barrier(0);
  load_step(min(1, F - 1), ir1, bs1);
  __builtin_amdgcn_sched_barrier(0);
  // The step count is padded to an even number; a padded step (step >= F)
  // reads a clamped frame and its stores are dropped, so the loop body has
  // no early exit.
  for (int step0 = 0; step0 < F; step0 += 2) {
    step_body(step0, ir0, bs0);
    step_body(step0 + 1, ir1, bs1);
  }
}

template <int DK, bool FROZEN, bool DECAY>
hipError_t launch_scan_f32(const float* Mat, const float* Bm, int F, int H, int d_v,
                           const ScanOptions& o, bool f32_tiles, float* S_fwd, float* S_rev,
                           hipStream_t stream) {
  const unsigned nwg = (unsigned)H * 2u * (unsigned)(d_v / 16);
  const float inv_u = FROZEN ? 1.0f / (float)o.tokens : 0.0f;
  const float inv_sqrt_u = FROZEN ? 1.0f / sqrtf((float)o.tokens) : 0.0f;
  const dim3 block(DK == 32 ? 128 : 256);
  if (f32_tiles) {
    if constexpr (FROZEN) return hipErrorInvalidValue;
    else
      hipLaunchKernelGGL((scan_f32_kernel<DK, false, DECAY, true>), dim3(nwg), block, 0, stream,
                         Mat, Bm, o.alpha, o.text_state, F, d_v, nwg, inv_u, inv_sqrt_u, S_fwd,
                         S_rev);
  } else {
    hipLaunchKernelGGL((scan_f32_kernel<DK, FROZEN, DECAY, false>), dim3(nwg), block, 0, stream,
                       Mat, Bm, o.alpha, o.text_state, F, d_v, nwg, inv_u, inv_sqrt_u, S_fwd,
                       S_rev);
  }
  return hipGetLastError();
}

template <int DK>
hipError_t launch_scan_t(bool exact_f32, const float* Mat, const float* Bm, int F, int H, int d_v,
                         const ScanOptions& o, bool f32_tiles, float* S_fwd, float* S_rev,
                         hipStream_t stream) {
  const bool decay = o.alpha != nullptr;
  if (!exact_f32) {
    if (o.frozen || decay || o.text_state != nullptr) return hipErrorInvalidValue;
    const unsigned nwg = (unsigned)H * 2u * (unsigned)(d_v / 16);
    hipLaunchKernelGGL(scan_bf16_kernel<DK>, dim3(nwg), dim3(kThreads), 0, stream, Mat, Bm, F, d_v,
                       nwg, S_fwd, S_rev);
    return hipGetLastError();
  }
#define VDA_SCAN_F32(FROZEN, DECAY) \
  launch_scan_f32<DK, FROZEN, DECAY>(Mat, Bm, F, H, d_v, o, f32_tiles, S_fwd, S_rev, stream)
  if (o.frozen) return decay ? VDA_SCAN_F32(true, true) : VDA_SCAN_F32(true, false);
  return decay ? VDA_SCAN_F32(false, true) : VDA_SCAN_F32(false, false);
#undef VDA_SCAN_F32
}

}  // namespace

hipError_t launch_state_scan(bool exact_f32, const float* Mat, const float* Bm, int F, int H,
                             int d_k, int d_v, const ScanOptions& o, float* S_fwd, float* S_rev,
                             hipStream_t stream, bool f32_tiles) {
  switch (d_k) {
    case 32: return launch_scan_t<32>(exact_f32, Mat, Bm, F, H, d_v, o, f32_tiles, S_fwd, S_rev, stream);
    case 64: return launch_scan_t<64>(exact_f32, Mat, Bm, F, H, d_v, o, f32_tiles, S_fwd, S_rev, stream);
    case 128: return launch_scan_t<128>(exact_f32, Mat, Bm, F, H, d_v, o, f32_tiles, S_fwd, S_rev, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace vda
