// Steps a3/a4 on the bf16 storage path for the joint rule: the forward and
// reverse state scans of Eq. A.1 (Algorithm 1 step 5),
//     P_t = (P_{t-1} Diag(alpha_t) + B_t) Inv_t,
//     R_t = (R_{t+1} Diag(alpha_t) + B_t) Inv_t,
// from S_T / 2 (Eq. 1b) or zero, with alpha = 1 unless a decay is given.
// The entering state of every frame (P_{t-1} forward, R_{t+1} reverse) is
// stored for the readout.
//
// Work split as in the other scans: one workgroup per (head, direction,
// 16-row block of the state); the rows of the state evolve independently.
// The product is formed transposed, Inv_t^T x^T, with the operand tiles that
// the inverse wrote (operand_tile_offset) as A-operands and the state as
// B-operand of v_mfma_f32_16x16x32_bf16: a lane then receives four
// consecutive columns of one state row, and output slices 2 w and 2 w + 1
// are exactly the B-operand of k step w of the next product.  So wave w of
// d_k / 32 owns the 32 state columns of k step w, in registers, all the way:
// it adds B_t (and applies the decay) where the product leaves them, stores
// the entering state, splits it and hands its operand (1 KB in each of two
// planes) to the other waves through LDS, double buffered, with one barrier
// per step (none at d_k = 32, one wave).  Each wave loads the tiles of its own
// two output slices straight into registers, one contiguous 1 KB piece per
// load instruction, two steps ahead of use: the two-slot ring refills a
// piece's registers as soon as its products are issued.
//
// What bounds it: the serial step, operand reads after the barrier, 6 d_k / 32
// products per wave, B_t and the split, at d_k = 128 about the time in which
// a compute unit can load the 64 KB of tiles (with every load from two
// frames only: 1.0 us a step at 16 heads, 1.2 with the real ones, 43 us for
// 36 frames and 226 MB; 0.54 and 0.62 at d_k = 64).  With all of the state in
// LDS and two barriers a step, passes were 3.5 us longer at 8 heads x 16
// frames (16 steps: 20.5 -> 18.4 us), 2 at 16 x 36, 4 in the frozen rule's
// map form; rings of three and four slots measured no faster (the loads are
// not late).
//
// Products: the state operand x is split into hi = bf16(x) and
// lo = bf16(x - hi) once per step, and hi*hi + hi*lo + lo*hi runs on the
// bf16 matrix cores with fp32 accumulation (about 16 mantissa bits per
// operand; relative error ~1e-5 per step, which the non-expansive frame maps
// of Prop. 1 keep from growing along the scan).
#include "vda_common.h"
#include "vda_inverse_body.h"
#include "vda_launch.h"

namespace vda {
namespace {

// Arguments of the tiled scan.  Frame scans: tiles = Inv_t tiles [H][F],
// add = B [H][F][d_v][d_k].  Map scans (CHUNKED), x <- x M + add_scale J:
// chunk scans take tiles = M_c tiles [H][2][C] and add = J_c
// [H][2][C][d_v][d_k] over the C chunks of the window grid (chunk, offset),
// one set per direction (mats_per_head = 2C, dir_stride = C); the frozen
// rule takes per-frame maps M_t = Diag(alpha_t)(I - A_t / U) and J_t = B_t
// scaled by 1 / sqrt(U), shared by both directions (chunks of one frame,
// mats_per_head = F, dir_stride = 0).
struct TiledScanArgs {
  const uint16_t* tiles;
  const float* add;
  const float* alpha;
  const float* text_state;
  int F, DV;
  unsigned nwg;
  int chunk, offset, C;
  int mats_per_head, dir_stride;
  float add_scale;
  float* S_fwd;
  float* S_rev;
};

// CHUNKED: the same recurrence over the chunk sequence,
//     x <- x M_c + J_c,
// storing the state entering chunk c at its first frame (forward) or its
// last frame (reverse).  The additive term comes after the product here, so
// step j adds J of the previous chunk (loaded one step late) to the product
// before it stores and splits the state; the last step's product is unused.
// At most 256 registers per lane (two waves per SIMD), so two workgroups
// share a compute unit when there are more chains' row blocks than compute
// units (e.g. 24 heads: 384 workgroups) instead of running in two rounds.
template <int DK, bool DECAY, bool CHUNKED>
__global__ __launch_bounds__(2 * DK) __attribute__((amdgpu_waves_per_eu(2)))
void scan_tiled_kernel(TiledScanArgs a) {
  static_assert(!(CHUNKED && DECAY), "chunk maps already hold the decay");
  constexpr int KB = DK / 32;  // 32-wide k steps, and waves
  constexpr uint32_t kPlane = DK * DK * 2;
  constexpr int kRow = 36;     // floats per 32-column row in LDS
  // The state's operand of a step: [step parity][k step][hi, lo][lane].
  __shared__ u32x4 xop[KB > 1 ? 2 : 1][KB][2][64];
  // Per wave: its 16 x 32 pieces of B_t and of the entering state on their
  // way between memory order (eight lanes on one 128-byte run of a row) and
  // the products' (a lane's row is lane % 16).  In memory the latter would
  // be 16 bytes of a different row per lane, which the texture addresser
  // takes four times as long for.
  __shared__ __align__(16) float xb[KB][16 * kRow], xs[KB][16 * kRow];
  const int F = a.F, DV = a.DV, C = a.C;

  const int nrb = DV / 16;
  const unsigned L = xcd_grouped_id(blockIdx.x, a.nwg);
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
  // This lane's state: row rb * 16 + li, columns col + 16 j + r (j < 2, r < 4).
  const int col = 32 * wave + 4 * lg;
  // In memory order: row mrow + 8 j, columns mcol .. mcol + 3 of the wave's 32.
  const int mrow = lane >> 3, mcol = (lane & 7) * 4;
  const uint32_t mem_off = (uint32_t)((rb * 16 + mrow) * DK + 32 * wave + mcol) * 4u;
  float* const bm = &xb[wave][mrow * kRow + mcol];       // memory order, + 8 kRow j
  const float* const bx = &xb[wave][li * kRow + 4 * lg]; // products' order, + 16 j
  float* const sx = &xs[wave][li * kRow + 4 * lg];
  const float* const sm = &xs[wave][mrow * kRow + mcol];
  floatx4 x[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  if (a.text_state != nullptr) {  // S_T / 2
    const float* ts = a.text_state + (size_t)hb * mat_b + (size_t)(rb * 16 + li) * DK + col;
#pragma unroll
    for (int j = 0; j < 2; ++j) x[j] = 0.5f * *reinterpret_cast<const floatx4*>(ts + 16 * j);
  }

  float* Sout = dir == 0 ? a.S_fwd : a.S_rev;
  // Entering states of this head, [F][d_v][d_k]: a range-checked buffer.
  const __amdgpu_buffer_rsrc_t srsrc =
      make_rsrc(Sout + (size_t)hb * F * mat_b, (uint32_t)(F * mat_b * sizeof(float)));
  // Steps: frames, or chunks; matrices (tiles) and additive terms of this
  // chain, range-checked (indices outside read as zero).
  const int nsteps = CHUNKED ? C : F;
  const size_t chain_mats =
      CHUNKED ? (size_t)hb * a.mats_per_head + (size_t)dir * a.dir_stride : (size_t)hb * F;
  const __amdgpu_buffer_rsrc_t brsrc =
      make_rsrc(a.add + chain_mats * mat_b, (uint32_t)(nsteps * mat_b * sizeof(float)));
  const __amdgpu_buffer_rsrc_t arsrc =
      make_rsrc(DECAY ? a.alpha + (size_t)hb * F * DK : a.add, DECAY ? (uint32_t)(F * DK * 4) : 0u);
  const __amdgpu_buffer_rsrc_t trsrc = make_rsrc(a.tiles + chain_mats * (DK * DK * 2),
                                                 (uint32_t)nsteps * (uint32_t)(DK * DK * 4));

  // Matrix of step `step` (frame or chunk in scan order), the index of its
  // additive term (chunks: the previous chunk's J, none before the first),
  // and the frame whose entering state the step stores (-1: none, for a
  // padded step past the end).
  auto frame_of = [&](int step) { return dir == 0 ? step : nsteps - 1 - step; };
  auto add_of = [&](int step) {
    if constexpr (CHUNKED) return step >= 1 ? frame_of(step - 1) : -1;
    return frame_of(step);
  };
  auto store_frame = [&](int step) {
    if (step >= nsteps) return -1;
    if constexpr (CHUNKED) {
      const int c = frame_of(step);
      return dir == 0 ? max(0, c * a.chunk - a.offset) : min(F - 1, (c + 1) * a.chunk - a.offset - 1);
    }
    return frame_of(step);
  };

  // Two-slot register ring, as separately named arrays (compile-time indices
  // only): step s uses slot s % 2, whose registers take step s + 2 (past the
  // end: a clamped, unused step, so no branch hides the loads from the
  // wait-count bookkeeping).
  struct Slot {
    u32x4 t[2][KB][2];  // tiles of slices 2 wave + j: [j][k step][plane]
    floatx4 b[2];       // B_t (J), memory order
    floatx4 al[2];      // alpha_t
  };
  Slot s0, s1;
  auto load_add = [&](int step, Slot& s) {
    const int ai = add_of(step);
    const uint32_t off = (uint32_t)ai * (uint32_t)(mat_b * 4u) + mem_off;
#pragma unroll
    for (int j = 0; j < 2; ++j)
      s.b[j] = __builtin_bit_cast(
          floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                       brsrc, (int)(ai >= 0 ? off + (uint32_t)(8 * DK * 4 * j) : kOutOfRange), 0, 0));
    if constexpr (DECAY) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
        s.al[j] = __builtin_bit_cast(
            floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                         arsrc, (int)((uint32_t)(frame_of(step) * DK + col + 16 * j) * 4u), 0, 0));
    }
  };
  const uint32_t toff = operand_tile_offset(DK, 0, 2 * wave, 0, lane);
  auto load_piece = [&](uint32_t fbase, Slot& s, int j, int ks) {
#pragma unroll
    for (int p = 0; p < 2; ++p)
      s.t[j][ks][p] = __builtin_bit_cast(
          u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                     trsrc, (int)(toff + (uint32_t)(j * KB + ks) * 1024u + (uint32_t)p * kPlane),
                     (int)fbase, 0));
  };
  auto tile_base = [&](int step) { return (uint32_t)frame_of(step) * (uint32_t)(DK * DK * 4); };

  // B of the coming step in the products' order, by way of this wave's LDS
  // (a wave's LDS operations run in order).
  floatx4 bn[2];
  auto turn_b = [&](const Slot& s) {
#pragma unroll
    for (int j = 0; j < 2; ++j) *reinterpret_cast<floatx4*>(bm + 8 * kRow * j) = s.b[j];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < 2; ++j) bn[j] = *reinterpret_cast<const floatx4*>(bx + 16 * j);
    __builtin_amdgcn_wave_barrier();
  };

  // Step `step` on slot s; o is the other slot, the coming step's.
  auto step_body = [&](int step, int par, Slot& s, Slot& o) {
    floatx4 u[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if constexpr (CHUNKED) {  // J of the previous chunk, after its product
#pragma unroll
        for (int r = 0; r < 4; ++r) x[j][r] = fmaf(bn[j][r], a.add_scale, x[j][r]);
        u[j] = x[j];
      } else {  // B of this frame, before its product
        u[j] = DECAY ? x[j] * s.al[j] + bn[j] : x[j] + bn[j];
      }
    }
    // The product's B-operand of k step `wave`, split into bf16 hi and lo.
    uint32_t h[4], l[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float v0 = u[q / 2][2 * (q % 2)], v1 = u[q / 2][2 * (q % 2) + 1];
      h[q] = pack_bf16x2(v0, v1);
      l[q] = pack_bf16x2(v0 - bf16_lo(h[q]), v1 - bf16_hi(h[q]));
    }
    bf16x8 xh[KB], xl[KB];
    if constexpr (KB > 1) {
      xop[par][wave][0][lane] = u32x4{h[0], h[1], h[2], h[3]};
      xop[par][wave][1][lane] = u32x4{l[0], l[1], l[2], l[3]};
    }
    // The later k steps' tiles of the step before, refilled here rather than
    // behind its products, so that the loads spread over the whole step (at
    // step 0: the same tiles again).
    if constexpr (KB > 1) {
      const uint32_t late = tile_base(min(step + 1, nsteps - 1));
#pragma unroll
      for (int ks = KB / 2; ks < KB; ++ks)
#pragma unroll
        for (int j = 0; j < 2; ++j) load_piece(late, o, j, ks);
    }
    // The entering state, on its way to memory.
#pragma unroll
    for (int j = 0; j < 2; ++j) *reinterpret_cast<floatx4*>(sx + 16 * j) = x[j];
    if constexpr (KB > 1) {
      lds_barrier();  // the state's operand is complete
#pragma unroll
      for (int ks = 0; ks < KB; ++ks) {
        xh[ks] = __builtin_bit_cast(bf16x8, xop[par][ks][0][lane]);
        xl[ks] = __builtin_bit_cast(bf16x8, xop[par][ks][1][lane]);
      }
    } else {
      xh[0] = __builtin_bit_cast(bf16x8, u32x4{h[0], h[1], h[2], h[3]});
      xl[0] = __builtin_bit_cast(bf16x8, u32x4{l[0], l[1], l[2], l[3]});
    }
    const int refill = min(step + 2, nsteps - 1);
    const uint32_t next = tile_base(refill);
    __builtin_amdgcn_wave_barrier();
    floatx4 y[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) y[j] = *reinterpret_cast<const floatx4*>(sm + 8 * kRow * j);
    load_add(refill, s);
    turn_b(o);
    const int sf = store_frame(step);
    const uint32_t soff = (uint32_t)sf * (uint32_t)(mat_b * 4u) + mem_off;
#pragma unroll
    for (int j = 0; j < 2; ++j)
      store_b128(srsrc, sf >= 0 ? soff + (uint32_t)(8 * DK * 4 * j) : kOutOfRange,
                 __builtin_bit_cast(u32x4, y[j]));
    // Even and odd k steps accumulate separately, and the two slices in turn:
    // four independent chains.  After a k step's products its tiles are
    // refilled.
    floatx4 acc[2][2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 2; ++e) acc[j][e] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KB; ++ks) {
      const int e = ks & 1;
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[j][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, s.t[j][ks][0]), xl[ks], acc[j][e], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[j][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, s.t[j][ks][1]), xh[ks], acc[j][e], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[j][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, s.t[j][ks][0]), xh[ks], acc[j][e], 0, 0, 0);
      if (KB == 1 || ks < KB / 2) {
#pragma unroll
        for (int j = 0; j < 2; ++j) load_piece(next, s, j, ks);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);  // the six products
      if (KB == 1 || ks < KB / 2)
        __builtin_amdgcn_sched_group_barrier(0x020, 4, 0);  // then the refill's four loads
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) x[j] = KB > 1 ? acc[j][0] + acc[j][1] : acc[j][0];
  };

  // Issue the ring in slot order (pinned against rescheduling) so slot 0 is
  // the oldest load on loop entry.
  auto fill = [&](int step, Slot& s) {
    load_add(step, s);
#pragma unroll
    for (int ks = 0; ks < KB; ++ks)
#pragma unroll
      for (int j = 0; j < 2; ++j) load_piece(tile_base(step), s, j, ks);
    __builtin_amdgcn_sched_barrier(0);
  };
  fill(0, s0);
  fill(min(1, nsteps - 1), s1);
  turn_b(s0);
  // The step count is padded to a multiple of two; a padded step
  // (step >= nsteps) reads a clamped matrix and stores nothing, so the loop
  // body has no early exit.
  for (int step = 0; step < nsteps; step += 2) {
    step_body(step, 0, s0, s1);
    step_body(step + 1, KB > 1 ? 1 : 0, s1, s0);
  }
}

// The frozen rule's per-frame maps as operand tiles, in place over A_t:
// M_t = Diag(alpha_t)(I - A_t / U), element [k][n] = alpha_k (delta_kn -
// A_t[k][n] / U), split into bf16 hi and lo planes (operand_tile_offset).
// One workgroup per frame reads its whole A_t (A is symmetric, so the eight
// k values of a lane slot are two contiguous runs of row n) before any
// thread writes.  Under a split plan the frames from first_split on are the
// sums of plan_splits token-range partials (partial s at A + s *
// part_stride), and `extra` workgroups after the frames (four per split
// frame, a quarter of B_t each) fold the B_t partials of those frames in
// place, as the inverse step does.
template <int DK>
__global__ __launch_bounds__(kThreads)
void frozen_tiles_kernel(float* __restrict__ A, const float* __restrict__ alpha, float inv_u,
                         unsigned first_split, int plan_splits, unsigned extra, size_t part_stride,
                         float* __restrict__ B_part, size_t b_mat, size_t b_stride) {
  constexpr int SLOTS = DK * DK / 8;                          // 8 elements per lane slot
  constexpr int SPT = (SLOTS + kThreads - 1) / kThreads;      // slots per thread
  const int tid = threadIdx.x;
  if (blockIdx.x >= gridDim.x - extra) {  // four workgroups per split frame
    const unsigned e = blockIdx.x - (gridDim.x - extra);
    const size_t f = first_split + e / 4;
    const size_t quarter = b_mat / 4;
    inv::fold_b_partials(B_part + f * b_mat, plan_splits, (e % 4) * quarter,
                         (e % 4 + 1) * quarter, b_stride, tid, kThreads);
    return;
  }
  const int splits = blockIdx.x >= first_split ? plan_splits : 1;
  float* a = A + (size_t)blockIdx.x * DK * DK;
  const float* al = alpha != nullptr ? alpha + (size_t)blockIdx.x * DK : nullptr;
  // Row segment (n, k0 .. k0 + 3) of slot i, half h: the eight k values of a
  // lane slot are two contiguous runs of row n (A is symmetric).  All of a
  // partial's segments are loaded in one memory round trip, and the
  // token-range partials are added in split order.
  auto seg = [&](int i, int h) -> size_t {
    const int sl = tid + kThreads * i;
    const int lane = sl % 64, tile = sl / 64;
    const int nb = tile / (DK / 32), ks = tile % (DK / 32);
    const int n = 16 * nb + lane % 16, g = lane / 16;
    return (size_t)n * DK + 32 * ks + 16 * h + 4 * g;
  };
  float4 r[SPT][2];
#pragma unroll
  for (int i = 0; i < SPT; ++i)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (tid + kThreads * i < SLOTS) r[i][h] = *reinterpret_cast<const float4*>(a + seg(i, h));
  for (int sp = 1; sp < splits; ++sp) {
    float4 x[SPT][2];
#pragma unroll
    for (int i = 0; i < SPT; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (tid + kThreads * i < SLOTS)
          x[i][h] = *reinterpret_cast<const float4*>(a + sp * part_stride + seg(i, h));
#pragma unroll
    for (int i = 0; i < SPT; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (tid + kThreads * i < SLOTS) {
          r[i][h].x += x[i][h].x;
          r[i][h].y += x[i][h].y;
          r[i][h].z += x[i][h].z;
          r[i][h].w += x[i][h].w;
        }
  }
  float v[SPT][8];
#pragma unroll
  for (int i = 0; i < SPT; ++i) {
    const int sl = tid + kThreads * i;
    if (sl >= SLOTS) continue;
    const int lane = sl % 64, tile = sl / 64;
    const int nb = tile / (DK / 32), ks = tile % (DK / 32);
    const int n = 16 * nb + lane % 16, g = lane / 16;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k0 = 32 * ks + 16 * h + 4 * g;
      const float rv[4] = {r[i][h].x, r[i][h].y, r[i][h].z, r[i][h].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = k0 + e;
        const float m = (k == n ? 1.0f : 0.0f) - rv[e] * inv_u;
        v[i][4 * h + e] = al != nullptr ? al[k] * m : m;
      }
    }
  }
  __syncthreads();  // every read of this frame's A_t is done before it is overwritten
  char* t0 = reinterpret_cast<char*>(a);
#pragma unroll
  for (int i = 0; i < SPT; ++i) {
    const int sl = tid + kThreads * i;
    if (sl >= SLOTS) continue;
    const int lane = sl % 64, tile = sl / 64;
    const int nb = tile / (DK / 32), ks = tile % (DK / 32);
    uint32_t hw[4], lw[4];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      const uint32_t hh = pack_bf16x2(v[i][e], v[i][e + 1]);
      hw[e / 2] = hh;
      lw[e / 2] = pack_bf16x2(v[i][e] - bf16_lo(hh), v[i][e + 1] - bf16_hi(hh));
    }
    *reinterpret_cast<u32x4*>(t0 + operand_tile_offset(DK, 0, nb, ks, lane)) =
        u32x4{hw[0], hw[1], hw[2], hw[3]};
    *reinterpret_cast<u32x4*>(t0 + operand_tile_offset(DK, 1, nb, ks, lane)) =
        u32x4{lw[0], lw[1], lw[2], lw[3]};
  }
}

template <int DK, bool DECAY, bool CHUNKED>
hipError_t launch_tiled_k(TiledScanArgs a, int H, hipStream_t stream) {
  a.nwg = (unsigned)H * 2u * (unsigned)(a.DV / 16);
  hipLaunchKernelGGL((scan_tiled_kernel<DK, DECAY, CHUNKED>), dim3(a.nwg), dim3(2 * DK), 0,
                     stream, a);
  return hipGetLastError();
}

template <int DK>
hipError_t launch_tiled_t(const TiledScanArgs& a, int H, bool chunked, hipStream_t stream) {
  if (chunked) return launch_tiled_k<DK, false, true>(a, H, stream);
  if (a.alpha != nullptr) return launch_tiled_k<DK, true, false>(a, H, stream);
  return launch_tiled_k<DK, false, false>(a, H, stream);
}

hipError_t launch_tiled(const TiledScanArgs& a, int H, int d_k, bool chunked, hipStream_t stream) {
  switch (d_k) {
    case 32: return launch_tiled_t<32>(a, H, chunked, stream);
    case 64: return launch_tiled_t<64>(a, H, chunked, stream);
    case 128: return launch_tiled_t<128>(a, H, chunked, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_chunk_sequence_scan(const void* Mt, const float* Jc, const float* text_state,
                                      int F, int H, int d_k, int d_v, int chunk, int offset,
                                      int C, float* S_fwd, float* S_rev, hipStream_t stream) {
  TiledScanArgs a{};
  a.tiles = static_cast<const uint16_t*>(Mt);
  a.add = Jc;
  a.text_state = text_state;
  a.F = F;
  a.DV = d_v;
  a.chunk = chunk;
  a.offset = offset;
  a.mats_per_head = 2 * C;
  a.dir_stride = C;
  a.add_scale = 1.0f;
  a.C = C;
  a.S_fwd = S_fwd;
  a.S_rev = S_rev;
  return launch_tiled(a, H, d_k, true, stream);
}

hipError_t launch_frozen_tiles(float* A, float* B_part, SplitPlan plan, const float* alpha, int F,
                               int H, int d_k, int d_v, int tokens, hipStream_t stream) {
  const long long count = (long long)H * F;
  const int splits = plan.splits > 1 && plan.tail > 0 ? plan.splits : 1;
  const unsigned first_split = splits > 1 ? (unsigned)(count - plan.tail) : (unsigned)count;
  const size_t part_stride = (size_t)plan.tail * d_k * d_k;  // partial p of frame f: f + p * tail
  const size_t b_mat = (size_t)d_v * d_k;
  const size_t b_stride = (size_t)plan.tail * b_mat;
  const unsigned extra = splits > 1 ? 4u * (unsigned)plan.tail : 0u;
  const dim3 grid((unsigned)count + extra);
  const float inv_u = 1.0f / (float)tokens;
#define VDA_FROZEN_TILES(DK)                                                                   \
  hipLaunchKernelGGL(frozen_tiles_kernel<DK>, grid, dim3(kThreads), 0, stream, A, alpha, inv_u, \
                     first_split, splits, extra, part_stride, B_part, b_mat, b_stride)
  switch (d_k) {
    case 32: VDA_FROZEN_TILES(32); break;
    case 64: VDA_FROZEN_TILES(64); break;
    case 128: VDA_FROZEN_TILES(128); break;
    default: return hipErrorInvalidValue;
  }
#undef VDA_FROZEN_TILES
  return hipGetLastError();
}

hipError_t launch_frozen_scan_tiled(const void* M_tiles, const float* Bm, const float* text_state,
                                    int F, int H, int d_k, int d_v, int tokens, float* S_fwd,
                                    float* S_rev, hipStream_t stream) {
  TiledScanArgs a{};
  a.tiles = static_cast<const uint16_t*>(M_tiles);
  a.add = Bm;
  a.text_state = text_state;
  a.F = F;
  a.DV = d_v;
  a.chunk = 1;
  a.offset = 0;
  a.C = F;
  a.mats_per_head = F;
  a.dir_stride = 0;
  a.add_scale = 1.0f / sqrtf((float)tokens);
  a.S_fwd = S_fwd;
  a.S_rev = S_rev;
  return launch_tiled(a, H, d_k, true, stream);
}

hipError_t launch_state_scan_tiled(const void* Inv_tiles, const float* Bm, int F, int H, int d_k,
                                   int d_v, const ScanOptions& o, float* S_fwd, float* S_rev,
                                   hipStream_t stream) {
  if (o.frozen) return hipErrorInvalidValue;
  TiledScanArgs a{};
  a.tiles = static_cast<const uint16_t*>(Inv_tiles);
  a.add = Bm;
  a.alpha = o.alpha;
  a.text_state = o.text_state;
  a.F = F;
  a.DV = d_v;
  a.S_fwd = S_fwd;
  a.S_rev = S_rev;
  return launch_tiled(a, H, d_k, false, stream);
}

}  // namespace vda
