// Device code of step a2, Inv_t = (I + A_t)^{-1} (Eq. 5).
//
// I + A_t is symmetric positive definite with every eigenvalue >= 1 (A_t is
// a Gram matrix weighted by beta >= 0; Appendix A.1), so elimination needs
// no pivoting and every leading block is invertible.
//
// One workgroup inverts one d_k x d_k matrix in fp32 by block sweeps with
// 16 x 16 blocks on v_mfma_f32_16x16x4_f32.  Sweeping block kb, with
// D = M[kb][kb] and the pivot row P_j = M[kb][j], sets
//     M[i][j] -= P_i^T D^{-1} P_j   (i, j != kb),
//     M[kb][j] = D^{-1} P_j,   M[kb][kb] = -D^{-1},
// keeps the matrix symmetric at every step, and leaves -M^{-1} after all of
// them.  So only one block of each symmetric pair is kept: half the
// products, registers and loads of an unsymmetric elimination.  Block {i, j},
// i > j, is held as M[j][i] until block j is swept, which is where it is
// P_i of step j, and as M[i][j] from then on, where it is P_j of step i;
// step j writes the new value P_i^T D^{-1} in that orientation directly.  A
// block's accumulator layout (lane (c, g) holds rows 4g .. 4g+3, column c)
// serves as the B-operand of the block and as the A-operand of its
// transpose, so with R_j = D^{-1} P_j every update takes its operands as they
// lie: M[j][i] -= R_j^T P_i before block j is swept, M[i][j] -= P_i^T R_j
// after, with R_j for the wave's own columns only.
//
// Column j's blocks i = j .. NB-1 belong to one update wave, of which there
// are three (one for d_k <= 64, whose products take less than a pivot
// block).  One more wave, with a SIMD to itself when the compute unit has one
// matrix, inverts the pivot blocks: during step kb, while the update waves
// apply D^{-1} of block kb, it brings diagonal block kb + 1 up
// to date from the published rows and inverts it by scalar Gauss-Jordan, so
// that the chain of 16 pivots per block is all that is serial.  Each step
// ends in one barrier, after which everything the next step reads is
// published in LDS (double buffered): P_j and D^{-1} of that step, and the
// diagonal block after it.
//
// The token-split partials of A_t are summed in split order while loading
// (fold_b_partials does the same for B_t).  All products and sums are fp32.
// Only A_t's blocks on and below the diagonal are read, as contiguous row
// segments.  The result is exactly symmetric off the diagonal blocks.
//
// The 16 x 16 diagonal blocks are symmetric only to the rounding of A_t's own
// operands: with bf16 storage beta * k is rounded to bf16 on one side of the
// product, so A_t[i][j] and A_t[j][i] of one block differ by it.  The sweeps
// take D^{-1} as its own transpose, an unsymmetric elimination would not; the
// two results differ by that rounding (bf16 passes by about 1e-3 of the
// result), and are equally far from 64 bits (B_t Inv_t at 1024 tokens of d_k =
// 128: 2.00e-3 and 2.00e-3; whole passes 3.1e-3 and 3.1e-3).
//
// What bounds it (d_k = 128, shader-clock stamps, one matrix): the pivot
// wave's chain, 8 x (1880 cycles of pivots, 117 each, + 700 for the next
// block's operands and update), under which the update waves' ~60 products
// of 32 cycles a step lie; then 3000 cycles each for loads and stores.  16
// matrices of two partials 20.4 -> 13.8 us, 504 matrices 37.9 -> 27.4, 700
// (100 frames x 7 heads) 46 -> 34, 1536 of d_k = 64 25.6 -> 21.8 (before: an
// unsymmetric elimination of all 64 blocks in four waves, one of which
// inverted the pivot block beside its own products).  With four update
// waves and the pivot wave beside one of them on a SIMD, a pivot block took
// 2900 cycles instead of 1880.
#pragma once

#include <type_traits>

#include "vda_common.h"

namespace vda {
namespace inv {

// Pivot block inverse by scalar Gauss-Jordan: lane (li, lg) holds
// D[4lg + r][li] in d[r] on entry and D^{-1} in the same layout on exit.
// Every cross-lane move is a VALU operation.  The four rows of a lane group
// are pivots in turn; copies of them, kept up to date in all four groups, are
// made once per four pivots by a 16-lane and a 32-lane row swap
// (v_permlane16_swap, v_permlane32_swap), so a pivot step reads its row and
// its pivot (DPP row_newbcast, as are the columns, folded into the
// multiply-adds) from its own lanes.  The reciprocal is the hardware
// estimate refined by one Newton step (error <= 1 ulp); the IEEE division
// sequence would sit on the serial path once per pivot.
template <int G>
__device__ __forceinline__ float row_of_group(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto t = __builtin_amdgcn_permlane16_swap(u, u, false, false);  // [r0 r0 r2 r2], [r1 r1 r3 r3]
  const uint32_t y = (G & 1) ? t[1] : t[0];
  const auto v = __builtin_amdgcn_permlane32_swap(y, y, false, false);  // lower / upper pair
  return __uint_as_float((G & 2) ? v[1] : v[0]);
}

template <int P>
__device__ __forceinline__ float lane_of_row(float x) {  // lane P of each row of 16, in all of them
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x150 + P, 0xf, 0xf, false));
}

// Pivot P = 4 G + E; row[f], f >= E: row 4 G + f in every lane group.
template <int P>
__device__ __forceinline__ void pivot_step(float (&d)[4], float (&row)[4], int li, int lg) {
  constexpr int G = P >> 2, E = P & 3;
  float inv = __builtin_amdgcn_rcpf(lane_of_row<P>(row[E]));
  inv = inv * fmaf(lane_of_row<P>(row[E]), -inv, 2.0f);
  const bool on_col = li == P;
  const float x = on_col ? 1.0f : row[E];
  const float m = on_col ? -1.0f : 0.0f;
  // One fused update for every element off the pivot row, d + column * ns,
  // with ns = -(new pivot row), and in the pivot column (where the column is
  // d) ns = -(1 + inv), which gives -d * inv, the eliminated column.
  const float ns = fmaf(x, -inv, m);
  // x += (lane P of x's row) * ns, one instruction each.  The wait states are
  // those a DPP read needs after a VALU write of its register, whoever wrote
  // it; the rows come first, so that the ones read next are old enough
  // when the block ends.
#define VDA_COL(x) "v_fmac_f32_dpp " x ", " x ", %[ns] row_newbcast:%[p] row_mask:0xf bank_mask:0xf\n\t"
#define VDA_COLS VDA_COL("%[d0]") VDA_COL("%[d1]") VDA_COL("%[d2]") VDA_COL("%[d3]")
#define VDA_D [d0] "+v"(d[0]), [d1] "+v"(d[1]), [d2] "+v"(d[2]), [d3] "+v"(d[3])
  if constexpr (E == 0)
    asm("s_nop 1\n\t" VDA_COL("%[r1]") VDA_COL("%[r2]") VDA_COL("%[r3]") VDA_COLS
        : VDA_D, [r1] "+v"(row[1]), [r2] "+v"(row[2]), [r3] "+v"(row[3]) : [ns] "v"(ns), [p] "n"(P));
  else if constexpr (E == 1)
    asm("s_nop 1\n\t" VDA_COL("%[r2]") VDA_COL("%[r3]") VDA_COLS
        : VDA_D, [r2] "+v"(row[2]), [r3] "+v"(row[3]) : [ns] "v"(ns), [p] "n"(P));
  else if constexpr (E == 2)
    asm("s_nop 1\n\t" VDA_COL("%[r3]") VDA_COLS
        : VDA_D, [r3] "+v"(row[3]) : [ns] "v"(ns), [p] "n"(P));
  else
    asm("s_nop 1\n\t" VDA_COLS : VDA_D : [ns] "v"(ns), [p] "n"(P));
#undef VDA_COL
#undef VDA_COLS
#undef VDA_D
  if (lg == G) d[E] = x * inv;  // the new pivot row
}

template <int G = 0>
__device__ __forceinline__ void invert_pivot_block(float (&d)[4], int li, int lg) {
  float row[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) row[f] = row_of_group<G>(d[f]);
  pivot_step<4 * G>(d, row, li, lg);
  pivot_step<4 * G + 1>(d, row, li, lg);
  pivot_step<4 * G + 2>(d, row, li, lg);
  pivot_step<4 * G + 3>(d, row, li, lg);
  if constexpr (G + 1 < 4) invert_pivot_block<G + 1>(d, li, lg);
}

// Floats of LDS that inverting one matrix takes: two sets of NB published
// blocks, two diagonal blocks, and two 16 x 16 blocks (row stride 20) per
// update wave for the transposes of the output.
__host__ __device__ constexpr int inverse_update_waves(int dk) { return dk == 128 ? 3 : 1; }
__host__ __device__ constexpr int inverse_threads(int dk) { return 64 * (inverse_update_waves(dk) + 1); }
__host__ __device__ constexpr int inverse_lds_floats(int dk) {
  return 2 * (dk / 16) * 256 + 2 * 256 + inverse_update_waves(dk) * 2 * 320;
}

__device__ __forceinline__ floatx4 read_block(const float* b, int lane) {
  return reinterpret_cast<const floatx4*>(b)[lane];
}

__device__ __forceinline__ void write_block(float* b, int lane, floatx4 v) {
  reinterpret_cast<floatx4*>(b)[lane] = v;
}

// Block (i, j), i >= j, of I + A_t, held as M[j][i]: lane (li, lg) holds
// M[16j + 4lg + s][16i + li], which by symmetry is a 16-byte piece of row
// 16i + li.
template <int DK>
__device__ __forceinline__ floatx4 load_block(const float* m, int i, int j, int li, int lg) {
  return *reinterpret_cast<const floatx4*>(m + (size_t)(16 * i + li) * DK + 16 * j + 4 * lg);
}

__device__ __forceinline__ void add_identity(floatx4& b, int li, int lg) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
    if (4 * lg + s == li) b[s] += 1.0f;
}

// Columns of update wave WV.  With NB = 8 three waves share the 36 blocks in
// whole columns (column j has NB - j), 12 each; with fewer blocks one wave
// has them all.
template <int NB, int WV>
struct WaveColumns {
  static constexpr int count = NB == 8 ? (WV == 2 ? 4 : 2) : NB;
  static constexpr int col(int c) {
    if (NB == 8) return WV == 0 ? (c == 0 ? 0 : 4) : WV == 1 ? (c == 0 ? 1 : 3) : (c == 0 ? 2 : 4 + c);
    return c;
  }
};

// One update wave.
template <int DK, int WV, InvLayout OUT>
struct UpdateWave {
  static constexpr int NB = DK / 16;
  using Cols = WaveColumns<NB, WV>;
  static constexpr int NC = Cols::count;
  static constexpr int CMIN = Cols::col(0);

  floatx4 a[NC][NB];  // blocks {i, col(c)}, i >= col(c)
  float* pub;         // [2][NB][256] published blocks
  float* diag;        // [2][256] the next diagonal block
  int lane, li, lg;

  __device__ __forceinline__ void load(const float* A_part, int splits, size_t part_stride) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int i = Cols::col(c); i < NB; ++i) a[c][i] = load_block<DK>(A_part, i, Cols::col(c), li, lg);
    // Further token ranges of a split frame, two per memory round trip.
    for (int s = 1; s < splits; s += 2) {
      const float* m0 = A_part + s * part_stride;
      const bool two = s + 1 < splits;
      const float* m1 = two ? m0 + part_stride : m0;
      floatx4 x[NC][NB], y[NC][NB];
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = Cols::col(c); i < NB; ++i) {
          x[c][i] = load_block<DK>(m0, i, Cols::col(c), li, lg);
          y[c][i] = load_block<DK>(m1, i, Cols::col(c), li, lg);
        }
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = Cols::col(c); i < NB; ++i) {
          a[c][i] += x[c][i];
          if (two) a[c][i] += y[c][i];
        }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) add_identity(a[c][Cols::col(c)], li, lg);
  }

  // Publishes what step KB reads of this wave's columns: P_j of that step and
  // the diagonal block after its pivot.
  template <int KB>
  __device__ __forceinline__ void publish() const {
    if constexpr (KB < NB) {
      float* pb = pub + (KB & 1) * (NB * 256);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int C = Cols::col(c);
        if (C < KB) write_block(pb + C * 256, lane, a[c][KB]);
        if (C == KB) {
#pragma unroll
          for (int i = KB + 1; i < NB; ++i) write_block(pb + i * 256, lane, a[c][i]);
        }
        if (C == KB + 1) write_block(diag + (KB & 1) * 256, lane, a[c][C]);
      }
    }
  }

  template <int KB>
  __device__ __forceinline__ void step() {
    const float* pb = pub + (KB & 1) * (NB * 256);
    const floatx4 d = read_block(pb + KB * 256, lane);  // D^{-1}
    floatx4 p[NB];
#pragma unroll
    for (int i = CMIN; i < NB; ++i)
      if (i != KB) p[i] = read_block(pb + i * 256, lane);
    const floatx4 z = {0.f, 0.f, 0.f, 0.f};
    // -R_C of the wave's columns (D^{-1} is symmetric: d serves as its
    // A-operand).
    floatx4 r[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) r[c] = z;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if (Cols::col(c) != KB)
          r[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(-d[s], p[Cols::col(c)][s], r[c], 0, 0, 0);
    floatx4 t[NB];  // the new blocks of column KB, if it is one of the wave's
#pragma unroll
    for (int i = KB + 1; i < NB; ++i) t[i] = z;
    // Products over the blocks in turn, so that the four of one block are
    // far apart.  The diagonal block of the next pivot is left to the pivot
    // wave.
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int C = Cols::col(c);
#pragma unroll
        for (int i = C; i < NB; ++i) {
          if (i == KB || (i == C && C == KB + 1)) continue;
          if (C == KB)
            t[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c][i][s], d[s], t[i], 0, 0, 0);
          else if (C > KB)
            a[c][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(r[c][s], p[i][s], a[c][i], 0, 0, 0);
          else
            a[c][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(p[i][s], r[c][s], a[c][i], 0, 0, 0);
        }
      }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int C = Cols::col(c);
      if (C == KB) {
#pragma unroll
        for (int i = KB + 1; i < NB; ++i) a[c][i] = t[i];
        a[c][KB] = -d;
      }
      if (C < KB) a[c][KB] = -r[c];
    }
    publish<KB + 1>();
    if constexpr (KB + 1 < NB) {
      lds_barrier();
      step<KB + 1>();
    }
  }

  // Column C of the result X = -M to Inv: block {i, C} as it is held
  // (M[i][C]) and, through this wave's LDS, transposed.
  template <int C>
  __device__ __forceinline__ void store_column(const floatx4 (&m)[NB], float* Inv, float* tp) const {
    char* t0 = reinterpret_cast<char*>(Inv);
    u32x2 hi[NB], lo[NB];
#pragma unroll
    for (int i = C; i < NB; ++i) {
      const floatx4 x = -m[i];
      floatx4 xt;  // X[16i + li][16C + 4lg + r]
      if (i > C) {
        float* b = tp + ((i - C) & 1) * 320;
#pragma unroll
        for (int s = 0; s < 4; ++s) b[(4 * lg + s) * 20 + li] = x[s];
        __builtin_amdgcn_wave_barrier();
        xt = *reinterpret_cast<const floatx4*>(b + li * 20 + 4 * lg);
        __builtin_amdgcn_wave_barrier();
      }
      if constexpr (OUT == InvLayout::kF32Tiles) {
        // Block (k, n) is lane-ordered piece (nb = n, chunk = k).
        floatx4* t = reinterpret_cast<floatx4*>(Inv) + lane;
        t[(C * NB + i) * 64] = x;
        if (i > C) t[(i * NB + C) * 64] = xt;
      } else if constexpr (OUT == InvLayout::kBf16Tiles) {
        // Split-bf16 operand tiles (operand_tile_offset): block (k, n) at lane
        // (li, lg) holds X[16k + 4lg + r][16n + li], which is half k % 2 of
        // that lane's 16 bytes of tile (nb = n, ks = k / 2).
        split_block(x, hi[i], lo[i]);
        if ((i & 1) == 1 && i > C) {
          char* t = t0 + operand_tile_offset(DK, 0, C, i / 2, lane);
          *reinterpret_cast<u32x4*>(t) = u32x4{hi[i - 1][0], hi[i - 1][1], hi[i][0], hi[i][1]};
          *reinterpret_cast<u32x4*>(t + (size_t)DK * DK * 2) =
              u32x4{lo[i - 1][0], lo[i - 1][1], lo[i][0], lo[i][1]};
        } else if ((i & 1) == 1) {  // the diagonal block alone in its pair
          char* t = t0 + operand_tile_offset(DK, 0, C, i / 2, lane) + 8;
          *reinterpret_cast<u32x2*>(t) = hi[i];
          *reinterpret_cast<u32x2*>(t + (size_t)DK * DK * 2) = lo[i];
        }
        if (i > C) {
          u32x2 ht, lt;
          split_block(xt, ht, lt);
          char* t = t0 + operand_tile_offset(DK, 0, i, C / 2, lane) + (C & 1) * 8;
          *reinterpret_cast<u32x2*>(t) = ht;
          *reinterpret_cast<u32x2*>(t + (size_t)DK * DK * 2) = lt;
        }
      } else {
        *reinterpret_cast<floatx4*>(Inv + (size_t)(16 * C + li) * DK + 16 * i + 4 * lg) = x;
        if (i > C)
          *reinterpret_cast<floatx4*>(Inv + (size_t)(16 * i + li) * DK + 16 * C + 4 * lg) = xt;
      }
    }
  }

  static __device__ __forceinline__ void split_block(floatx4 x, u32x2& hi, u32x2& lo) {
    const uint32_t h01 = pack_bf16x2(x[0], x[1]), h23 = pack_bf16x2(x[2], x[3]);
    hi = u32x2{h01, h23};
    lo = u32x2{pack_bf16x2(x[0] - bf16_lo(h01), x[1] - bf16_hi(h01)),
               pack_bf16x2(x[2] - bf16_lo(h23), x[3] - bf16_hi(h23))};
  }

  __device__ __forceinline__ void run(const float* A_part, int splits, size_t part_stride,
                                      float* Inv, float* tp) {
    load(A_part, splits, part_stride);
    publish<0>();
    lds_barrier();
    step<0>();
    store_column<Cols::col(0)>(a[0], Inv, tp);
    if constexpr (NC > 1) store_column<Cols::col(1)>(a[1], Inv, tp);
    if constexpr (NC > 2) store_column<Cols::col(2)>(a[2], Inv, tp);
    if constexpr (NC > 3) store_column<Cols::col(3)>(a[3], Inv, tp);
  }
};

// The pivot wave: D^{-1} of every block step, one step ahead of the update
// waves.
template <int DK>
__device__ __forceinline__ void run_pivot_wave(const float* A_part, int splits, size_t part_stride,
                                               float* pub, const float* diag, int lane) {
  constexpr int NB = DK / 16;
  const int li = lane & 15, lg = lane >> 4;
  // The pivot blocks are this matrix's critical path: the SIMD's arbiter
  // prefers this wave over the update waves it shares the SIMD with.
  __builtin_amdgcn_s_setprio(2);
  floatx4 d = load_block<DK>(A_part, 0, 0, li, lg);
  for (int s = 1; s < splits; ++s) d += load_block<DK>(A_part + s * part_stride, 0, 0, li, lg);
  add_identity(d, li, lg);
  for (int kb = 0; kb < NB; ++kb) {
    float e[4] = {d[0], d[1], d[2], d[3]};
    invert_pivot_block(e, li, lg);
    const floatx4 inv = {e[0], e[1], e[2], e[3]};
    write_block(pub + ((kb & 1) * NB + kb) * 256, lane, inv);
    lds_barrier();  // step kb is published
    if (kb + 1 < NB) {
      d = read_block(diag + (kb & 1) * 256, lane);
      const floatx4 p = read_block(pub + ((kb & 1) * NB + kb + 1) * 256, lane);
      floatx4 r = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 4; ++s) r = __builtin_amdgcn_mfma_f32_16x16x4f32(-inv[s], p[s], r, 0, 0, 0);
#pragma unroll
      for (int s = 0; s < 4; ++s) d = __builtin_amdgcn_mfma_f32_16x16x4f32(r[s], p[s], d, 0, 0, 0);
    }
  }
  __builtin_amdgcn_s_setprio(0);
}

// Sum the token-split partials of B_t into the first one (in place, in
// partial order) over the element range [lo, hi) of the matrix; all threads
// of the workgroup take part.  Each thread holds up to four 16-byte pieces,
// and the pieces of the first four partials are loaded together, so up to
// four take one memory round trip (bf16 storage has no more); each further
// one (fp32 storage plans up to eight ranges) takes another.
__device__ __forceinline__ void fold_b_partials(float* b0, int splits, size_t lo, size_t hi,
                                                size_t b_stride, int tid, int nthreads) {
  const size_t step = (size_t)nthreads * 4;
  for (size_t idx0 = lo + (size_t)tid * 4; idx0 < hi; idx0 += 4 * step) {
    floatx4 a[4][4];  // [partial][piece]
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const size_t idx = idx0 + e * step;
        a[s][e] = s < splits && idx < hi
                      ? *reinterpret_cast<const floatx4*>(b0 + s * b_stride + idx)
                      : floatx4{0.f, 0.f, 0.f, 0.f};
      }
    floatx4 sum[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) sum[e] = ((a[0][e] + a[1][e]) + a[2][e]) + a[3][e];
    for (int s = 4; s < splits; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const size_t idx = idx0 + e * step;
        if (idx < hi) sum[e] += *reinterpret_cast<const floatx4*>(b0 + s * b_stride + idx);
      }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const size_t idx = idx0 + e * step;
      if (idx < hi) *reinterpret_cast<floatx4*>(b0 + idx) = sum[e];
    }
  }
}

// Inverts one matrix with the inverse_threads(DK) threads of the workgroup;
// `lds` is inverse_lds_floats(DK) floats, 16-byte aligned.  The matrix is the
// sum of `splits` partials at A_part + s * part_stride + base; the result
// goes to Inv + base (which may alias the first partial: every wave has read
// its blocks before the first barrier), d_k * d_k * 4 bytes in layout OUT.
template <int DK, InvLayout OUT>
__device__ __forceinline__ void invert_matrix(const float* A_part, int splits, size_t part_stride,
                                              size_t base, float* Inv, float* lds, int tid) {
  constexpr int NB = DK / 16, W = inverse_update_waves(DK);
  float* pub = lds;
  float* diag = pub + 2 * NB * 256;
  const int lane = tid & 63;
  // The wave's role; 256 workgroups apart, likely on the same compute unit,
  // the roles lie on different SIMDs, so that pivot waves do not share one.
  const int wave = __builtin_amdgcn_readfirstlane((tid >> 6) + (W == 3 ? blockIdx.x >> 8 : 0)) % (W + 1);
  float* tp = diag + 2 * 256 + wave * 640;
  const float* a = A_part + base;
  float* out = Inv + base;
  auto update = [&](auto wv) {
    UpdateWave<DK, decltype(wv)::value, OUT> u;
    u.pub = pub;
    u.diag = diag;
    u.lane = lane;
    u.li = lane & 15;
    u.lg = lane >> 4;
    u.run(a, splits, part_stride, out, tp);
  };
  // Every branch takes the same NB barriers.
  if (wave == W)
    run_pivot_wave<DK>(a, splits, part_stride, pub, diag, lane);
  else if (wave == 0)
    update(std::integral_constant<int, 0>{});
  else if (wave == 1)
    update(std::integral_constant<int, 1 % W>{});
  else
    update(std::integral_constant<int, 2 % W>{});
}

}  // namespace inv
}  // namespace vda
