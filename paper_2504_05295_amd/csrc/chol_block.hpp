// The 64 x 64 diagonal block of the Cholesky factorisations: L11 = chol(C11) and W11 = L11^-1, by three waves.
//
// The block is the one sequential part of a step: every panel of every factorisation waits for it.  It is taken in four
// steps of 16 columns, each a 16 x 16 elimination on the vector unit (lane = row; the chain from one pivot to the next
// is a broadcast within the row of lanes, a reciprocal, a product and a multiply-add) followed by rank-16 products
// on the fp32 matrix unit:
//   step s    eliminate tile (s, s), which gives W_ss = L_ss^-1 (forward substitution on the identity, in the same column steps)
//             L_is = T_is W_ss^T (i > s);   T_ij -= L_is L_js^T (i >= j > s)
//             row s of the inverse: W_sj = -W_ss sum_{j <= k < s} L_sk W_kj
// An fp32 matrix instruction keeps its SIMD's vector unit busy too (measured: 44 + 4 n cycles for one and n multiply-adds of
// the same wave), so only the products that lead to the next diagonal tile stand in the eliminating wave:
//   chain_wave    the eliminations, L_{s+1,s} and the last update of T_{s+1,s+1}
//   update_wave   the other L_is (and L11 for memory), the other updates; hands T_{s+1,s}, T_{s+1,s+1} to the chain
//   inverse_wave  the rows of the inverse
// on three SIMDs.  Measured in one workgroup on an idle GPU: 3.6 us a block; 9.2-10.2 us column by column over all 64 columns, with
// one wave eliminating and two following it; 5.7 us with everything in one wave.  The eliminations are 64 columns of 16 to 23
// instructions, about 2.4 us of it; the rest is the three hand-overs between steps, the first loads and the last row of W.
// A step: 256 x 256 r = 64 in fp32 75.2 -> 70.1 us, 1111 x 1733 r = 139 in fp32 190.5 -> 170.4, 2048 x 2048 r = 512 in bf16 mode 302 ->
// 285, Double Dion 4096 x 4096 r = 256 and 1024 1368 -> 1238.
// Tiles pass from wave to wave in their own places of the block in LDS, announced by counters: LDS
// operations of one wave are processed in issue order, so data stored before a counter is visible to whoever sees
// the counter.
// Tile layout in registers: lane l, register v holds element [l % 16][4 (l / 16) + v], a 16-byte LDS access.  With v =
// 0..3 as the four k-steps of a 16 x 16 product this is at once the layout of both operands and of the result: the instruction
// given the registers of X and Y adds Y X^T to its accumulator, in this very layout.  The inverse needs products
// without the transposition, so its wave keeps it transposed (V_jk = W_kj^T) until it is written out; a diagonal
// tile is transposed by a product with the identity.
#pragma once
#include <type_traits>
#include <utility>

#include "internal.hpp"

namespace dion {

typedef __attribute__((address_space(3))) float lds_float;
typedef __attribute__((address_space(3))) f32x4_t lds_f32x4;

constexpr int CB = CHOL_NB;   // 64
constexpr int CBP = CB + 4;   // LDS row stride (floats): conflict-free 16-byte reads

namespace chol_block {

// compile-time loop: the body sees its index as a constant, so register arrays are indexed statically
template <int B, int... Is, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, Is...>, F&& f) {
  (f(std::integral_constant<int, B + Is>{}), ...);
}
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) static_for_impl<B>(std::make_integer_sequence<int, E - B>{}, f);
}

// x of lane SRC of this lane's row of sixteen
template <int SRC>
__device__ __forceinline__ float row_bcast(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x150 + SRC, 0xf, 0xf, true));
}
// acc + Y X^T
__device__ __forceinline__ f32x4_t mm(f32x4_t acc, f32x4_t Y, f32x4_t X) {
#pragma unroll
  for (int v = 0; v < 4; ++v) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(X[v], Y[v], acc, 0, 0, 0);
  return acc;
}
// the same on a dependent chain half as long
__device__ __forceinline__ f32x4_t mm_short(f32x4_t acc, f32x4_t Y, f32x4_t X) {
  f32x4_t b = {0.f, 0.f, 0.f, 0.f};
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(X[0], Y[0], acc, 0, 0, 0);
  b = __builtin_amdgcn_mfma_f32_16x16x4f32(X[1], Y[1], b, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(X[2], Y[2], acc, 0, 0, 0);
  b = __builtin_amdgcn_mfma_f32_16x16x4f32(X[3], Y[3], b, 0, 0, 0);
  return acc + b;
}
// y[q] = x of the lanes of row q of sixteen, in every row
__device__ __forceinline__ void row_copies(float (&y)[4], float xf) {
  const unsigned x = __float_as_uint(xf);
  const auto half = __builtin_amdgcn_permlane32_swap(x, x, false, false);        // rows (0 1 0 1), (2 3 2 3)
  const auto lo = __builtin_amdgcn_permlane16_swap(half[0], half[0], false, false);   // rows (0 0 0 0), (1 1 1 1)
  const auto hi = __builtin_amdgcn_permlane16_swap(half[1], half[1], false, false);   // rows (2 2 2 2), (3 3 3 3)
  y[0] = __uint_as_float(lo[0]);
  y[1] = __uint_as_float(lo[1]);
  y[2] = __uint_as_float(hi[0]);
  y[3] = __uint_as_float(hi[1]);
}
// the whole row of the tile in every lane
__device__ __forceinline__ void spread(float (&a)[16], const f32x4_t& T) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    float y[4];
    row_copies(y, T[v]);
#pragma unroll
    for (int q = 0; q < 4; ++q) a[4 * q + v] = y[q];
  }
}

// One column of an elimination: a[k] += f a_j of lane k for k > j, w[v] += f w[v] of lane j, "of lane" within the row of sixteen,
// and the next column's pivot and its reciprocal.  f: 0 in the lanes up to j, else -a_j / pivot; without RANK it comes as a_j and
// is multiplied here.  The broadcast is the multiply-add's own data-parallel operand, which the compiler would leave as
// a move in front of it, twice the instructions; hence by hand.
// A register that a vector instruction writes may be such an operand only with two other instructions or wait states in
// between.  The hardware does not check that; the compiler does, for its own instructions only, and it may put a copy of
// any operand right in front of a statement.  So it holds inside the statement, whatever stands before it: a whole column is
// one statement, that begins with two wait states, and behind a[j + 1], which the next pivot's broadcast reads, come two
// other instructions.  (Without RANK the first wait state is also the one that the product needs behind the reciprocal, and the
// product is the second.)
#define DION_BCAST(OP, D, S, LANE) OP " " D ", " S " row_newbcast:" #LANE " row_mask:0xf bank_mask:0xf\n\t"
#define DION_A(J, K) DION_BCAST("v_fmac_f32_dpp", "%[a" #K "]", "%[a" #J "], %[f]", K)
#define DION_W(J, V) DION_BCAST("v_fmac_f32_dpp", "%[w" #V "]", "%[w" #V "], %[f]", J)
#define DION_FROM_15(J) DION_A(J, 15)
#define DION_FROM_14(J) DION_A(J, 14) DION_FROM_15(J)
#define DION_FROM_13(J) DION_A(J, 13) DION_FROM_14(J)
#define DION_FROM_12(J) DION_A(J, 12) DION_FROM_13(J)
#define DION_FROM_11(J) DION_A(J, 11) DION_FROM_12(J)
#define DION_FROM_10(J) DION_A(J, 10) DION_FROM_11(J)
#define DION_FROM_9(J) DION_A(J, 9) DION_FROM_10(J)
#define DION_FROM_8(J) DION_A(J, 8) DION_FROM_9(J)
#define DION_FROM_7(J) DION_A(J, 7) DION_FROM_8(J)
#define DION_FROM_6(J) DION_A(J, 6) DION_FROM_7(J)
#define DION_FROM_5(J) DION_A(J, 5) DION_FROM_6(J)
#define DION_FROM_4(J) DION_A(J, 4) DION_FROM_5(J)
#define DION_FROM_3(J) DION_A(J, 3) DION_FROM_4(J)
#define DION_FROM_2(J) DION_A(J, 2) DION_FROM_3(J)
#define DION_RCP "v_rcp_f32 %[rcp], %[piv]\n\t"
#define DION_CHAIN(J, K)                                                                                                      \
  DION_A(J, K) DION_W(J, 0) DION_W(J, 1) DION_BCAST("v_mov_b32_dpp", "%[piv]", "%[a" #K "]", K) DION_W(J, 2) DION_W(J, 3)
#define DION_OPERANDS                                                                                                         \
  [a0] "+v"(a[0]), [a1] "+v"(a[1]), [a2] "+v"(a[2]), [a3] "+v"(a[3]), [a4] "+v"(a[4]), [a5] "+v"(a[5]), [a6] "+v"(a[6]),      \
      [a7] "+v"(a[7]), [a8] "+v"(a[8]), [a9] "+v"(a[9]), [a10] "+v"(a[10]), [a11] "+v"(a[11]), [a12] "+v"(a[12]),             \
      [a13] "+v"(a[13]), [a14] "+v"(a[14]), [a15] "+v"(a[15]), [w0] "+v"(w0), [w1] "+v"(w1), [w2] "+v"(w2), [w3] "+v"(w3),    \
      [f] "+v"(f), [piv] "=&v"(piv), [rcp] "+v"(rcp)
#define DION_COLUMN(J, K, REST)                                                                                               \
  if constexpr (COL == J) {                                                                                                   \
    if constexpr (RANK) asm("s_nop 1\n\t" DION_CHAIN(J, K) REST : DION_OPERANDS);                                             \
    else asm("s_nop 0\n\tv_mul_f32_e64 %[f], -%[f], %[rcp]\n\t" DION_CHAIN(J, K) REST : DION_OPERANDS);                       \
  }
template <bool RANK, int COL>
__device__ __forceinline__ void column(float (&a)[16], f32x4_t& w, float f, float& piv, float& rcp) {
  float w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3];
  DION_COLUMN(0, 1, DION_RCP DION_FROM_2(0))
  DION_COLUMN(1, 2, DION_RCP DION_FROM_3(1))
  DION_COLUMN(2, 3, DION_RCP DION_FROM_4(2))
  DION_COLUMN(3, 4, DION_RCP DION_FROM_5(3))
  DION_COLUMN(4, 5, DION_RCP DION_FROM_6(4))
  DION_COLUMN(5, 6, DION_RCP DION_FROM_7(5))
  DION_COLUMN(6, 7, DION_RCP DION_FROM_8(6))
  DION_COLUMN(7, 8, DION_RCP DION_FROM_9(7))
  DION_COLUMN(8, 9, DION_RCP DION_FROM_10(8))
  DION_COLUMN(9, 10, DION_RCP DION_FROM_11(9))
  DION_COLUMN(10, 11, DION_RCP DION_FROM_12(10))
  DION_COLUMN(11, 12, DION_RCP DION_FROM_13(11))
  DION_COLUMN(12, 13, DION_RCP DION_FROM_14(12))
  DION_COLUMN(13, 14, DION_RCP DION_FROM_15(13))
  DION_COLUMN(14, 15, "")
  w = f32x4_t{w0, w1, w2, w3};   // (column 15 has no rows below it)
}
#undef DION_BCAST
#undef DION_A
#undef DION_W
#undef DION_FROM_15
#undef DION_FROM_14
#undef DION_FROM_13
#undef DION_FROM_12
#undef DION_FROM_11
#undef DION_FROM_10
#undef DION_FROM_9
#undef DION_FROM_8
#undef DION_FROM_7
#undef DION_FROM_6
#undef DION_FROM_5
#undef DION_FROM_4
#undef DION_FROM_3
#undef DION_FROM_2
#undef DION_RCP
#undef DION_CHAIN
#undef DION_OPERANDS
#undef DION_COLUMN

typedef __attribute__((address_space(3))) volatile int lds_counter;
enum { W_DONE = 0, T_DONE, L_DONE, SUM_DONE, COUNTERS };   // all zero when a block starts

__device__ __forceinline__ void wait_for(lds_counter* n, int value) {   // (every counter gets there: the waits form no cycle)
  while (*n < value) {}
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void announce(lds_counter* n, int value) {
  asm volatile("" ::: "memory");
  *n = value;
}
__device__ __forceinline__ lds_f32x4* tile_at(lds_float* S, int i, int j, int lane) {
  return (lds_f32x4*)(S + (16 * i + (lane & 15)) * CBP + 16 * j + 4 * (lane >> 4));
}
// tile (i, j) of W from its transpose
__device__ __forceinline__ void put_transposed(lds_float* S, int i, int j, int lane, const f32x4_t& V) {
#pragma unroll
  for (int v = 0; v < 4; ++v) S[(16 * i + 4 * (lane >> 4) + v) * CBP + 16 * j + (lane & 15)] = V[v];
}
__device__ __forceinline__ f32x4_t unit_tile(int lane) {
  f32x4_t one;
#pragma unroll
  for (int v = 0; v < 4; ++v) one[v] = (lane & 15) == 4 * (lane >> 4) + v ? 1.f : 0.f;
  return one;
}
constexpr f32x4_t ZERO = {0.f, 0.f, 0.f, 0.f};
// last row of the inverse, column tile j: from the sum that inverse_wave has left in the tile's place
__device__ __forceinline__ void last_row_tile(lds_float* S, int j, int lane, const f32x4_t& W3) {
  const f32x4_t sum = *tile_at(S, 3, j, lane);
  put_transposed(S, 3, j, lane, mm_short(ZERO, sum, W3));
}

// S: the block (row-major in LDS, stride CBP; its lower triangle), which W11 replaces, with zeros above the diagonal; complete when
// all three waves are through.  report: a pivot outside (piv_lo, piv_hi) is reported to *status, unless a
// code is there already (an earlier stage failed).
// RANK (the factorisation that tolerates linearly dependent columns): a column whose pivot is not above its threshold
// (thr of lane j: a fraction of the Gram matrix' original diagonal entry) is dependent on the columns before it: it eliminates
// nothing, so that the factorisation goes on as if it were not there, and becomes a zero column of L and a zero row and
// column of W.  nullmask[j] (if given) records the decision.
template <bool RANK>
__device__ __forceinline__ void chain_wave(lds_float* S, lds_counter* sync, int lane, float piv_lo, float piv_hi, bool report,
                                           int* status, float thr, int* nullmask) {
  const int c = lane & 15;
  float thr_row[4] = {0.f, 0.f, 0.f, 0.f}, pivots[4];
  if constexpr (RANK) row_copies(thr_row, thr);
  f32x4_t diag = *tile_at(S, 0, 0, lane), sub = *tile_at(S, 1, 0, lane), next = *tile_at(S, 1, 1, lane);
  const f32x4_t one = unit_tile(lane);
  static_for<0, 4>([&](auto sc) __attribute__((always_inline)) {
    constexpr int s = decltype(sc)::value;
    float a[16];
    spread(a, diag);
    f32x4_t w = one;
    float piv_lane = 0.f, piv = row_bcast<0>(a[0]), rcp = __builtin_amdgcn_rcpf(piv);
    static_for<0, 16>([&](auto jc) __attribute__((always_inline)) {
      constexpr int j = decltype(jc)::value;
      const float piv_j = piv;
      float f = c > j ? a[j] : 0.f;
      if constexpr (RANK) {
        f = -f * rcp;
        f = piv > row_bcast<j>(thr_row[s]) ? f : 0.f;
      }
      column<RANK, j>(a, w, f, piv, rcp);
      piv_lane = c == j ? piv_j : piv_lane;
      if constexpr (j == 11 && s < 3) {
        // (s = 0: update_wave has the block in its registers, tile (0, 0) may be written; else the next step's tiles,
        // whose reads are in flight across the last columns)
        wait_for(sync + T_DONE, s + 1);
        if constexpr (s > 0) {
          sub = *tile_at(S, s + 1, s, lane);
          next = *tile_at(S, s + 1, s + 1, lane);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    float rs = __builtin_amdgcn_rsqf(piv_lane);
    rs = rs * (1.5f - 0.5f * piv_lane * rs * rs);   // one Newton step on the hardware estimate
    if constexpr (RANK) rs = piv_lane > thr_row[s] ? rs : 0.f;
    pivots[s] = piv_lane;
    w *= rs;
    *tile_at(S, s, s, lane) = w;
    announce(sync + W_DONE, s + 1);
    if constexpr (s < 3) {
      const f32x4_t l = mm_short(ZERO, sub, w);
      diag = next - mm_short(ZERO, l, l);   // (the sum by itself: with `next` in the accumulator its parts are rounded at next's size)
    } else {
      wait_for(sync + SUM_DONE, 1);
      last_row_tile(S, 2, lane, w);
    }
  });
  if (report) {
    bool bad = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool dependent = RANK && !(pivots[i] > thr_row[i]);
      bad = bad || !(pivots[i] == pivots[i]) || (!dependent && !(pivots[i] > piv_lo && pivots[i] < piv_hi));   // a NaN pivot is no dependent column
      if (RANK && nullmask && lane < 16) nullmask[16 * i + c] = dependent ? 1 : 0;
    }
    if (__ballot(bad) != 0 && lane == 0 && *status == 0) *status = ST_BREAKDOWN;
  }
}

// Lout: L11 goes there (leading dimension ld), if given.
__device__ __forceinline__ void update_wave(lds_float* S, lds_counter* sync, int lane, float* Lout, long long ld) {
  const int c = lane & 15, g = lane >> 4;
  f32x4_t T[4][4], L[4][4];
  static_for<0, 4>([&](auto ic) __attribute__((always_inline)) {
    constexpr int i = decltype(ic)::value;
    static_for<0, i + 1>([&](auto jc) __attribute__((always_inline)) { T[i][decltype(jc)::value] = *tile_at(S, i, decltype(jc)::value, lane); });
    // (diagonal tiles: the upper triangle is the lower one's mirror image; L_ii = T_ii W_ii^T wants it)
    f32x4_t mirror;
#pragma unroll
    for (int v = 0; v < 4; ++v) mirror[v] = S[(16 * i + 4 * g + v) * CBP + 16 * i + c];
#pragma unroll
    for (int v = 0; v < 4; ++v) T[i][i][v] = 4 * g + v > c ? mirror[v] : T[i][i][v];
  });
  announce(sync + T_DONE, 1);   // (reads before it have been issued, and are processed before it)
  static_for<0, 4>([&](auto qc) __attribute__((always_inline)) {
    constexpr int q = decltype(qc)::value;
    wait_for(sync + W_DONE, q + 1);
    const f32x4_t W = *tile_at(S, q, q, lane);
    static_for<q + 1, 4>([&](auto ic) __attribute__((always_inline)) { L[decltype(ic)::value][q] = mm(ZERO, T[decltype(ic)::value][q], W); });
    // (the chain has read tiles (q + 1, q) and (q + 1, q + 1) before it announced W_qq)
    if constexpr (q < 2) {
      T[q + 2][q + 1] -= mm(ZERO, L[q + 2][q], L[q + 1][q]);
      T[q + 2][q + 2] -= mm(ZERO, L[q + 2][q], L[q + 2][q]);
      *tile_at(S, q + 2, q + 1, lane) = T[q + 2][q + 1];
      *tile_at(S, q + 2, q + 2, lane) = T[q + 2][q + 2];
      announce(sync + T_DONE, q + 2);
    }
    if constexpr (q < 3) {
      static_for<q + 1, 4>([&](auto ic) __attribute__((always_inline)) { *tile_at(S, decltype(ic)::value, q, lane) = L[decltype(ic)::value][q]; });
      announce(sync + L_DONE, q + 1);
      // the rest of the updates; T_{q+1,q+1} once more, for its L
      T[q + 1][q + 1] -= mm(ZERO, L[q + 1][q], L[q + 1][q]);
      if constexpr (q == 0)
        static_for<1, 4>([&](auto jc) __attribute__((always_inline)) { T[3][decltype(jc)::value] -= mm(ZERO, L[3][0], L[decltype(jc)::value][0]); });
    } else {
      wait_for(sync + SUM_DONE, 1);
      last_row_tile(S, 1, lane, W);
    }
    if (Lout) {
      f32x4_t d = mm(ZERO, T[q][q], W);
#pragma unroll
      for (int v = 0; v < 4; ++v) d[v] = 4 * g + v > c ? 0.f : d[v];
      static_for<0, 4>([&](auto jc) __attribute__((always_inline)) {
        constexpr int j = decltype(jc)::value;
        f32x4_t x = ZERO;
        if constexpr (j < q) x = L[q][j];
        else if constexpr (j == q) x = d;
        *(f32x4_t*)(Lout + (16 * q + c) * ld + 16 * j + 4 * g) = x;
      });
    }
  });
}

__device__ __forceinline__ void inverse_wave(lds_float* S, lds_counter* sync, int lane) {
  f32x4_t V[3][3], Sum[3];
  const f32x4_t one = unit_tile(lane);
  static_for<0, 4>([&](auto qc) __attribute__((always_inline)) {
    constexpr int q = decltype(qc)::value;
    wait_for(sync + W_DONE, q + 1);
    const f32x4_t W = *tile_at(S, q, q, lane);
    // row q: W_qj = -W_qq sum_j, from the sums of the tiles of L and of the rows above
    if constexpr (q < 3) {
      static_for<0, q>([&](auto jc) __attribute__((always_inline)) {
        constexpr int j = decltype(jc)::value;
        V[j][q] = mm(ZERO, Sum[j], W);
        put_transposed(S, q, j, lane, V[j][q]);
      });
      V[q][q] = mm(ZERO, one, W);
      // the sums of the next row, negated
      wait_for(sync + L_DONE, q + 1);
      f32x4_t Lrow[3];
      static_for<0, q + 1>([&](auto kc) __attribute__((always_inline)) { Lrow[decltype(kc)::value] = -*tile_at(S, q + 1, decltype(kc)::value, lane); });
      static_for<0, q + 1>([&](auto jc) __attribute__((always_inline)) {
        constexpr int j = decltype(jc)::value;
        Sum[j] = ZERO;
        static_for<j, q + 1>([&](auto kc) __attribute__((always_inline)) { Sum[j] = mm(Sum[j], V[j][decltype(kc)::value], Lrow[decltype(kc)::value]); });
      });
      if constexpr (q == 2) {   // the last row is shared among the three waves
        *tile_at(S, 3, 1, lane) = Sum[1];
        *tile_at(S, 3, 2, lane) = Sum[2];
        announce(sync + SUM_DONE, 1);
      }
      // zeros above the diagonal
      static_for<q + 1, 4>([&](auto jc) __attribute__((always_inline)) { *tile_at(S, q, decltype(jc)::value, lane) = ZERO; });
    } else {
      put_transposed(S, 3, 0, lane, mm_short(ZERO, Sum[0], W));
    }
  });
}

// All three, as waves 0 to 2 of a workgroup (other waves return at once).  sync: COUNTERS words of LDS, zero and visible
// before the call; a barrier has to follow.
template <bool RANK>
__device__ __forceinline__ void factor_invert(float* S, lds_counter* sync, int wave, int lane, float piv_lo, float piv_hi, float* Lout,
                                              long long ld, int* status, float thr, int* nullmask) {
  if (wave == 0) chain_wave<RANK>((lds_float*)S, sync, lane, piv_lo, piv_hi, Lout != nullptr, status, thr, nullmask);
  else if (wave == 1) update_wave((lds_float*)S, sync, lane, Lout, ld);
  else if (wave == 2) inverse_wave((lds_float*)S, sync, lane);
}

}  // namespace chol_block
}  // namespace dion
