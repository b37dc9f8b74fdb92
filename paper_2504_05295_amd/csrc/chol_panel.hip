// The r x r Cholesky factorisation of Cholesky-QR (Appendix A), blocked right-looking with 64-wide panels.
// Three drivers share the code for the 64 x 64 diagonal block: one launch per panel with no dependency between
// workgroups (below; large batches), up to three panels in one workgroup per matrix (chol_small_kernel), and the whole
// factorisation in one launch with workgroups that hand results on through flags (chol_stream_kernel further down).
//
// One panel step as a single launch:
// For the 64-wide panel starting at row/column k0 of the rp x rp Gram matrix C (lower triangle):
//   L11 = chol(C11),  W11 = L11^-1                       (64 x 64)
//   L21 = C21 W11^T                                       (rows below the diagonal block)
//   C22 -= L21 L21^T                                      (trailing matrix, lower tiles)
// Workgroup 0 writes L11 and W11.  Every other workgroup owns one 64x64 tile (i, j) of the trailing
// matrix; it redoes the small diagonal factorisation itself (cheaper than a grid-wide wait), forms
// the two panel blocks L21_i and L21_j it needs with fp32 MFMA, and updates its tile.  The workgroups
// of column j = 1 also store their L21_i into L.
//
// Inside a workgroup the diagonal block is the latency-critical part: three waves share it (chol_block.hpp), wave 3
// meanwhile fetches the two panel blocks C21_i, C21_j into LDS.
#include "chol_block.hpp"
#include "chol_order.hpp"

namespace dion {

namespace {
// acc = As[64 x 64] * Bs[64 x 64]^T for this wave's 32x32 quadrant (LDS tiles, k contiguous).  The operands of two k-steps are
// read ahead of the products, by order: left alone the compiler reads each right before its use where registers look
// scarce, and every k-step waits for the LDS.
__device__ __forceinline__ f32x16_t mma_64(const float* As, const float* Bs, int wm, int wn, int lr, int lk) {
  f32x16_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  f32x4_t a[CB / 8], b[CB / 8];
#pragma unroll
  for (int k = 0; k < CB / 8; ++k) {
    a[k] = *(const f32x4_t*)(As + (wm * 32 + lr) * CBP + 8 * k + lk * 4);
    b[k] = *(const f32x4_t*)(Bs + (wn * 32 + lr) * CBP + 8 * k + lk * 4);
  }
#pragma unroll
  for (int k = 0; k < CB / 8; ++k)
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[k][s], b[k][s], acc, 0, 0, 0);
  __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
  for (int k = 0; k < CB / 8 - 2; ++k) {
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x8, 4, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x8, 8, 0);
  return acc;
}
}  // namespace

template <bool RANK>
__global__ void __launch_bounds__(256, 2) chol_panel_kernel(CholPanelPtrs p, int k0, int rp, float piv_lo, float piv_hi, int mode) {
  // mode 0: fused (workgroup 0 writes L11/W11, the others own tiles and redo the factorisation)
  // mode 1: diagonal block only (one workgroup per matrix)      mode 2: tiles only, W11 read back from memory
  // Modes 1+2 are used when there are so many tiles (large batches) that redoing the factorisation in
  // every workgroup would cost more than a second launch.
  const long long mat = (long long)blockIdx.y * p.stride;
  float* C = p.C + mat;
  float* L = p.L + mat;
  float* W = p.W + mat;
  int* status = p.status + blockIdx.y;
  const float* thr = RANK ? p.thr + mat + k0 : nullptr;
  int* nullmask = RANK ? p.nullmask + mat + k0 : nullptr;
  // Only the second Cholesky-QR pass carries a skip flag (set when it needs no factorisation); the first pass
  // starts its loads without this extra memory round trip.
  if (p.skip && p.skip[mat] != 0) return;   // uniform for the whole workgroup
  const long long ld = rp;
  __shared__ __attribute__((aligned(16))) float S0[CB * CBP];   // C11, later W11
  __shared__ __attribute__((aligned(16))) float S1[CB * CBP];   // C21_i, later L21_i
  __shared__ __attribute__((aligned(16))) float S2[CB * CBP];   // C21_j, later L21_j
  __shared__ volatile int sync[chol_block::COUNTERS];           // of the diagonal block's waves
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave & 1, wn = wave >> 1, lr = lane & 31, lk = lane >> 5;

  // tile (i, j), 1 <= j <= i, in units of 64 rows/columns below/right of the diagonal block
  const bool writer = mode != 2 && blockIdx.x == 0;
  int i = 1, j = 1;
  if (!writer) {
    const int q = (mode == 2) ? blockIdx.x : blockIdx.x - 1;
    i = (int)((sqrtf(8.f * q + 1.f) - 1.f) * 0.5f) + 1;
    while ((i - 1) * i / 2 > q) --i;
    while (i * (i + 1) / 2 <= q) ++i;
    j = q - (i - 1) * i / 2 + 1;
  }
  const long long rowi = k0 + (long long)CB * i, rowj = k0 + (long long)CB * j;

  for (int idx = t; idx < CB * CB / 4; idx += 256) {
    const int rr = idx >> 4, cc = (idx & 15) * 4;
    const long long at = (long long)(k0 + rr) * ld + k0 + cc;
    f32x4_t v = *(const f32x4_t*)((mode == 2) ? W + at : C + at);
    if (mode != 2) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (cc + e > rr) v[e] = 0.f;
    }
    *(f32x4_t*)(S0 + rr * CBP + cc) = v;
  }
  if (t < chol_block::COUNTERS) sync[t] = 0;
  // this thread's 16 entries of the trailing tile, fetched now so that they arrive during the factorisation
  float cold[16];
  if (!writer) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = wm * 32 + 8 * (v / 4) + 4 * lk + (v % 4), cc = wn * 32 + lr;
      cold[v] = C[(rowi + row) * ld + rowj + cc];
    }
  }
  __syncthreads();

  if (mode == 2) {
    for (int idx = t; idx < CB * CB / 4; idx += 256) {
      const int rr = idx >> 4, cc = (idx & 15) * 4;
      *(f32x4_t*)(S1 + rr * CBP + cc) = *(const f32x4_t*)(C + (rowi + rr) * ld + k0 + cc);
      if (j != i) *(f32x4_t*)(S2 + rr * CBP + cc) = *(const f32x4_t*)(C + (rowj + rr) * ld + k0 + cc);
    }
  } else if (wave < 3) {
    chol_block::factor_invert<RANK>(S0, (chol_block::lds_counter*)sync, wave, lane, piv_lo, piv_hi,
                                    writer ? L + (long long)k0 * ld + k0 : nullptr, ld, status, RANK ? thr[lane] : 0.f, writer ? nullmask : nullptr);
  } else if (!writer) {
    for (int idx = lane; idx < CB * CB / 4; idx += 64) {
      const int rr = idx >> 4, cc = (idx & 15) * 4;
      *(f32x4_t*)(S1 + rr * CBP + cc) = *(const f32x4_t*)(C + (rowi + rr) * ld + k0 + cc);
      if (j != i) *(f32x4_t*)(S2 + rr * CBP + cc) = *(const f32x4_t*)(C + (rowj + rr) * ld + k0 + cc);
    }
  }
  __syncthreads();
  if (writer) {
    for (int idx = t; idx < CB * CB / 4; idx += 256) {
      const int rr = idx >> 4, cc = (idx & 15) * 4;
      *(f32x4_t*)(W + (long long)(k0 + rr) * ld + k0 + cc) = *(const f32x4_t*)(S0 + rr * CBP + cc);
    }
    return;
  }
  const f32x16_t li = mma_64(S1, S0, wm, wn, lr, lk);   // L21_i = C21_i W11^T
  f32x16_t lj = li;
  if (j != i) lj = mma_64(S2, S0, wm, wn, lr, lk);
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int row = wm * 32 + 8 * (v / 4) + 4 * lk + (v % 4), cc = wn * 32 + lr;
    S1[row * CBP + cc] = li[v];
    if (j != i) S2[row * CBP + cc] = lj[v];
    if (j == 1) L[(rowi + row) * ld + k0 + cc] = li[v];
  }
  __syncthreads();
  const f32x16_t up = mma_64(S1, (j != i) ? S2 : S1, wm, wn, lr, lk);   // L21_i L21_j^T
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int row = wm * 32 + 8 * (v / 4) + 4 * lk + (v % 4), cc = wn * 32 + lr;
    C[(rowi + row) * ld + rowj + cc] = cold[v] - up[v];
  }
}

// ---------------------------------------------------------------------------------------------------------
// Up to three panels (r <= 192): the whole step from the Gram matrix to W = L^-1 in one workgroup per matrix, which waits
// for nobody else.  At this size every kernel in the chain is launch latency (4-5 us each): a pass took a launch per
// panel, two products per merge of the inverse, one to add up the partial Gram matrices and one to pad, and an adaptive
// pass as many again, most of them only to find out that there was nothing to do.  The lower triangle of the matrix
// lives in LDS (six tiles, 102 KB); tile (k, k) turns into W11(k), tile (i, k) into L[i][k] and, once row i of
// the inverse is through, into W(i, k).  What bounds it is the chain of the diagonal blocks (3.7 us each) and the tile products,
// about 600 of 16 x 16 x 16 at three panels, 8 us of the compute unit's fp32 matrix units.  Per step k, with a barrier after each line:
//   D(k);   L[i][k] = C[i][k] W11^T (i > k)  and  Y(e) = sum_{e <= p < k} L[k][p] W(p, e) (e < k), in registers;   both to LDS
//   C[i][j] -= L[i][k] L[j][k]^T (i >= j > k)  and  W(k, e) = -W11 Y(e);   W(k, e) to LDS
// by eight waves, on 16 x 16 tiles in the register layout of chol_block.hpp, zero ones of W11 and those above the diagonal left
// out: the first line by strips of sixteen rows (wave % 4) and tiles (wave / 4), the second tile by tile.  A step against four
// waves with a 32 x 32 quadrant of every 64 x 64 product each: 1111 x 1733 r = 139 in fp32 170 -> 158 us, two layers of d = 768,
// r = 192 360 -> 346, 256 x 256 r = 64 in fp32 70.1 -> 68.7.
// FAST DECISION (adaptive, i.e. tau2 > 0): as launch_first_order_inverse describes it, in here.
template <int NB>
__global__ void __launch_bounds__(512, 2) chol_small_kernel(CholSmallArgs p) {
  const long long mat = (long long)blockIdx.x * p.stride;
  if (p.skip && p.skip[mat] != 0) return;   // uniform
  using chol_block::mm;
  using chol_block::ZERO;
  constexpr int TILES = NB * (NB + 1) / 2;
  __shared__ __attribute__((aligned(16))) float T[TILES][CB * CBP];
  __shared__ float red[512];
  __shared__ volatile int sync[chol_block::COUNTERS];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int c16 = lane & 15, g4 = 4 * (lane >> 4);
  const int ld = p.rp, r = p.r;
  float* C = p.C + mat;
  float* L = p.L + mat;
  float* W = p.W + mat;
  auto tile = [&](int i, int j) __attribute__((always_inline)) -> float* { return T[i * (i + 1) / 2 + j]; };
  auto sub = [&](float* S, int i, int j) __attribute__((always_inline)) -> lds_f32x4* { return chol_block::tile_at((lds_float*)S, i, j, lane); };
  // the transpose of 16 x 16 tile (i, j) of S: with it as the right operand mm adds Y S(i, j)
  auto sub_t = [&](const float* S, int i, int j) __attribute__((always_inline)) {
    f32x4_t x;
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = S[(16 * i + g4 + v) * CBP + 16 * j + c16];
    return x;
  };
  auto at = [&](float* M, int i, int j, int si, int sj) __attribute__((always_inline)) {   // this lane's four entries of tile (si, sj) of tile (i, j)
    return (f32x4_t*)(M + (long long)(i * CB + 16 * si + c16) * ld + j * CB + 16 * sj + g4);
  };
  // The lower tiles in: the loads of all tiles and of UN splits are in flight together (tile by tile the cut-short pass took
  // 11 us at three panels, five of them round trips to memory); partial results are added up in the order of the splits.
  // Rows and columns from r up become the identity's, entries above the diagonal zero.
  constexpr int UN = NB == 1 ? 4 : 2;
  const int trow = t >> 4, tcol = (t & 15) * 4;
  f32x4_t acc[TILES][2];
#pragma unroll
  for (int x = 0; x < TILES; ++x)
#pragma unroll
    for (int q = 0; q < 2; ++q) acc[x][q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  {
    const float* src = (p.nsplit > 1 ? p.Cpart + mat : C) + (long long)trow * ld + tcol;
#pragma unroll 1
    for (int sp = 0; sp < p.nsplit; sp += UN) {
      f32x4_t v[UN][TILES][2];
#pragma unroll
      for (int u = 0; u < UN; ++u)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j <= i; ++j)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
              f32x4_t& w = v[u][i * (i + 1) / 2 + j][q];
              w = f32x4_t{0.f, 0.f, 0.f, 0.f};
              if (sp + u < p.nsplit)
                w = *(const f32x4_t*)(src + (long long)(sp + u) * p.split_stride + (long long)(i * CB + 32 * q) * ld + j * CB);
            }
#pragma unroll
      for (int u = 0; u < UN; ++u)
#pragma unroll
        for (int x = 0; x < TILES; ++x)
#pragma unroll
          for (int q = 0; q < 2; ++q) acc[x][q] += v[u][x][q];
    }
  }
  float dist = 0.f;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j <= i; ++j)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        f32x4_t& c = acc[i * (i + 1) / 2 + j][q];
        const int row = i * CB + trow + 32 * q;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int col = j * CB + tcol + e;
          if (row >= r || col >= r) c[e] = row == col ? 1.f : 0.f;
          else if (col > row) c[e] = 0.f;
          else {
            const float d = c[e] - (row == col ? 1.f : 0.f);
            dist += (row == col ? 1.f : 2.f) * d * d;
          }
        }
        *(f32x4_t*)(tile(i, j) + (trow + 32 * q) * CBP + tcol) = c;
        if (p.nsplit > 1) *(f32x4_t*)(C + (long long)row * ld + j * CB + tcol) = c;
      }
  if (p.tau2 > 0.f) {
    red[t] = dist;
    __syncthreads();
    for (int sft = 256; sft > 0; sft >>= 1) {
      if (t < sft) red[t] += red[t + sft];
      __syncthreads();
    }
    const bool fast = red[0] <= p.tau2;   // false for NaN
    if (t == 0) p.fast[mat] = fast ? 1 : 0;
    if (fast) {
      if (!p.decision_only)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j <= i; ++j)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
              const int rr = trow + 32 * q;
              f32x4_t v = acc[i * (i + 1) / 2 + j][q];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                if (i != j || tcol + e != rr) v[e] = -v[e];
                else v[e] = 1.f - 0.5f * (v[e] - 1.f);
              }
              *(f32x4_t*)(W + (long long)(i * CB + rr) * ld + j * CB + tcol) = v;
            }
      return;   // uniform
    }
  }
  const int q = wave & 3, half = wave >> 2;
#pragma unroll 1   // (three copies of the diagonal block's code are more than the instruction cache holds)
  for (int k = 0; k < NB; ++k) {
    float* S0 = tile(k, k);
    if (t < chol_block::COUNTERS) sync[t] = 0;
    __syncthreads();
    chol_block::factor_invert<false>(S0, (chol_block::lds_counter*)sync, wave, lane, p.piv_lo, p.piv_hi, L + (long long)k * CB * (ld + 1), ld,
                                     p.status + blockIdx.x, 0.f, nullptr);
    __syncthreads();
    // rows 16 q of one of the NB - 1 tiles of this line: the tiles L[i][k], i > k, then the sums Y(e), e < k
    f32x4_t out[4] = {ZERO, ZERO, ZERO, ZERO};
    const int i1 = k + 1 + half, e1 = i1 - NB;   // i1 < NB: L[i1][k]; else, e1 < k: Y(e1)
    if (i1 < NB) {
      f32x4_t y[4], w[10];   // (operands are read ahead of the products: see mma_64)
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = *sub(tile(i1, k), q, e);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e <= j; ++e) w[j * (j + 1) / 2 + e] = *sub(S0, j, e);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e <= j; ++e) out[j] = mm(out[j], y[e], w[j * (j + 1) / 2 + e]);
    } else if (e1 < k) {
#pragma unroll 1
      for (int m = e1; m < k; ++m) {
        f32x4_t y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = *sub(tile(k, m), q, e);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          f32x4_t x[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = sub_t(tile(m, e1), e, j);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (m > e1 || e >= j) out[j] = mm(out[j], y[e], x[e]);   // (W11(e1) is lower triangular)
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 2; ++e)   // W11 out
      *(f32x4_t*)(W + (long long)(k * CB + trow + 32 * e) * ld + k * CB + tcol) = *(const f32x4_t*)(S0 + (trow + 32 * e) * CBP + tcol);
    __syncthreads();
    if (i1 < NB) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        *sub(tile(i1, k), q, j) = out[j];
        *at(L, i1, k, q, j) = out[j];
      }
    } else if (e1 < k) {
#pragma unroll
      for (int j = 0; j < 4; ++j) *sub(tile(k, e1), q, j) = out[j];
    }
    __syncthreads();
    // the updates, their 16 x 16 tiles dealt out to the waves
    int n = wave;
#pragma unroll
    for (int i = 1; i < NB; ++i)
#pragma unroll
      for (int j = 1; j <= i; ++j) {
        if (j <= k) continue;   // (uniform)
        const int count = i == j ? 10 : 16;
        for (; n < count; n += 8) {
          const int si = i != j ? n >> 2 : n >= 6 ? 3 : n >= 3 ? 2 : n >= 1 ? 1 : 0, sj = i != j ? n & 3 : n - si * (si + 1) / 2;
          const f32x4_t old = *sub(tile(i, j), si, sj);
          f32x4_t c = ZERO, y[4], x[4];   // (summed up by itself: with `old` in the accumulator every partial sum is rounded at its size)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            y[e] = *sub(tile(i, k), si, e);
            x[e] = *sub(tile(j, k), sj, e);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int e = 0; e < 4; ++e) c = mm(c, y[e], x[e]);
          *sub(tile(i, j), si, sj) = old - c;
        }
        n -= count;
      }
    // W(k, e) = -W11 Y(e): tiles (half, q) and (half + 2, q)
    f32x4_t z[NB > 1 ? NB - 1 : 1][2];
#pragma unroll
    for (int e1 = 0; e1 + 1 < NB; ++e1) {
      if (e1 >= k) continue;   // (uniform)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int si = half + 2 * u;
        f32x4_t y[4], x[4], c = ZERO;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          y[e] = *sub(S0, si, e);
          x[e] = sub_t(tile(k, e1), e, q);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (e <= si) c = mm(c, y[e], x[e]);
        z[e1][u] = -c;
        *at(W, k, e1, si, q) = z[e1][u];
      }
    }
    if (k > 0 && k + 1 < NB) {
      __syncthreads();   // row k of Y is read
#pragma unroll
      for (int e1 = 0; e1 + 1 < NB; ++e1)
        if (e1 < k)
#pragma unroll
          for (int u = 0; u < 2; ++u) *sub(tile(k, e1), half + 2 * u, q) = z[e1][u];
    }
  }
}

hipError_t launch_chol_small(CholSmallArgs p, int batch, hipStream_t s) {
  if (p.nsplit < 1 || p.rp % CB || p.r > p.rp || p.split_stride % 4) return hipErrorInvalidValue;
  switch (p.rp / CB) {
    case 1: hipLaunchKernelGGL(chol_small_kernel<1>, dim3(batch), dim3(512), 0, s, p); break;
    case 2: hipLaunchKernelGGL(chol_small_kernel<2>, dim3(batch), dim3(512), 0, s, p); break;
    case 3: hipLaunchKernelGGL(chol_small_kernel<3>, dim3(batch), dim3(512), 0, s, p); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------
// The whole factorisation in one launch, for one or a few matrices (where a launch per panel leaves the GPU
// waiting on launch latencies and on workgroups that each redo the diagonal block).
//
// The 64x64 tiles of the lower triangle have fixed owners: tile (i, j) belongs to workgroup
// (i mod pr) * pc + (j mod pc), except that (i, i-1) goes with (i, i).  An owner does everything that
// happens to its tile, in panel order k = 0, 1, ...:
//   D(k)      tile (k, k):        factor it, publish L11, W11 = L11^-1                  -> wflag[k]
//   T(i, k)   tile (i, k), i > k: L[i][k] = C[i][k] W11^T, publish it                   -> lflag[i] = k + 1
//   U(i,j,k)  tile (i, j), j > k: C[i][j] -= L[i][k] L[j][k]^T                          (needs lflag[i], lflag[j] > k)
// so tile data never changes hands; only W11 and the finished tiles of L cross between workgroups, through
// memory, with device-scope stores and loads, each announced by a flag that is written once the stores have
// completed.  The owner of (k+1, k+1) also owns (k+1, k): the chain D(k) -> T(k+1, k) -> U(k+1, k+1, k)
// -> D(k+1), which bounds the run time, crosses workgroups once per panel, and that workgroup takes it before
// its other work.  Every workgroup handles its tasks in an order in which a task only waits for tasks that
// come earlier in the common order (panel, then D < T < U), so somebody can always proceed.
// Flags carry the number of the launch (epoch, a counter kept in device memory) and need no clearing.  Waits are bounded: a workgroup that
// gives up raises the abort word, everybody else sees it at the next wait, and the status word reports a wait
// timeout for the matrix (not a breakdown: nothing is known about its numerics); all workgroups must be resident at once, which the host guarantees by the grid size.
namespace {
typedef unsigned long long u64;
typedef __attribute__((address_space(1))) float gfloat;
typedef __attribute__((address_space(1))) int gint;
typedef __attribute__((address_space(1))) u64 gu64;
typedef __attribute__((address_space(1))) f32x4_t gf32x4;

__device__ __forceinline__ u64 flag_load(const gu64* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void flag_store(gu64* p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Data that crosses between workgroups (W11 and the tiles of L) is written with device-scope stores, which go past the caches
// that are private to a compute unit or to one part of the chip; no cache-wide write-back is needed then, only that
// the writer's stores have completed before its flag goes out.  Tiles that are written more than once before they change hands
// are read with device-scope loads, finished tiles with ordinary ones (see tile_to_regs).
// Addresses are a base that is the same in all lanes plus a 32-bit byte offset per lane: the base and its steps from row to
// row stay in scalar registers (64-bit addresses per lane took up to 130 registers that the kernels below had to spill).
typedef __attribute__((address_space(1))) char gchar;
typedef unsigned lane_off;
__device__ __forceinline__ float shared_load(const gfloat* base, lane_off o) {
  return __int_as_float(__hip_atomic_load((const gint*)((const gchar*)base + o), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void shared_store(gfloat* base, lane_off o, float v) {
  __hip_atomic_store((gint*)((gchar*)base + o), __float_as_int(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float own_load(const gfloat* base, lane_off o) { return *(const gfloat*)((const gchar*)base + o); }
__device__ __forceinline__ void own_store(gfloat* base, lane_off o, float v) { *(gfloat*)((gchar*)base + o) = v; }

// A row step in bytes that the compiler forgets the origin of: the sixteen row addresses are then a running sum, two scalar
// additions each, where it would keep sixteen multiples in registers that it has not got, and move them in and out.
__device__ __forceinline__ unsigned row_step(int rows, int ld) {
  unsigned b = 4u * (unsigned)(rows * ld);
  asm volatile("" : "+s"(b));
  return b;
}
template <class T>
__device__ __forceinline__ T* advance(T* p, unsigned bytes) { return (T*)((gchar*)p + bytes); }
// f(v, row address) for a thread's 16 entries of a tile in the result layout of the 32x32 product: rows 8 (v / 4) + v % 4
template <class F>
__device__ __forceinline__ void for_rows(gfloat* base, int ld, F f) {
  const unsigned one = row_step(1, ld), five = row_step(5, ld);
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    f(v, base);
    base = advance(base, (v & 3) == 3 ? five : one);
  }
}

// Rows r0, r0 + step, ... (N of them) of a tile from LDS to memory, column c each.  (All reads come before the first store:
// one by one, a store would hold back the read behind it, 130 cycles each.)
template <int N>
__device__ __forceinline__ void rows_to_shared(gfloat* dst, int ld, const float* S, int r0, int step, int c) {
  float v[N];
#pragma unroll
  for (int e = 0; e < N; ++e) v[e] = S[(r0 + step * e) * CBP + c];
  __builtin_amdgcn_sched_barrier(0);
  const lane_off o = 4u * (unsigned)(r0 * ld + c);
  const unsigned bytes = row_step(step, ld);
#pragma unroll
  for (int e = 0; e < N; ++e) {
    shared_store(dst, o, v[e]);
    dst = advance(dst, bytes);
  }
}
__device__ __forceinline__ void lds_to_shared_tile(gfloat* dst, int ld, const float* S, int t) { rows_to_shared<16>(dst, ld, S, t >> 6, 4, t & 63); }
// Finished tiles of L and W, W11 included, are read with ordinary loads, 16 bytes each, and so come out of the L2 of this part
// of the chip from the second reader on: nobody reads them before their flag, so that no cache of this launch can hold
// them as they were, and a tile shares no cache line with another.  (Device-scope loads went to memory for every reader: at
// 16 panels 167 us with them and 148 without, at 32 415 and 356.)  Thread t has the columns 4 (t % 16) .. + 4 of rows t / 16 + 16 q.
struct tile_regs { f32x4_t v[4]; };
__device__ __forceinline__ void tile_to_regs(tile_regs& r, const gfloat* src, int ld, int t) {
  const lane_off o = 4u * (unsigned)((t >> 4) * ld + (t & 15) * 4);
  const unsigned step = row_step(16, ld);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    r.v[q] = *(const gf32x4*)((const gchar*)src + o);
    src = advance(src, step);
  }
}
template <bool TRANSPOSED>
__device__ __forceinline__ void regs_to_lds(float* S, const tile_regs& r, int t) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = (t >> 4) + 16 * q, c = (t & 15) * 4;
    if (TRANSPOSED) {
#pragma unroll
      for (int e = 0; e < 4; ++e) S[(c + e) * CBP + row] = r.v[q][e];
    } else {
      *(f32x4_t*)(S + row * CBP + c) = r.v[q];
    }
  }
}
__device__ __forceinline__ void tile_to_lds(float* S, const gfloat* src, int ld, int t) {
  tile_regs r;
  tile_to_regs(r, src, ld, t);
  __builtin_amdgcn_sched_barrier(0);   // (all four in flight before the first is waited for)
  regs_to_lds<false>(S, r, t);
}

struct StreamCtx {
  gfloat* C;
  gfloat* L;
  gfloat* W;
  int* status;
  gu64* wflag;
  gu64* lflag;
  gu64* abort_word;
  u64 epoch;
  unsigned spin_limit;
  int ld;
  float piv_lo, piv_hi;
};

// Polls until ready() holds, on behalf of the threads with `mine`; returns false for everybody when a wait
// was given up (here or, as the abort word tells, elsewhere).
template <class F, class Barrier>
__device__ __forceinline__ bool wait_until(const StreamCtx& x, chol_block::lds_counter* gave_up, bool mine, F ready, Barrier barrier) {
  if (mine) {
    unsigned n = 0;
    while (!ready()) {
      __builtin_amdgcn_s_sleep(2);
      if (++n > x.spin_limit) {
        flag_store(x.abort_word, x.epoch);
        if (*x.status == 0) *x.status = ST_TIMEOUT;
        *gave_up = 1;
        break;
      }
      if ((n & 31u) == 0 && flag_load(x.abort_word) == x.epoch) {
        *gave_up = 1;
        break;
      }
    }
  }
  barrier();
  return *gave_up == 0;
}
template <class F>
__device__ __forceinline__ bool wait_until(const StreamCtx& x, chol_block::lds_counter* gave_up, bool mine, F ready) {
  return wait_until(x, gave_up, mine, ready, [] { __syncthreads(); });
}
// 32-bit flags: the low 32 bits of the launch's epoch
typedef __attribute__((address_space(1))) unsigned gu32;
__device__ __forceinline__ unsigned flag_load32(const gu32* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void flag_store32(gu32* p, unsigned v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
}  // namespace

// An adaptive pass' decision (see launch_first_order_inverse), taken by every workgroup of a factorisation launch from the
// same partial sums in the same order, so all of a matrix' workgroups take the same one.  True: the factorisation is not
// needed, and the first-order inverse, where it is wanted, is in W.  In here it costs the factorisation 2 us when it runs
// and saves a launch of its own (5-7 us) always.  `red`: 256 floats of LDS.
__device__ __forceinline__ bool chol_fast_decision(const CholStreamArgs& p, long long mat, float* red) {
  const int t = threadIdx.x;   // (256 threads do it, in the same order in every workgroup, whatever its size)
  float acc = 0.f;
  for (int k = t; t < 256 && k < GRAM_DEFECT_PARTS; k += 256) acc += p.defect[mat + k];
  if (t < 256) red[t] = acc;
  __syncthreads();
  for (int sft = 128; sft > 0; sft >>= 1) {
    if (t < sft) red[t] += red[t + sft];
    __syncthreads();
  }
  const bool fast = red[0] <= p.tau2;   // false for NaN
  __syncthreads();
  if (blockIdx.x == 0 && t == 0) p.fast[mat] = fast ? 1 : 0;
  if (fast && !p.decision_only && t < 256) {
    const float* C = p.C + mat;
    float* W = p.W + mat;
    const int ppr = p.rp / 4;   // pieces of four columns per row
    for (int idx = (int)blockIdx.x * 256 + t; idx < p.rp * ppr; idx += (int)gridDim.x * 256) {
      const int i = idx / ppr, j0 = 4 * (idx % ppr);
      if (j0 > (i | (CB - 1))) continue;   // above the block diagonal W is zero and stays so
      const f32x4_t c = *(const f32x4_t*)(C + (long long)i * p.rp + j0);
      f32x4_t v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = j0 + e;
        v[e] = j > i ? 0.f : i >= p.r ? (i == j ? 1.f : 0.f) : i == j ? 1.f - 0.5f * (c[e] - 1.f) : 0.f - c[e];
      }
      *(f32x4_t*)(W + (long long)i * p.rp + j0) = v;
    }
  }
  return fast;
}

template <bool RANK>
__global__ void __launch_bounds__(256, 1) chol_stream_kernel(CholStreamArgs p) {
  const long long mat = (long long)blockIdx.y * p.stride;
  if (p.skip && p.skip[mat] != 0) return;   // uniform for the whole grid row of this matrix
  const int nb = p.rp / CB, pr = p.pr, pc = p.pc;
  StreamCtx x;
  x.C = (gfloat*)(p.C + mat);
  x.L = (gfloat*)(p.L + mat);
  x.W = (gfloat*)(p.W + mat);
  x.status = p.status + blockIdx.y;
  x.wflag = (gu64*)(p.sync + (long long)blockIdx.y * p.sync_stride);
  x.lflag = x.wflag + nb;
  x.abort_word = x.lflag + nb;
  x.epoch = *p.step_counter * 8ull + (u64)p.pass;   // unique per launch: step counter kept on the device, pass within the step
  x.spin_limit = p.spin_limit;
  x.ld = p.rp;
  x.piv_lo = p.piv_lo;
  x.piv_hi = p.piv_hi;
  const int ld = p.rp;
  const float* thr = RANK ? p.thr + mat : nullptr;
  int* nullmask = RANK ? p.nullmask + mat : nullptr;

  __shared__ __attribute__((aligned(16))) float S0[CB * CBP];   // diagonal block / W11
  __shared__ __attribute__((aligned(16))) float S1[CB * CBP];
  __shared__ __attribute__((aligned(16))) float S2[CB * CBP];
  __shared__ volatile int sync[chol_block::COUNTERS];
  __shared__ int gave_up_word;
  chol_block::lds_counter* const gave_up = (chol_block::lds_counter*)&gave_up_word;   // (not through a generic pointer: see chol_block.hpp)
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave & 1, wn = wave >> 1, lr = lane & 31, lk = lane >> 5;
  const int wg = blockIdx.x, a = wg / pc, b = wg % pc;
  // this thread's part of a 64x64 tile in the MFMA result layout: rows frow + 8 (v / 4) + v % 4, column fcol
  const int frow = wm * 32 + 4 * lk, fcol = wn * 32 + lr;
  const lane_off fo = 4u * (unsigned)(frow * ld + fcol);
  if (t == 0) *gave_up = 0;
  __syncthreads();
  if (p.tau2 > 0.f && chol_fast_decision(p, mat, S1)) return;   // uniform for the whole grid row of this matrix

  int s0_holds = -1;             // panel whose W11 is in S0
  // A tile of L that sits in S1 and still has to be written out and announced; the wave that has nothing
  // to do during the next D does that, off the chain of dependent steps.
  gu64* pending_flag = nullptr;
  gfloat* pending_tile = nullptr;
  u64 pending_value = 0;

  // D(k).  in_lds: the block is already in S0 (lower part, zeros above the diagonal).
  auto do_diag = [&](int k, bool in_lds) __attribute__((always_inline)) {
    const int at = (k * CB) * ld + k * CB;
    if (!in_lds) {
      for (int idx = t; idx < CB * CB / 4; idx += 256) {
        const int rr = idx >> 4, cc = (idx & 15) * 4;
        f32x4_t v = *(const gf32x4*)(x.C + at + rr * ld + cc);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (cc + e > rr) v[e] = 0.f;
        *(f32x4_t*)(S0 + rr * CBP + cc) = v;
      }
    }
    if (t < chol_block::COUNTERS) sync[t] = 0;
    __syncthreads();
    if (wave < 3) {
      chol_block::factor_invert<RANK>(S0, (chol_block::lds_counter*)sync, wave, lane, x.piv_lo, x.piv_hi, (float*)(x.L + at), ld, x.status,
                                      RANK ? thr[k * CB + lane] : 0.f, RANK ? nullmask + k * CB : nullptr);
    } else if (pending_flag) {
      rows_to_shared<32>(pending_tile, ld, S1, 0, 1, lane);
      rows_to_shared<32>(pending_tile + 32 * ld, ld, S1 + 32 * CBP, 0, 1, lane);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (lane == 0) flag_store(pending_flag, pending_value);
    }
    pending_flag = nullptr;
    __syncthreads();
    lds_to_shared_tile(x.W + at, ld, S0, t);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's stores have completed before the barrier
    __syncthreads();
    if (t == 0) flag_store(x.wflag + k, x.epoch);
    s0_holds = k;
  };

  // T(i, k); leaves L[i][k] in S1 as well.  defer_flag: the flag goes out during the next D
  auto do_column_tile = [&](int i, int k, bool defer_flag) __attribute__((always_inline)) -> bool {
    __syncthreads();   // earlier readers of S0 / S1 are through
    tile_to_lds(S1, x.C + (i * CB) * ld + k * CB, ld, t);
    if (s0_holds != k) {
      if (!wait_until(x, gave_up, t == 0, [&] { return flag_load(x.wflag + k) == x.epoch; })) return false;
      tile_to_lds(S0, x.W + (k * CB) * ld + k * CB, ld, t);
      s0_holds = k;
    }
    __syncthreads();
    const f32x16_t li = mma_64(S1, S0, wm, wn, lr, lk);   // L[i][k] = C[i][k] W11^T
    __syncthreads();
    gfloat* dst = x.L + (i * CB) * ld + k * CB;
#pragma unroll
    for (int v = 0; v < 16; ++v) S1[(frow + 8 * (v / 4) + (v % 4)) * CBP + fcol] = li[v];
    if (!defer_flag) for_rows(dst, ld, [&](int v, gfloat* row) { shared_store(row, fo, li[v]); });
    if (defer_flag) {
      pending_flag = x.lflag + i;
      pending_tile = dst;
      pending_value = (x.epoch << 32) | (u64)(k + 1);
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();   // S1 is complete (and, unless deferred, everybody's stores have completed)
    if (!defer_flag && t == 0) flag_store(x.lflag + i, (x.epoch << 32) | (u64)(k + 1));
    return true;
  };

  // U(i, j, k)
  auto do_update = [&](int i, int j, int k) __attribute__((always_inline)) {
    gfloat* ct = x.C + (i * CB) * ld + j * CB;
    float cold[16];
    for_rows(ct, ld, [&](int v, gfloat* row) { cold[v] = own_load(row, fo); });
    __syncthreads();   // earlier readers of S1 / S2 are through
    tile_to_lds(S1, x.L + (i * CB) * ld + k * CB, ld, t);
    if (j != i) tile_to_lds(S2, x.L + (j * CB) * ld + k * CB, ld, t);
    __syncthreads();
    const f32x16_t up = mma_64(S1, (j != i) ? S2 : S1, wm, wn, lr, lk);
    for_rows(ct, ld, [&](int v, gfloat* row) { own_store(row, fo, cold[v] - up[v]); });
  };

  // U(k1, k1, k1 - 1) with L[k1][k1 - 1] in S1; the result goes straight into S0 for D(k1) and nowhere else
  auto do_update_to_diag = [&](int k1) __attribute__((always_inline)) {
    gfloat* ct = x.C + (k1 * CB) * ld + k1 * CB;
    float cold[16];
    for_rows(ct, ld, [&](int v, gfloat* row) { cold[v] = own_load(row, fo); });
    const f32x16_t up = mma_64(S1, S1, wm, wn, lr, lk);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = frow + 8 * (v / 4) + (v % 4);
      S0[row * CBP + fcol] = (fcol <= row) ? cold[v] - up[v] : 0.f;
    }
    s0_holds = -1;
  };

  // Step k handles panel k after the diagonal block k+1 has been taken care of (step -1: block 0 only).
  for (int k = -1; k + 1 < nb; ++k) {
    // the chain: T(k+1, k), U(k+1, k+1, k), D(k+1)
    if (((k + 1) % pr) * pc + ((k + 1) % pc) == wg) {
      if (k >= 0) {
        if (!do_column_tile(k + 1, k, true)) return;
        do_update_to_diag(k + 1);
      }
      do_diag(k + 1, k >= 0);
    }
    if (k < 0) continue;
    // the other tiles of column k
    if (k % pc == b) {
      for (int i = a + ((k + 1 - a + pr - 1) / pr) * pr; i < nb; i += pr) {
        if (i <= k || i == k + 1) continue;
        if (!do_column_tile(i, k, false)) return;
      }
    }
    // wait for the tiles of L that this workgroup's updates need: one thread per block row
    {
      bool need = false;
      if (t > k && t < nb) {
        need = (t % pr) == a || (t % pc) == b;   // rows of regular tiles (as i or as j)
        if ((t % pr) * pc + (t % pc) == wg || ((t + 1) < nb && ((t + 1) % pr) * pc + ((t + 1) % pc) == wg)) need = true;   // tiles (i, i-1)
      }
      if (!wait_until(x, gave_up, need, [&] {
            const u64 v = flag_load(x.lflag + t);
            return (unsigned)(v >> 32) == (unsigned)x.epoch && (unsigned)v >= (unsigned)(k + 1);   // (the tag holds the epoch's low 32 bits)
          }))
        return;
    }
    for (int j = b + ((k + 1 - b + pc - 1) / pc) * pc; j < nb; j += pc) {
      if (j <= k) continue;
      for (int i = a + ((j - a + pr - 1) / pr) * pr; i < nb; i += pr) {
        if (i < j || i == j + 1) continue;
        if (i == j && j == k + 1) continue;   // went into D(k+1) above
        do_update(i, j, k);
      }
    }
    for (int i = k + 2; i < nb; ++i)
      if ((i % pr) * pc + (i % pc) == wg) do_update(i, i - 1, k);
  }
}

// ---------------------------------------------------------------------------------------------------------
// The same factorisation with the chain of dependent steps kept inside ONE workgroup (used when a matrix has sixteen
// workgroups or more to itself).  In the kernel above the chain D(k) -> T(k+1, k) -> U(k+1, k+1, k) -> D(k+1) changes
// workgroups once per panel, and that hand-over (W11 out to memory, a flag, a poll, W11 back in) is about a quarter of
// the panel period.  Here workgroup 0 does nothing but the chain, for all k, with W11 never leaving its LDS on the
// way, and the others ("helpers": pr x pc of them, numbered from 1) do everything else:
//   chain     D(k);  L[k+1][k] = C'[k+1][k] W11^T;  C''[k+1][k+1] = C'[k+1][k+1] - L[k+1][k] L[k+1][k]^T  -> D(k+1)
//   helpers   every other T(i, k) and all updates U(i, j, p) except the last one of a diagonal tile
// where C'[k+1][k] and C'[k+1][k+1] are those two tiles with the updates of all panels before k applied.  They come through
// memory, announced by a flag each, while the chain factors D(k); W11 and L[k+1][k] go out likewise, each as soon as
// the last wave's stores of it have completed; the chain waits for nothing but its own stores.
// That hand-over, W11(k) out, T(k+2, k), the last update of the two tiles of row k+2, and back in, is what bounds the
// panel period now.  So near the diagonal every tile has a team of its own: of row i, team number (3 i + d) mod (number of teams) keeps
// (i, i-d), d = 0, 1, and a private copy of (i, i-2), which it turns into L[i][i-2] for the last update of its tile;
// team d = 2 has such a copy only, and its L[i][i-2] is the one that goes out, as early as can be: the row below waits for it
// with the update before its last one.  (Measured with one owner of all three: its
// updates, 3.5 us each one after the other, bounded the period at 13 us.  With the chain's workgroup doing the last update
// of (k+1, k) and (k+1, k+1) itself beside D(k), a panel period more for the hand-over: 10 us, the fp32 matrix units of one
// compute unit being what bounds it then.)
// The chain's workgroup has eight waves, two to a SIMD; the eliminating wave's SIMD has no other work beside D(k).
// A helper workgroup is two teams of four waves that know nothing of each other (a barrier of their own each): while one
// waits for its tiles, the other multiplies.
// Tiles that cross between workgroups are written with device-scope stores; the two look-ahead tiles, which their owner reads
// and writes before the chain does, are only ever read with device-scope loads too.  Waits are bounded as above.
//
// FUSE_INV: the helpers also form W = L^-1, row by row behind the factorisation, so that no separate pass over L
// follows it.  With W'(j, e) the running value of tile (j, e), e < j, that starts at zero,
//   UW(j, e, p)  W'(j, e) -= L[j][p] W(p, e)        for e <= p < j        (needs lflag[j] > p and row p of W)
//   TW(p, e)     W(p, e) = W11(p) W'(p, e)           once UW(p, e, p - 1) is through   -> vflag[p][e]
// and W(p, p) = W11(p) as the chain leaves it (wflag[p]; the last one is announced when the chain ends).  Tile (j, e)
// belongs to team (j mod pr) pc + (e mod pc), which applies UW(j, e, p) for j >= p + 2 after the look-ahead work of
// panel p + 1 (before it, the chain found its next tiles 3 us late) and UW(p + 1, e, p) right before TW(p + 1, e),
// also in panel p + 1: a helper only ever waits for tiles of row p of W while it works on panel p + 1, and their
// owners produce them from flags of the chain and of row p - 1 alone, so the order of the factorisation's own tasks
// is untouched.  (With dependent columns their rows and columns of W11, hence of W, are zero; nothing else changes.  The
// separate inverse pass that the rank-tolerant factorisation used to need took 63-80 us at r = 1024.)  Running values are the owner's private data (ordinary accesses); finished tiles are written and
// read with device-scope accesses like the tiles of L.
template <bool RANK, bool FUSE_INV>
__global__ void __launch_bounds__(512, 2) chol_chain_kernel(CholStreamArgs p) {
  const long long mat = (long long)blockIdx.y * p.stride;
  if (p.skip && p.skip[mat] != 0) return;   // uniform for the whole grid row of this matrix
  const int nb = p.rp / CB, pr = 2 * p.pr, pc = p.pc;   // grid of teams
  StreamCtx x;
  x.C = (gfloat*)(p.C + mat);
  x.L = (gfloat*)(p.L + mat);
  x.W = (gfloat*)(p.W + mat);
  x.status = p.status + blockIdx.y;
  x.wflag = (gu64*)(p.sync + (long long)blockIdx.y * p.sync_stride);
  x.lflag = x.wflag + nb;
  gu64* const cflag = x.lflag + nb;
  x.abort_word = cflag + nb;
  gu64* const vflag = x.wflag + p.vflag_off;   // FUSE_INV: nb x nb words, [p][e] = tile (p, e) of W is final
  gfloat* const Tcopy = (gfloat*)(p.T + mat);  // (i, i-2+d): team d's copy of (i, i-2), d = 0..2
  // 32-bit flags, two to a word: W11(k) is out; the tile (i, i-d) may go to the chain (d = 2: L[i][0 .. i-2] is out)
  auto w11_flag = [&](int k) __attribute__((always_inline)) { return (gu32*)(x.wflag + k); };
  auto near_flag = [&](int i, int d) __attribute__((always_inline)) { return d == 0 ? (gu32*)(x.wflag + i) + 1 : (gu32*)(cflag + i) + (d - 1); };
  x.epoch = *p.step_counter * 8ull + (u64)p.pass;
  x.spin_limit = p.spin_limit;
  x.ld = p.rp;
  x.piv_lo = p.piv_lo;
  x.piv_hi = p.piv_hi;
  const int ld = p.rp;
  const float* thr = RANK ? p.thr + mat : nullptr;
  int* nullmask = RANK ? p.nullmask + mat : nullptr;

  // chain: diagonal block / W11, L[k+1][k], the two look-ahead tiles of row k+1; helpers: three tiles to a team
  __shared__ __attribute__((aligned(16))) float S[6][CB * CBP];
  __shared__ volatile int sync[chol_block::COUNTERS];
  __shared__ int stored[2];   // waves whose parts of W11(k) / of L[k+1][k] are in memory
  __shared__ int gave_up_word;
  chol_block::lds_counter* const gave_up = (chol_block::lds_counter*)&gave_up_word;   // (not through a generic pointer: see chol_block.hpp)
  __shared__ int arrived[2];  // of a helper's teams: waves that have come to a barrier, all barriers so far
  const int lane = threadIdx.x & 63;
  const unsigned ep = (unsigned)x.epoch;
  if (threadIdx.x == 0) *gave_up = 0;
  if (threadIdx.x < 2) arrived[threadIdx.x] = 0;
  __syncthreads();
  if (p.tau2 > 0.f && chol_fast_decision(p, mat, S[0])) return;   // uniform for the whole grid row of this matrix
  const u64 ep32 = x.epoch << 32;
  auto tile_at = [&](gfloat* base, int i, int j) __attribute__((always_inline)) { return base + (i * CB) * ld + j * CB; };

  if (blockIdx.x == 0) {
    // ---------------------------------------------------------------- the chain
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    using chol_block::mm;
    using chol_block::ZERO;
    float* const S0 = S[0];
    float* const SL = S[1];   // L[k+1][k]
    float* const SB = S[2];   // C'[k+1][k]
    float* const SD = S[3];   // C'[k+1][k+1]
    auto sub = [&](float* T, int i, int j) __attribute__((always_inline)) -> lds_f32x4* { return chol_block::tile_at((lds_float*)T, i, j, lane); };
    // diagonal tile 0 (its lower triangle is used)
    for (int idx = t; idx < CB * CB / 4; idx += 512) {
      const int rr = idx >> 4, cc = (idx & 15) * 4;
      *(f32x4_t*)(S0 + rr * CBP + cc) = *(const gf32x4*)(x.C + rr * ld + cc);
    }
    float thr_next = RANK ? thr[lane] : 0.f;   // (of the next diagonal block: fetched a step ahead)
    // this wave's stores have completed, and it is the last of `waves` to say so
    auto last_of = [&](int what, int waves) __attribute__((always_inline)) -> bool {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      return lane == 0 && __hip_atomic_fetch_add(&stored[what], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == waves - 1;
    };
    for (int k = 0; k < nb; ++k) {
      const int at = (k * CB) * ld + k * CB;
      if (t < chol_block::COUNTERS) sync[t] = 0;
      __syncthreads();
      if (t >= 192 && t < 194) stored[t - 192] = 0;   // (between two barriers: its last use lies before the one above, the next behind the one below)
#ifdef DION_CHOL_TIMING
      if (t == 0 && p.dbg) p.dbg[8 * k + 0] = wall_clock64();
#endif
      if (wave < 3) {
        chol_block::factor_invert<RANK>(S0, (chol_block::lds_counter*)sync, wave, lane, x.piv_lo, x.piv_hi, (float*)(x.L + at), ld, x.status,
                                        thr_next, RANK ? nullmask + k * CB : nullptr);
        if (RANK && k + 1 < nb) thr_next = thr[(k + 1) * CB + lane];
      }
      if (wave >= 3 && wave != 4 && k + 1 < nb) {
        // four waves fetch the two tiles of row k+1, sixteen rows of each, once they carry all updates up to panel k-1 (those of
        // row 1 have none: nothing to wait for)
        const int row0 = 16 * (wave == 3 ? 3 : wave - 5);
        unsigned n = 0;
        bool ready = k < 1, ok = true;
        float vs[16], vd[16];
        auto request = [&](float (&v)[16], int j) __attribute__((always_inline)) {
          const gfloat* src = tile_at(x.C, k + 1, j) + row0 * ld;
          const unsigned step = row_step(1, ld);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            v[r] = shared_load(src, 4u * lane);
            src = advance(src, step);
          }
        };
#ifdef DION_CHOL_TIMING
        if (t == 192 && p.dbg) p.dbg[8 * k + 3] = wall_clock64();
#endif
        while (!ready) {
          // (d = 2 too: this row's count of finished tiles is raised further by the chain only when that team has set it)
          const unsigned f0 = flag_load32(near_flag(k + 1, 0)), f1 = flag_load32(near_flag(k + 1, 1)), f2 = flag_load32(near_flag(k + 1, 2));
          ready = f0 == ep && f1 == ep && f2 == ep;
          if (ready) break;
          __builtin_amdgcn_s_sleep(1);
          const bool too_long = ++n > x.spin_limit;
          if (too_long) {
            flag_store(x.abort_word, x.epoch);
            if (*x.status == 0) *x.status = ST_TIMEOUT;
          }
          if (too_long || ((n & 31u) == 0 && flag_load(x.abort_word) == x.epoch)) {
            *gave_up = 1;
            ok = false;
            break;
          }
        }
#ifdef DION_CHOL_TIMING
        if (t == 192 && p.dbg) p.dbg[8 * k + 4] = wall_clock64();
#endif
        if (ok) {
          // (all loads of both are issued before the first of them is waited for: one memory round trip)
          request(vs, k);
          request(vd, k + 1);
#pragma unroll
          for (int r = 0; r < 16; ++r) SB[(row0 + r) * CBP + lane] = vs[r];
#pragma unroll
          for (int r = 0; r < 16; ++r) SD[(row0 + r) * CBP + lane] = vd[r];
        }
#ifdef DION_CHOL_TIMING
        if (t == 192 && p.dbg) p.dbg[8 * k + 5] = wall_clock64();
#endif
      }
      __syncthreads();
#ifdef DION_CHOL_TIMING
      if (t == 0 && p.dbg) p.dbg[8 * k + 1] = wall_clock64();
#endif
      if (*gave_up) return;   // uniform: written before the barrier
      // W11 out to the helpers, announced by the last wave whose part is in memory
      rows_to_shared<8>(x.W + at, ld, S0, wave, 8, lane);
      if (k + 1 == nb) {
        if (last_of(0, 8)) flag_store32(w11_flag(k), ep);
        break;
      }
      // L[k+1][k] = C'[k+1][k] W11^T: rows 16 (wave % 4), columns 32 (wave / 4)
      const int q = wave & 3, h = wave >> 2;
      f32x4_t l0 = ZERO, l1 = ZERO, y[4], w0[4], w1[4];   // (operands are read ahead of the products: see mma_64)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y[e] = *sub(SB, q, e);
        w0[e] = *sub(S0, 2 * h, e);
        w1[e] = *sub(S0, 2 * h + 1, e);
      }
      __builtin_amdgcn_sched_barrier(0);
      l0 = mm(l0, y[0], w0[0]);   // (W11 is lower triangular)
      l1 = mm(mm(l1, y[0], w1[0]), y[1], w1[1]);
      if (h == 1) {
        l0 = mm(mm(l0, y[1], w0[1]), y[2], w0[2]);
        l1 = mm(mm(l1, y[2], w1[2]), y[3], w1[3]);
      }
      *sub(SL, q, 2 * h) = l0;
      *sub(SL, q, 2 * h + 1) = l1;
      if (last_of(0, 8)) flag_store32(w11_flag(k), ep);
      __syncthreads();
      if (wave >= 4) rows_to_shared<16>(tile_at(x.L, k + 1, k), ld, SL, wave - 4, 4, lane);
      // the next diagonal block (its lower triangle): ten tiles, numbered along the rows, wave w takes w and, of them, 8 and 9
      for (int n = wave; n < 10; n += 8) {
        const int i = n >= 6 ? 3 : n >= 3 ? 2 : n >= 1 ? 1 : 0, j = n - i * (i + 1) / 2;
        const f32x4_t old = *sub(SD, i, j);
        f32x4_t c = ZERO, yl[4], xl[4];   // (summed up by itself: with `old` in the accumulator every partial sum is rounded at its size)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          yl[e] = *sub(SL, i, e);
          xl[e] = *sub(SL, j, e);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e) c = mm(c, yl[e], xl[e]);
        *sub(S0, i, j) = old - c;
      }
      if (wave >= 4 && last_of(1, 4)) flag_store(x.lflag + k + 1, ep32 | (u64)(k + 1));   // (they have one tile each: no time lost)
#ifdef DION_CHOL_TIMING
      if (t == 0 && p.dbg) p.dbg[8 * k + 2] = wall_clock64();
#endif
    }
    return;
  }

  // ------------------------------------------------------------------ a helper
  // (said to be the same in all lanes, so that everything that follows from them is scalar)
  const int team = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), t = threadIdx.x & 255;   // (within the team)
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  float* const S0 = S[3 * team];
  float* const S1 = S[3 * team + 1];
  float* const S2 = S[3 * team + 2];
  const int wm = wave & 1, wn = wave >> 1, lr = lane & 31, lk = lane >> 5;
  const int frow = wm * 32 + 4 * lk, fcol = wn * 32 + lr;
  const lane_off fo = 4u * (unsigned)(frow * ld + fcol);
  // The team's barrier: LDS operations of a wave are processed in issue order, so what its waves have read and written
  // before it is read and written when the count is full.
  int arrivals = 0;
  auto barrier = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    arrivals += 4;
    if (lane == 0) __hip_atomic_fetch_add(&arrived[team], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    while (*(chol_block::lds_counter*)&arrived[team] < arrivals) {}
    asm volatile("" ::: "memory");
  };
  // A wave that leaves because a wait was given up, by this team or the other one, leaves arrivals for all barriers to come: its
  // team's other waves, who may have looked at the word before it was set, must not wait for it.
  auto wait_team = [&](bool mine, auto ready) __attribute__((always_inline)) -> bool {
    const bool ok = wait_until(x, gave_up, mine, ready, barrier);
    if (!ok && lane == 0) __hip_atomic_fetch_add(&arrived[team], 1 << 24, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return ok;
  };
  // Ownership: the near-diagonal tiles and the copies of (i, i-2) as above; any other tile (i, j) to
  // team (i mod pr) pc + (j mod pc).
  const int teams = pr * pc, h = 2 * ((int)blockIdx.x - 1) + team, a = h / pc, b = h % pc;
  // Near-diagonal tasks that run at one time go to different workgroups: beside another team's products their own take twice
  // as long.  In which order: see near_order.
  const int near_x = ((int)blockIdx.x - 1 + p.near_shift) % (teams / 2);
  const int near_h = team * (teams / 2) + (p.near_far ? teams / 2 - 1 - near_x : near_x);
  auto near_of = [&](int i) __attribute__((always_inline)) {   // which d of row i is this team's (>= 3: none)
    const int d = (near_h - 3 * i) % teams;
    return d < 0 ? d + teams : d;
  };
  int s0_holds = -1;   // panel whose W11 is in S0
  // T(i, p): L[i][p] = C[i][p] W11(p)^T, published; leaves it in S1 as well
  auto column_tile = [&](int i, int p_) __attribute__((always_inline)) -> bool {
    barrier();   // earlier readers of S0 / S1 are through
    tile_to_lds(S1, tile_at(x.C, i, p_), ld, t);
    if (s0_holds != p_) {
      if (!wait_team(t == 0, [&] { return flag_load32(w11_flag(p_)) == ep; })) return false;
      tile_to_lds(S0, tile_at(x.W, p_, p_), ld, t);
      s0_holds = p_;
    }
    barrier();
    const f32x16_t li = mma_64(S1, S0, wm, wn, lr, lk);
    barrier();
    gfloat* dst = tile_at(x.L, i, p_);
#pragma unroll
    for (int v = 0; v < 16; ++v) S1[(frow + 8 * (v / 4) + (v % 4)) * CBP + fcol] = li[v];
    for_rows(dst, ld, [&](int v, gfloat* row) { shared_store(row, fo, li[v]); });
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    barrier();   // S1 is complete, everybody's stores have completed
    if (t == 0) flag_store(x.lflag + i, ep32 | (u64)(p_ + 1));
    return true;
  };
  // U(i, j, p): C[i][j] -= L[i][p] L[j][p]^T
  auto update = [&](int i, int j, int p_) __attribute__((always_inline)) {
    gfloat* ct = tile_at(x.C, i, j);
    float cold[16];
    tile_regs li, lj;
    // (all three tiles are requested before the first wait: one memory round trip per update, not three)
    for_rows(ct, ld, [&](int v, gfloat* row) { cold[v] = own_load(row, fo); });
    tile_to_regs(li, tile_at(x.L, i, p_), ld, t);
    tile_to_regs(lj, tile_at(x.L, j, p_), ld, t);
    barrier();   // earlier readers of S1 / S2 are through
    regs_to_lds<false>(S1, li, t);
    regs_to_lds<false>(S2, lj, t);
    barrier();
    const f32x16_t up = mma_64(S1, S2, wm, wn, lr, lk);
    for_rows(ct, ld, [&](int v, gfloat* row) { own_store(row, fo, cold[v] - up[v]); });
  };
  // this team's copy of (i, i-2) while panel p is worked on: the original has no update yet when p = 0
  auto copy_of = [&](int i, int d, int p_) __attribute__((always_inline)) { return p_ == 0 ? tile_at(x.C, i, i - 2) : tile_at(Tcopy, i, i - 2 + d); };
  // U(i, i-d, p) (d < 2), and U(i, i-2, p) on the copy
  auto near_update = [&](int i, int d, int p_) __attribute__((always_inline)) {
    gfloat* ct = tile_at(x.C, i, i - d);
    gfloat* from = copy_of(i, d, p_);
    gfloat* to = tile_at(Tcopy, i, i - 2 + d);
    float cold[16], cold2[16];
    tile_regs li, l2, l1;
    tile_to_regs(li, tile_at(x.L, i, p_), ld, t);
    tile_to_regs(l2, tile_at(x.L, i - 2, p_), ld, t);
    if (d == 1) tile_to_regs(l1, tile_at(x.L, i - 1, p_), ld, t);
    for_rows(from, ld, [&](int v, gfloat* row) { cold2[v] = own_load(row, fo); });
    if (d < 2) for_rows(ct, ld, [&](int v, gfloat* row) { cold[v] = shared_load(row, fo); });
    barrier();   // earlier readers of S0 / S1 / S2 are through
    regs_to_lds<false>(S1, li, t);
    regs_to_lds<false>(S2, l2, t);
    if (d == 1) {
      regs_to_lds<false>(S0, l1, t);
      s0_holds = -1;
    }
    barrier();
    if (d < 2) {
      const f32x16_t up = mma_64(S1, d ? S0 : S1, wm, wn, lr, lk);
      for_rows(ct, ld, [&](int v, gfloat* row) { shared_store(row, fo, cold[v] - up[v]); });
    }
    const f32x16_t up2 = mma_64(S1, S2, wm, wn, lr, lk);
    for_rows(to, ld, [&](int v, gfloat* row) { own_store(row, fo, cold2[v] - up2[v]); });
  };
  auto row_ready = [&](int row, int cols) __attribute__((always_inline)) {   // L[row][0 .. cols) are out
    const u64 v = flag_load(x.lflag + row);
    return (unsigned)(v >> 32) == (unsigned)x.epoch && (unsigned)v >= (unsigned)cols;
  };
  // ---- the inverse (FUSE_INV), in bf16 mode split into its halves, too: the triangular product reads those
  uint16_t* const wh = p.wh ? p.wh + 2 * mat : nullptr;
  uint16_t* const wl = p.wl + 2 * mat;
  auto w_ready = [&](int p_, int e) __attribute__((always_inline)) {   // tile (p_, e) of W is final
    return e == p_ ? flag_load32(w11_flag(p_)) == ep : flag_load(vflag + p_ * nb + e) == x.epoch;
  };
  // UW(j, e, p): W'(j, e) -= L[j][p] W(p, e); the first one, p = e, starts from zero
  auto w_update = [&](int j, int e, int p_) __attribute__((always_inline)) {
    gfloat* wt = tile_at(x.W, j, e);
    float cold[16];
    for_rows(wt, ld, [&](int v, gfloat* row) { cold[v] = p_ > e ? own_load(row, fo) : 0.f; });
    tile_regs lj, wp;
    tile_to_regs(lj, tile_at(x.L, j, p_), ld, t);
    tile_to_regs(wp, tile_at(x.W, p_, e), ld, t);
    barrier();   // earlier readers of S1 / S2 are through
    regs_to_lds<false>(S1, lj, t);
    regs_to_lds<true>(S2, wp, t);
    barrier();
    const f32x16_t up = mma_64(S1, S2, wm, wn, lr, lk);   // L[j][p] (W(p, e)^T)^T
    for_rows(wt, ld, [&](int v, gfloat* row) { own_store(row, fo, cold[v] - up[v]); });
  };
  // Row p_ of W into the running values of the rows from p_ + 2 down that this helper has tiles in (L[j][p_] is out:
  // the wait before the updates of panel p_ covers the rows j = a mod pr)
  auto w_rest = [&](int p_) __attribute__((always_inline)) -> bool {
    const int j0 = a + ((p_ + 2 - a + pr - 1) / pr) * pr;
    if (j0 >= nb || b > p_) return true;   // (uniform)
    if (!wait_team(t <= p_ && t % pc == b, [&] { return w_ready(p_, t); })) return false;
    for (int j = j0; j < nb; j += pr)
      for (int e = b; e <= p_; e += pc) w_update(j, e, p_);
    return true;
  };
  // Row p_ of W, for the tiles of it that this helper owns: their last update, then W(p_, e) = W11(p_) W'(p_, e)
  auto w_row = [&](int p_) __attribute__((always_inline)) -> bool {
    if (p_ < 1 || p_ % pr != a || b > p_ - 1) return true;   // (uniform)
    if (!wait_team(t < p_ && t % pc == b, [&] { return w_ready(p_ - 1, t); })) return false;
    if (!wait_team(t == 0, [&] { return row_ready(p_, p_); })) return false;
    for (int e = b; e < p_; e += pc) w_update(p_, e, p_ - 1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's parts of the running values are in memory
    for (int e = b; e < p_; e += pc) {
      gfloat* wt = tile_at(x.W, p_, e);
      float run[16];
      for_rows(wt, ld, [&](int v, gfloat* row) { run[v] = own_load(row, fo); });
      barrier();   // earlier readers of S0 / S1 are through
#pragma unroll
      for (int v = 0; v < 16; ++v) S1[fcol * CBP + frow + 8 * (v / 4) + (v % 4)] = run[v];   // W'(p_, e)^T
      if (s0_holds != p_) {
        if (!wait_team(t == 0, [&] { return flag_load32(w11_flag(p_)) == ep; })) return false;
        tile_to_lds(S0, tile_at(x.W, p_, p_), ld, t);
        s0_holds = p_;
      }
      barrier();
      const f32x16_t res = mma_64(S0, S1, wm, wn, lr, lk);   // W11(p_) W'(p_, e)
      for_rows(wt, ld, [&](int v, gfloat* row) { shared_store(row, fo, res[v]); });
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      barrier();   // everybody's stores have completed
      if (t == 0) flag_store(vflag + p_ * nb + e, x.epoch);
      if (wh) {   // (behind the flag: nobody in this launch waits for them)
        const long long at = (long long)(p_ * CB + frow) * ld + e * CB + fcol;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const long long o = at + (8 * (v / 4) + (v % 4)) * ld;
          const uint32_t h = pack_bf16x2(res[v], 0.f);
          gstore<uint16_t>(wh + o, (uint16_t)h);
          gstore<uint16_t>(wl + o, (uint16_t)pack_bf16x2(res[v] - bf16_lo(h), 0.f));
        }
      }
    }
    return true;
  };
  // the halves of W11(p_), by one team
  auto w_diag = [&](int p_) __attribute__((always_inline)) -> bool {
    if (!wh || p_ % pr != a || p_ % pc != b) return true;   // (uniform)
    if (!wait_team(t == 0, [&] { return flag_load32(w11_flag(p_)) == ep; })) return false;
    tile_regs w;
    tile_to_regs(w, tile_at(x.W, p_, p_), ld, t);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const long long o = (long long)(p_ * CB + (t >> 4) + 16 * q) * ld + p_ * CB + (t & 15) * 4;
      const f32x4_t f = w.v[q];
      const uint32_t h01 = pack_bf16x2(f[0], f[1]), h23 = pack_bf16x2(f[2], f[3]);
      gstore<u32x2_t>(wh + o, u32x2_t{h01, h23});
      gstore<u32x2_t>(wl + o, u32x2_t{pack_bf16x2(f[0] - bf16_lo(h01), f[1] - bf16_hi(h01)), pack_bf16x2(f[2] - bf16_lo(h23), f[3] - bf16_hi(h23))});
    }
    return true;
  };

  // L[t][.] is read by this team: as row or column of its other tiles, or as row i, i - 2, i - d of a near-diagonal task
  // (near_of(i + 1) = near_of(i) - 3; nine teams at least, so that the three rows of a task are told apart)
  const int dt = near_of(t);
  const bool reads_row = t % pr == a || t % pc == b || dt < 3 || dt == 4 || (dt >= 6 && dt < 9);
  int near0 = near_h;   // first near-diagonal task (3 i + d) of the rows that are left
  for (int p_ = 0; p_ + 1 < nb; ++p_) {
    // Row p_ + 2 feeds the chain: L[p_+2][p_] and with it the last update of the near-diagonal tile, before anything else of
    // this panel.
    const int d0 = near_of(p_ + 2);
    if (p_ + 2 < nb && d0 < 3) {
      // (What does not depend on W11(p_) is fetched before the wait for it, and one wait for all stores comes before the
      // flag: this path decides whether the chain finds its tiles ready.  L[p_+1][p_], which d = 1 needs as well, goes
      // out a microsecond after W11(p_): one wait for both.)
      const int i = p_ + 2, d = d0;
      barrier();   // earlier readers of S0 / S1 / S2 are through
      tile_to_lds(S1, copy_of(i, d, p_), ld, t);
      gfloat* ct = tile_at(x.C, i, i - d);
      float cold[16];
      tile_regs w11, lj;
      if (d < 2) {
        for_rows(ct, ld, [&](int v, gfloat* row) { cold[v] = shared_load(row, fo); });
      }
      if (!wait_team(t == 0, [&] { return d == 1 ? row_ready(p_ + 1, p_ + 1) : flag_load32(w11_flag(p_)) == ep; })) return;
      tile_to_regs(w11, tile_at(x.W, p_, p_), ld, t);
      if (d == 1) tile_to_regs(lj, tile_at(x.L, p_ + 1, p_), ld, t);
      regs_to_lds<false>(S0, w11, t);
      if (d == 1) regs_to_lds<false>(S2, lj, t);
      s0_holds = p_;
      barrier();
      const f32x16_t li = mma_64(S1, S0, wm, wn, lr, lk);   // L[i][p_]
      if (d < 2) {
        barrier();   // S1 has been read
#pragma unroll
        for (int v = 0; v < 16; ++v) S1[(frow + 8 * (v / 4) + (v % 4)) * CBP + fcol] = li[v];
        barrier();
        const f32x16_t up = mma_64(S1, d ? S2 : S1, wm, wn, lr, lk);
        for_rows(ct, ld, [&](int v, gfloat* row) { shared_store(row, fo, cold[v] - up[v]); });
      } else {
        gfloat* dst = tile_at(x.L, i, p_);
        for_rows(dst, ld, [&](int v, gfloat* row) { shared_store(row, fo, li[v]); });
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      barrier();   // everybody's stores have completed
      if (t == 0) {
        if (d == 2) {
          // (in this order: seeing the second flag, the chain goes on to raise the first one's count)
          flag_store(x.lflag + i, ep32 | (u64)(p_ + 1));
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        flag_store32(near_flag(i, d), ep);
      }
    }
    // the other tiles of column p_ that this team turns into tiles of L (three rows below the diagonal and further)
    if (p_ % pc == b)
      for (int i = a + ((p_ + 3 - a + pr - 1) / pr) * pr; i < nb; i += pr)
        if (!column_tile(i, p_)) return;
    // row p_ + 3, which is next to feed the chain, before the rest
    const int d1 = near_of(p_ + 3);
    if (p_ + 3 < nb && d1 < 3) {
      const int i = p_ + 3;
      if (!wait_team(t == i || t == i - 2 || (t == i - 1 && d1 == 1), [&] { return row_ready(t, p_ + 1); })) return;
      near_update(i, d1, p_);
    }
    // the inverse: row p_ - 1 of W into the rows from p_ + 1 down (kept until now so that it does not stand between
    // the previous panel and this one's look-ahead work), then this team's part of row p_
    if (FUSE_INV && p_ >= 1 && !w_rest(p_ - 1)) return;
    if (FUSE_INV && !w_row(p_)) return;
    if (FUSE_INV && !w_diag(p_)) return;
    // the tiles of L that this team's other updates of panel p_ need: one thread per block row (a superset)
    {
      const bool need = t > p_ && t < nb && reads_row;
      if (!wait_team(need, [&] { return row_ready(t, p_ + 1); })) return;
    }
    while (near0 < 3 * (p_ + 4)) near0 += teams;
    for (int n = near0; n < 3 * nb; n += teams) near_update(n / 3, n % 3, p_);
    // updates of the tiles three and more below the diagonal
    for (int j = b + ((p_ + 1 - b + pc - 1) / pc) * pc; j < nb; j += pc)
      for (int i = a + ((j + 3 - a + pr - 1) / pr) * pr; i < nb; i += pr) update(i, j, p_);
  }
  if (FUSE_INV && w_row(nb - 1)) w_diag(nb - 1);   // (row nb - 2 of W has no rows from nb down to go into)
}

hipError_t launch_chol_stream(CholStreamArgs p, int batch, hipStream_t s) {
  // 32 KB of unused dynamic LDS on top of the 52 KB the kernel declares: one workgroup per compute unit, so the
  // workgroup on the critical chain shares its unit with nobody
  if (p.chain) {
    // (102 KB of LDS: more than half of a compute unit's, so one workgroup each)
    // (the inverse needs a flag word per tile of W, and its waits one thread per panel; measured up to 64 panels)
    if (p.vflag_off > 0 && p.rp / CB > FUSED_INV_MAX_NB) return hipErrorInvalidValue;
    if (2 * p.pr * p.pc < 9) return hipErrorInvalidValue;   // (what `reads_row` takes for granted)
    const NearOrder order = near_order(p.rp / CB, p.pr, p.pc);
    p.near_far = order.far;
    p.near_shift = order.shift;
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(p.pr * p.pc + 1, batch), dim3(512), 0, s, p);
      return hipGetLastError();
    };
    if (p.thr) return p.vflag_off > 0 ? go(chol_chain_kernel<true, true>) : go(chol_chain_kernel<true, false>);
    return p.vflag_off > 0 ? go(chol_chain_kernel<false, true>) : go(chol_chain_kernel<false, false>);
  }
  if (p.thr) hipLaunchKernelGGL(chol_stream_kernel<true>, dim3(p.pr * p.pc, batch), dim3(256), 32768, s, p);
  else hipLaunchKernelGGL(chol_stream_kernel<false>, dim3(p.pr * p.pc, batch), dim3(256), 32768, s, p);
  return hipGetLastError();
}

hipError_t launch_chol_panel(CholPanelPtrs p, int batch, int k0, int rp, float piv_lo, float piv_hi, hipStream_t s) {
  const int nb = (rp - k0 - CB) / CB;
  const int tiles = nb * (nb + 1) / 2;
  auto go = [&](int blocks, int mode) {
    if (p.thr) hipLaunchKernelGGL(chol_panel_kernel<true>, dim3(blocks, batch), dim3(256), 0, s, p, k0, rp, piv_lo, piv_hi, mode);
    else hipLaunchKernelGGL(chol_panel_kernel<false>, dim3(blocks, batch), dim3(256), 0, s, p, k0, rp, piv_lo, piv_hi, mode);
    return hipGetLastError();
  };
  if ((long long)(1 + tiles) * batch <= 1024 || tiles == 0) return go(1 + tiles, 0);
  hipError_t e = go(1, 1);
  if (e != hipSuccess) return e;
  return go(tiles, 2);
}

}  // namespace dion
