// Complex FP64 products on the FP64 matrix cores, the main loop shared by every
// dense FP64 kernel of the library:
//     C_z(m, n) = sum_k A_z(m, k) B_z(n, k),   z = 0 .. batch - 1,
// on planar operands (separate re and im planes, row stride ld), both
// contiguous along k.
#pragma once

#include <hip/hip_runtime.h>

#include "formats.h"

namespace fq {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ d4 mfma_f64(double a, double b, d4 c) {
  // D(16x16) += A(16x4) B(4x16); lane l supplies A(l%16, kq(l)) and
  // B(kq(l), l%16) with kq(l) = l/16, and holds D(4*r + l/16, l%16), r = 0..3
  // (layout measured with one-hot operands on gfx950).
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

struct Operands {
  const double* ar;
  const double* ai;
  const double* br;
  const double* bi;
  int ld;       // row stride of A and B (elements)
  int kdim;     // reduction length, multiple of BK
  int tiles_n;  // tiles along n
  int tiles_m;
  long a_bs;    // batch strides (elements) of A and B: operand z at + z * stride
  long b_bs;
};

// Tile (tm, tn), tm <= tn, number t of the upper triangle of a tiles x tiles
// grid, column by column.
__device__ __forceinline__ void tri_coords(int t, int& tm, int& tn) {
  int c = (int)((__builtin_sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
  while ((c + 1) * (c + 2) / 2 <= t) ++c;
  while (c * (c + 1) / 2 > t) --c;
  tn = c;
  tm = t - c * (c + 1) / 2;
}

// One workgroup computes a BM x BN complex tile with WGM x WGN waves. K is
// consumed in BK-wide stages through two LDS stages with one barrier each: the
// next stage is written from registers (loaded one stage earlier) while the
// waves multiply out of the current one. Within a stage, lane l reads the k
// pair (8p + 2(l/16), +1) of its row with one 16-byte LDS read and feeds two
// MFMA k-steps; A and B use the same k order, so the sum over k is unchanged.
// The staged 16-byte chunks of A and B are dealt to the threads as one list, so
// a tile may have fewer A chunks than threads.
//
// GAUSS: three real products per k-step instead of four, T1 = Ar Br, T2 = Ai Bi,
// T3 = (Ar + Ai)(Br + Bi), Re = T1 - T2, Im = T3 - T1 - T2 (Gauss's complex
// multiplication). The sums Ar + Ai and Br + Bi are formed in registers from
// the fragments just read, so LDS keeps two planes per operand.
//
// HERM: C is known to be Hermitian: the grid holds the tiles on and above the
// diagonal and the epilogue writes each element above it twice.
//
// TRANS_B: B is stored transposed, B_z(n, k) at row k, column n (so that
// C = A B^T reads a state-major block as the operator it stands for); the
// staging transposes it on the way into LDS.
template <int BM, int BN, int BK, int WGM, int WGN, bool CONJ_A, bool CONJ_B, bool TRANS_B,
          bool GAUSS, bool HERM, int MINW, class Epi>
__global__ __launch_bounds__(WGM* WGN * 64, MINW) void zgemm_nt_f64_kernel(Operands op, Epi epi) {
  constexpr int NT = WGM * WGN * 64;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int FM = WTM / 16, FN = WTN / 16;
  constexpr int S = BK + 2;    // LDS row stride (doubles): conflict-free 16-byte reads
  constexpr int CPR = BK / 2;  // 16-byte chunks per row
  constexpr int RC = (BM + BN) * CPR / NT;  // chunks per thread and plane
  static_assert((BM + BN) * CPR % NT == 0, "load split");
  static_assert(BM * CPR % 64 == 0, "a wave's chunks belong to one operand");
  static_assert(BK % 8 == 0, "BK");
  static_assert(!HERM || BM == BN, "Hermitian products take square tiles");

  __shared__ __attribute__((aligned(16))) double sh[2][2][(BM + BN) * S];  // [stage][re, im]

  int tm, tn;
  if constexpr (HERM) {
    tri_coords(blockIdx.x, tm, tn);
  } else {
    tile_coords(blockIdx.x, op.tiles_m, op.tiles_n, tm, tn);
    if (tm >= op.tiles_m) return;  // grid padding
  }
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int wm = wid / WGN, wn = wid % WGN;
  const long ld = op.ld;

  // 4M: accR = Re, accI = Im; GAUSS: accR = T1, accI = T2, accS = T3
  constexpr int SM = GAUSS ? FM : 1, SN = GAUSS ? FN : 1;
  d4 accR[FM][FN], accI[FM][FN], accS[SM][SN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      accR[i][j] = d4{0, 0, 0, 0};
      accI[i][j] = d4{0, 0, 0, 0};
    }
#pragma unroll
  for (int i = 0; i < SM; ++i)
#pragma unroll
    for (int j = 0; j < SN; ++j) accS[i][j] = d4{0, 0, 0, 0};

  // this thread's chunks: global addresses (at k = 0) and LDS offsets
  const double* gr[RC];
  const double* gi[RC];
  int lo[RC];
  bool of_a[RC];
#pragma unroll
  for (int r = 0; r < RC; ++r) {
    const int c = tid + r * NT, row = c / CPR, col = 2 * (c % CPR);
    const bool is_a = row < BM;
    long off = is_a ? (long)(m0 + row) * ld + col + blockIdx.y * op.a_bs
                    : (long)(n0 + row - BM) * ld + col + blockIdx.y * op.b_bs;
    lo[r] = row * S + col;
    if (TRANS_B && !is_a) {  // chunk: columns n, n + 1 of one row k
      const int cb = c - BM * CPR, kr = cb / (BN / 2), nc = 2 * (cb % (BN / 2));
      off = (long)kr * ld + n0 + nc + blockIdx.y * op.b_bs;
      lo[r] = (BM + nc) * S + kr;
    }
    gr[r] = (is_a ? op.ar : op.br) + off;
    gi[r] = (is_a ? op.ai : op.bi) + off;
    of_a[r] = is_a;
  }
  d2 vr[RC], vi[RC];
  auto gload = [&](int k0) {
#pragma unroll
    for (int r = 0; r < RC; ++r) {
      const long step = TRANS_B && !of_a[r] ? (long)k0 * ld : (long)k0;
      vr[r] = *reinterpret_cast<const d2*>(gr[r] + step);
      vi[r] = *reinterpret_cast<const d2*>(gi[r] + step);
    }
  };
  auto lstore = [&](int st) {
#pragma unroll
    for (int r = 0; r < RC; ++r) {
      const bool neg = of_a[r] ? CONJ_A : CONJ_B;
      const d2 im = neg ? -vi[r] : vi[r];
      if (TRANS_B && !of_a[r]) {
        sh[st][0][lo[r]] = vr[r][0];
        sh[st][0][lo[r] + S] = vr[r][1];
        sh[st][1][lo[r]] = im[0];
        sh[st][1][lo[r] + S] = im[1];
      } else {
        *reinterpret_cast<d2*>(&sh[st][0][lo[r]]) = vr[r];
        *reinterpret_cast<d2*>(&sh[st][1][lo[r]]) = im;
      }
    }
  };

  const int nk = op.kdim / BK;
  gload(0);
  lstore(0);
  if (nk > 1) gload(BK);
  __syncthreads();
  for (int kb = 0; kb < nk; ++kb) {
    const int cur = kb & 1;
    if (kb + 1 < nk) lstore(cur ^ 1);  // that stage was last read before the previous barrier
    if (kb + 2 < nk) gload((kb + 2) * BK);
    const int rr = lane & 15;
#pragma unroll
    for (int p = 0; p < BK / 8; ++p) {
      const int kk = 8 * p + 2 * (lane >> 4);
      d2 far_[FM], fai[FM], fbr[FN], fbi[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const int row = wm * WTM + i * 16 + rr;
        far_[i] = *reinterpret_cast<const d2*>(&sh[cur][0][row * S + kk]);
        fai[i] = *reinterpret_cast<const d2*>(&sh[cur][1][row * S + kk]);
      }
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int row = BM + wn * WTN + j * 16 + rr;
        fbr[j] = *reinterpret_cast<const d2*>(&sh[cur][0][row * S + kk]);
        fbi[j] = *reinterpret_cast<const d2*>(&sh[cur][1][row * S + kk]);
      }
      if constexpr (GAUSS) {
        d2 fbs[FN];
#pragma unroll
        for (int j = 0; j < FN; ++j) fbs[j] = fbr[j] + fbi[j];
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          const d2 fas = far_[i] + fai[i];
#pragma unroll
          for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int j = 0; j < FN; ++j) accR[i][j] = mfma_f64(far_[i][t], fbr[j][t], accR[i][j]);
#pragma unroll
            for (int j = 0; j < FN; ++j) accI[i][j] = mfma_f64(fai[i][t], fbi[j][t], accI[i][j]);
#pragma unroll
            for (int j = 0; j < FN; ++j)
              accS[i % SM][j % SN] = mfma_f64(fas[t], fbs[j][t], accS[i % SM][j % SN]);
          }
        }
      } else {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) accR[i][j] = mfma_f64(far_[i][t], fbr[j][t], accR[i][j]);
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) accI[i][j] = mfma_f64(far_[i][t], fbi[j][t], accI[i][j]);
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) accR[i][j] = mfma_f64(-fai[i][t], fbi[j][t], accR[i][j]);
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) accI[i][j] = mfma_f64(fai[i][t], fbr[j][t], accI[i][j]);
        }
      }
    }
    __syncthreads();
  }

  epi.batch(blockIdx.y);
  const bool mirror = HERM && tm != tn;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm * WTM + i * 16 + 4 * r + (lane >> 4);
        const int n = n0 + wn * WTN + j * 16 + (lane & 15);
        double re = accR[i][j][r], im = accI[i][j][r];
        if constexpr (GAUSS) {
          const double t1 = re, t2 = im;
          re = t1 - t2;
          im = accS[i % SM][j % SN][r] - t1 - t2;
        }
        if constexpr (HERM)
          epi.herm(m, n, re, im, mirror);
        else
          epi(m, n, re, im);
      }
  epi.finish();
}

}  // namespace fq
