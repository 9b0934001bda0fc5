// Complex FP64 products on the FP64 matrix cores, the main loop shared by every
// dense FP64 kernel of the library:
//     C_z(m, n) = sum_k A_z(m, k) B_z(n, k),   z = 0 .. batch - 1,
// on planar operands (separate re and im planes, row stride ld), both
// contiguous along k.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

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

// How B is stored: B_z(n, k) at row n, column k, or (B_TRANS) at row k, column n, so that
// C = A B^T reads a state-major block as the operator it stands for. B_SHIFTED: B_TRANS
// with a number subtracted from the diagonal.
enum BLayout { B_ROWS = 0, B_TRANS = 1, B_SHIFTED = 2 };

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
  bool few = false;  // few rows of A: take the kernels below rather than tiles
  bool tiles = false;  // tiles for more rows: sums over k in the same order in any block
  double sr = 0.0, si = 0.0;  // B_SHIFTED: subtracted from B's diagonal
};

// One workgroup computes a BM x BN complex tile with WGM x WGN waves. K is
// consumed in BK-wide stages through two LDS stages with one barrier each: the
// next stage is written from registers (loaded one stage earlier) while the
// waves multiply out of the current one. Within a stage, lane l reads the k
// pair (8p + 2(l/16), +1) of its row with one 16-byte LDS read and feeds two
// MFMA k-steps; A and B use the same k order, so the sum over k is unchanged.
// The staged 16-byte chunks of A and B are dealt to the threads as one list, so
// a tile may have fewer A chunks than threads.
//
// Three real products per k-step instead of four, T1 = Ar Br, T2 = Ai Bi,
// T3 = (Ar + Ai)(Br + Bi), Re = T1 - T2, Im = T3 - T1 - T2 (Gauss's complex
// multiplication). The sums Ar + Ai and Br + Bi are formed in registers from
// the fragments just read, so LDS keeps two planes per operand.
//
// HERM: C is known to be Hermitian: the grid holds the tiles on and above the
// diagonal and the epilogue writes each element above it twice.
//
// LB: with B_TRANS and B_SHIFTED the staging transposes B on the way into LDS. These
// products multiply dense operators, where the rounding of the running sums is the whole
// error: every 32 k the sums are added to totals and start again from zero (N = 256: 2.5
// times less error, as with the eight partial sums of zgemm_split_kernel; every 16 k gains
// no more and takes 46.9 us where this takes 44.2 and none 40.0: 32 products of 256 states).
template <int BM, int BN, int BK, int WGM, int WGN, bool CONJ_A, bool CONJ_B, int LB, bool HERM,
          int MINW, class Epi>
__global__ __launch_bounds__(WGM* WGN * 64, MINW) void zgemm_nt_f64_kernel(Operands op, Epi epi) {
  constexpr bool TRANS_B = LB != B_ROWS, FOLD = TRANS_B;
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
  static_assert(!FOLD || BK == 8 || BK == 16, "sums of 32 k");

  __shared__ __attribute__((aligned(16))) double sh[2][2][(BM + BN) * S];  // [stage][re, im]

  int tm, tn;
  if constexpr (HERM) {
    if (!tri_tile(blockIdx.x, op.tiles_n, tm, tn)) return;
  } else {
    tile_coords(blockIdx.x, op.tiles_m, op.tiles_n, tm, tn);
    if (tm >= op.tiles_m) return;  // grid padding
  }
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int wm = wid / WGN, wn = wid % WGN;
  const long ld = op.ld;

  d4 acc1[FM][FN], acc2[FM][FN], acc3[FM][FN];  // T1, T2, T3
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc1[i][j] = acc2[i][j] = acc3[i][j] = d4{0, 0, 0, 0};
  constexpr int TM = FOLD ? FM : 1, TN = FOLD ? FN : 1;
  d4 totR[TM][TN], totI[TM][TN];  // FOLD: Re, Im
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) totR[i][j] = totI[i][j] = d4{0, 0, 0, 0};

  // this thread's chunks: global addresses (at k = 0) and LDS offsets
  const double* gr[RC];
  const double* gi[RC];
  int lo[RC];
  bool of_a[RC];
  int diag[RC];  // B_SHIFTED: column minus row of a chunk's first element at k = 0
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
      diag[r] = n0 + nc - kr;
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
  auto lstore = [&](int st, int k0) {
#pragma unroll
    for (int r = 0; r < RC; ++r) {
      if constexpr (LB == B_SHIFTED) {
        if (!of_a[r] && (diag[r] == k0 || diag[r] + 1 == k0)) {
          const int e = diag[r] == k0 ? 0 : 1;
          vr[r][e] -= op.sr;
          vi[r][e] -= op.si;
        }
      }
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
  lstore(0, 0);
  if (nk > 1) gload(BK);
  __syncthreads();
  for (int kb = 0; kb < nk; ++kb) {
    const int cur = kb & 1;
    if (kb + 1 < nk) lstore(cur ^ 1, (kb + 1) * BK);  // that stage was last read before the previous barrier
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
      d2 fbs[FN];
#pragma unroll
      for (int j = 0; j < FN; ++j) fbs[j] = fbr[j] + fbi[j];
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const d2 fas = far_[i] + fai[i];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
          for (int j = 0; j < FN; ++j) acc1[i][j] = mfma_f64(far_[i][t], fbr[j][t], acc1[i][j]);
#pragma unroll
          for (int j = 0; j < FN; ++j) acc2[i][j] = mfma_f64(fai[i][t], fbi[j][t], acc2[i][j]);
#pragma unroll
          for (int j = 0; j < FN; ++j) acc3[i][j] = mfma_f64(fas[t], fbs[j][t], acc3[i][j]);
        }
      }
    }
    if constexpr (FOLD) {
      if ((kb + 1) % (32 / BK) == 0) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            totR[i % TM][j % TN] += acc1[i][j] - acc2[i][j];
            totI[i % TM][j % TN] += acc3[i][j] - acc1[i][j] - acc2[i][j];
            acc1[i][j] = acc2[i][j] = acc3[i][j] = d4{0, 0, 0, 0};
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
        double re, im;
        if constexpr (FOLD) {
          re = totR[i % TM][j % TN][r];
          im = totI[i % TM][j % TN][r];
        } else {
          const double t1 = acc1[i][j][r], t2 = acc2[i][j][r];
          re = t1 - t2;
          im = acc3[i][j][r] - t1 - t2;
        }
        if constexpr (HERM)
          epi.herm(m, n, re, im, mirror);
        else
          epi(m, n, re, im);
      }
  epi.finish();
}

// Epilogues that read another operand may load it ahead of the sum: prefetch(m, n).
template <class Epi, class = void>
struct HasPrefetch : std::false_type {};
template <class Epi>
struct HasPrefetch<Epi, std::void_t<decltype(&Epi::prefetch)>> : std::true_type {};

// The same product where tiles would leave most of the chip idle (few rows m
// against a large operator, small N): a workgroup takes 16 FM rows of A and 16
// rows of B, its W waves share the reduction in steps of 8 k and meet in LDS, and
// fragments go straight from global memory to registers. Against 32 x 32 tiles,
// whose four waves each walk the whole reduction behind a barrier per 16 k: N =
// 256, all rows, 13.1 -> 5.8 us; N = 512, 192 rows, 23.7 -> 13.2 us; N = 128 7.6
// -> 3.9 us. What bounds it is the vector memory path: a fragment load touches 16
// rows of 64 bytes (N = 2048, 16 rows: 31.8 us, the same without the MFMAs, 18 us
// without the loads of A). Splitting the reduction over workgroups as well loses
// to the device-scope fences that takes (124 us). HERM and LB as above.
template <int FM, int W, bool CONJ_A, bool CONJ_B, int LB, bool HERM, class Epi>
__global__ __launch_bounds__(W * 64) void zgemm_split_kernel(Operands op, Epi epi) {
  static_assert(!HERM || FM == 1, "Hermitian products take square tiles");
  static_assert(W * 64 >= FM * 256, "at most one element per thread");
  constexpr bool TRANS_B = LB != B_ROWS;
  __shared__ double red[W][FM * 8][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int tm = blockIdx.y, tn = blockIdx.x;
  if constexpr (HERM) tri_coords(blockIdx.x, tm, tn);
  const int m0 = tm * 16 * FM, n0 = tn * 16;
  // this thread's element of the result
  const int q = threadIdx.x, l = q & 63, qi = q >> 8, qr = (q >> 6) & 3;
  const int qm = m0 + 16 * qi + 4 * qr + (l >> 4), qn = n0 + (l & 15);
  epi.batch(blockIdx.z);
  if constexpr (HasPrefetch<Epi>::value)
    if (q < FM * 256) epi.prefetch(qm, qn);
  const int rr = lane & 15, kp = 2 * (lane >> 4);
  const long ld = op.ld;
  const int units = op.kdim / 8;
  const long bo = blockIdx.z * op.b_bs + (TRANS_B ? kp * ld + n0 + rr : (n0 + rr) * ld + kp);
  const double* br = op.br + bo;
  const double* bi = op.bi + bo;
  const long ao = blockIdx.z * op.a_bs + (m0 + rr) * ld + kp;
  const double* ar = op.ar + ao;
  const double* ai = op.ai + ao;
  d4 a1[FM], a2[FM], a3[FM];  // T1, T2, T3 of Gauss's three products
#pragma unroll
  for (int i = 0; i < FM; ++i) a1[i] = a2[i] = a3[i] = d4{0, 0, 0, 0};
#pragma unroll 8 / FM
  for (int u = wave; u < units; u += W) {
    const long k = 8L * u;
    d2 fbr, fbi;
    if constexpr (TRANS_B) {
      fbr = d2{br[k * ld], br[(k + 1) * ld]};
      fbi = d2{bi[k * ld], bi[(k + 1) * ld]};
      if constexpr (LB == B_SHIFTED) {
        const int e = n0 + rr - kp - (int)k;  // the diagonal element of this pair, if 0 or 1
        if (e == 0 || e == 1) {
          fbr[e] -= op.sr;
          fbi[e] -= op.si;
        }
      }
    } else {
      fbr = *reinterpret_cast<const d2*>(br + k);
      fbi = *reinterpret_cast<const d2*>(bi + k);
    }
    if constexpr (CONJ_B) fbi = -fbi;
    const d2 fbs = fbr + fbi;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const d2 fr = *reinterpret_cast<const d2*>(ar + 16L * i * ld + k);
      d2 fi = *reinterpret_cast<const d2*>(ai + 16L * i * ld + k);
      if constexpr (CONJ_A) fi = -fi;
      const d2 fs = fr + fi;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        a1[i] = mfma_f64(fr[t], fbr[t], a1[i]);
        a2[i] = mfma_f64(fi[t], fbi[t], a2[i]);
        a3[i] = mfma_f64(fs[t], fbs[t], a3[i]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      red[wave][8 * i + r][lane] = a1[i][r] - a2[i][r];
      red[wave][8 * i + 4 + r][lane] = a3[i][r] - a1[i][r] - a2[i][r];
    }
  __syncthreads();
  if (q < FM * 256) {
    const int v = 8 * qi + qr;
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      re += red[w][v][l];
      im += red[w][v + 4][l];
    }
    if constexpr (HERM)
      epi.herm(qm, qn, re, im, tm != tn);
    else
      epi(qm, qn, re, im);
  }
  epi.finish();
}

// Sums over the 64 lanes of N values per lane (N a power of two up to 64), by
// halving: at each step a lane keeps one half of its values and gets the other
// lane's share of them, so N - 1 exchanges and a few single ones replace 6 N.
// The sum of value i ends in v[0] of the lanes whose high bits are i.
template <int N, int O>
__device__ __forceinline__ void lane_sums(double* v, int lane) {
  if constexpr (N > 1) {
    constexpr int H = N / 2;
    const bool up = lane & O;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const double keep = up ? v[i + H] : v[i], send = up ? v[i] : v[i + H];
      v[i] = keep + __shfl_xor(send, O);
    }
    if constexpr (O > 1) lane_sums<H, O / 2>(v, lane);
  } else {
    v[0] += __shfl_xor(v[0], O);
    if constexpr (O > 1) lane_sums<1, O / 2>(v, lane);
  }
}

// Up to 8 rows m (S = 1, 2, 4, 8; 16 in two blocks): a wave takes 4 rows of B and
// S rows of A, its lanes consecutive k, so that every load is one contiguous
// KiB; W = 4 waves share k. Bound by reading B: N = 2048, 8 states 17.1 us
// (67 MB at 3.9 TB/s; 32 us on the matrix cores above, where half of the
// 16-row block is padding), N = 4096 49 us (5.5 TB/s, partly from the
// Infinity Cache), one state 11.4 and 38 us.
template <int S, class Epi>
__global__ __launch_bounds__(256) void zgemm_few_states_kernel(Operands op, Epi epi) {
  constexpr int R = 4, W = 4, V = 2 * S * R;
  __shared__ double red[W][V];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m0 = blockIdx.y * S, n0 = blockIdx.x * R;
  const long ld = op.ld;
  double c[V];  // (s, r): re, im
#pragma unroll
  for (int v = 0; v < V; ++v) c[v] = 0.0;
  for (int k = (wave * 64 + lane) * 2; k < op.kdim; k += W * 128) {
    d2 hr[R], hi[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      hr[r] = *reinterpret_cast<const d2*>(op.br + (long)(n0 + r) * ld + k);
      hi[r] = *reinterpret_cast<const d2*>(op.bi + (long)(n0 + r) * ld + k);
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const d2 xr = *reinterpret_cast<const d2*>(op.ar + (long)(m0 + s) * ld + k);
      const d2 xi = *reinterpret_cast<const d2*>(op.ai + (long)(m0 + s) * ld + k);
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          double& re = c[2 * (s * R + r)];
          double& im = c[2 * (s * R + r) + 1];
          re = fma(xr[t], hr[r][t], re);
          re = fma(-xi[t], hi[r][t], re);
          im = fma(xr[t], hi[r][t], im);
          im = fma(xi[t], hr[r][t], im);
        }
    }
  }
  lane_sums<V, 32>(c, lane);
  constexpr int per = 64 / V;  // lanes that hold the same sum
  if (lane % per == 0) red[wave][lane / per] = c[0];
  __syncthreads();
  epi.batch(0);
  const int q = threadIdx.x;
  if (q < S * R) {
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      re += red[w][2 * q];
      im += red[w][2 * q + 1];
    }
    epi(m0 + q / R, n0 + q % R, re, im);
  }
}

}  // namespace fq
