// Dense-operator kernels for gfx950: the Chebyshev products on FP64 matrix
// cores with the recurrence, the Bessel-weighted accumulation and the step
// phase fused into the epilogue, plus the O(N^2) helpers around them.
//
// Complex products use Gauss's three real MFMA products per operand pair on
// planar (real / imaginary) operands (zgemm_f64.h). Every product has the form
//     C(m, n) = sum_k A(m, k) B(n, k)
// with both operands contiguous along k ("NT"), which is what the state-major
// storage of the propagated block gives: A = P_l^T (row j = state j) and
// B = the rescaled Hamiltonian (row i = basis index i).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "epilogues.h"
#include "formats.h"
#include "internal.h"
#include "zgemm_f64.h"

namespace fq {
namespace {

// ---- epilogues ------------------------------------------------------------------------------

template <int KIND>
struct EpiCheb {
  ChebTerm t;
  long ld;
  __device__ __forceinline__ void batch(int) {}
  __device__ __forceinline__ void operator()(int m, int n, double ar, double ai) const {
    const long idx = (long)m * ld + n;
    if (KIND == CHEB_FIRST) {
      const double xr = t.p_re[idx], xi = t.p_im[idx];
      t.o_re[idx] = ar;
      t.o_im[idx] = ai;
      t.y_re[idx] = t.c0r * xr - t.c0i * xi + t.cr * ar - t.ci * ai;
      t.y_im[idx] = t.c0r * xi + t.c0i * xr + t.cr * ai + t.ci * ar;
    } else if (KIND == CHEB_FIRST_LAST) {
      const double xr = t.p_re[idx], xi = t.p_im[idx];
      if (t.save_re) {
        t.save_re[idx] = ar;
        t.save_im[idx] = ai;
      }
      const double sr = t.c0r * xr - t.c0i * xi + t.cr * ar - t.ci * ai;
      const double si = t.c0r * xi + t.c0i * xr + t.cr * ai + t.ci * ar;
      t.o_re[idx] = t.phr * sr - t.phi * si;
      t.o_im[idx] = t.phr * si + t.phi * sr;
    } else if (KIND == CHEB_MID) {
      const double pr = 2.0 * ar - t.p_re[idx], pi = 2.0 * ai - t.p_im[idx];
      t.o_re[idx] = pr;
      t.o_im[idx] = pi;
      t.y_re[idx] += t.cr * pr - t.ci * pi;
      t.y_im[idx] += t.cr * pi + t.ci * pr;
    } else {  // CHEB_LAST
      const double pr = 2.0 * ar - t.p_re[idx], pi = 2.0 * ai - t.p_im[idx];
      if (t.save_re) {
        t.save_re[idx] = pr;
        t.save_im[idx] = pi;
      }
      const double sr = t.y_re[idx] + t.cr * pr - t.ci * pi;
      const double si = t.y_im[idx] + t.cr * pi + t.ci * pr;
      t.o_re[idx] = t.phr * sr - t.phi * si;
      t.o_im[idx] = t.phr * si + t.phi * sr;
    }
  }
  __device__ __forceinline__ void finish() const {}
};

struct EpiStore {
  double* cr;
  double* ci;
  long ld;
  double alr, ali, ber, bei;
  __device__ __forceinline__ void batch(int) {}
  __device__ __forceinline__ void operator()(int m, int n, double ar, double ai) const {
    const long idx = (long)m * ld + n;
    double r = alr * ar - ali * ai, i = alr * ai + ali * ar;
    if (ber != 0.0 || bei != 0.0) {
      const double xr = cr[idx], xi = ci[idx];
      r += ber * xr - bei * xi;
      i += ber * xi + bei * xr;
    }
    cr[idx] = r;
    ci[idx] = i;
  }
  __device__ __forceinline__ void finish() const {}
};

// The larger of two values, NaN if either is one (fmax drops it).
__device__ __forceinline__ double max_or_nan(double a, double b) {
  return a > b || a != a ? a : b;
}

// The Gram matrix is Hermitian: an element above the diagonal's tiles counts twice. A NaN
// is carried to the maximum: its bits compare above those of every number there.
struct EpiUnitarity {
  int n;
  double* out;
  double mx = 0.0, ss = 0.0;
  __device__ __forceinline__ void batch(int) {}
  __device__ __forceinline__ void herm(int m, int c, double ar, double ai, bool mirror) {
    if (m < n && c < n) {
      const double dr = ar - (m == c ? 1.0 : 0.0);
      const double a2 = dr * dr + ai * ai;
      mx = max_or_nan(a2, mx);
      ss += mirror ? 2.0 * a2 : a2;
    }
  }
  __device__ void finish() {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      mx = max_or_nan(mx, __shfl_xor(mx, o));
      ss += __shfl_xor(ss, o);
    }
    if ((threadIdx.x & 63) == 0) {
      atomicMax(reinterpret_cast<unsigned long long*>(out), (unsigned long long)__double_as_longlong(sqrt(mx)));
      atomicAdd(out + 1, ss);
    }
  }
};

// ---- step operators as matrix polynomials ------------------------------------------------------
// All matrices of a batch lie at base + z * bs, re plane then im plane.

// O = 2 acc - f1 S1 - f2 S2 (each S optional), Hermitian: an element above the diagonal is
// also written below it.
struct EpiPolyT {
  double* o;
  const double *s1, *s2;
  long ld, plane, bs;
  double f1, f2;
  __device__ __forceinline__ void batch(int z) {
    o += z * bs;
    if (s1) s1 += z * bs;
    if (s2) s2 += z * bs;
  }
  __device__ __forceinline__ void herm(int m, int c, double ar, double ai, bool mirror) const {
    const long idx = (long)m * ld + c;
    double r = 2.0 * ar, i = 2.0 * ai;
    if (s1) {
      r -= f1 * s1[idx];
      i -= f1 * s1[plane + idx];
    }
    if (s2) {
      r -= f2 * s2[idx];
      i -= f2 * s2[plane + idx];
    }
    o[idx] = r;
    o[plane + idx] = i;
    if (mirror) {
      const long tdx = (long)c * ld + m;
      o[tdx] = r;
      o[plane + tdx] = -i;
    }
  }
  __device__ __forceinline__ void finish() const {}
};

// Clenshaw block and its adjoint: O = [O +] f acc + fa A - fs S (S optional, A the product's
// first operand).
struct EpiPolyBlock {
  double* o;
  const double *a, *sub;
  long ld, plane, bs, a_bs;
  double f, fa, fs;
  bool add;
  __device__ __forceinline__ void batch(int z) {
    o += z * bs;
    a += z * a_bs;
    if (sub) sub += z * bs;
  }
  __device__ __forceinline__ void operator()(int m, int c, double ar, double ai) const {
    const long idx = (long)m * ld + c;
    double r = f * ar, i = f * ai;
    if (fa != 0.0) {
      r = fma(fa, a[idx], r);
      i = fma(fa, a[plane + idx], i);
    }
    if (add) {
      r += o[idx];
      i += o[plane + idx];
    }
    if (sub) {
      r -= fs * sub[idx];
      i -= fs * sub[plane + idx];
    }
    o[idx] = r;
    o[plane + idx] = i;
  }
  __device__ __forceinline__ void finish() const {}
};

// O = acc + c0 X (X optional).
struct EpiPolyApply {
  double* o;
  const double* x;
  long ld, plane, bs, x_bs;
  PolyScalar c;
  double px = 0.0, pxi = 0.0;  // prefetched elements of X
  bool ahead = false;
  __device__ __forceinline__ void batch(int z) {
    o += z * bs;
    if (x) x += z * x_bs;
  }
  __device__ __forceinline__ void prefetch(int m, int n) {
    if (!x) return;
    const long idx = (long)m * ld + n;
    px = x[idx];
    pxi = x[plane + idx];
    ahead = true;
  }
  __device__ __forceinline__ void operator()(int m, int n, double ar, double ai) const {
    const long idx = (long)m * ld + n;
    if (x) {
      const double xr = ahead ? px : x[idx], xi = ahead ? pxi : x[plane + idx];
      ar = fma(c.r, xr, fma(-c.i, xi, ar));
      ai = fma(c.r, xi, fma(c.i, xr, ai));
    }
    o[idx] = ar;
    o[plane + idx] = ai;
  }
  __device__ __forceinline__ void finish() const {}
};

// ---- adjoint epilogues -----------------------------------------------------------------------
// A "stack" holds two state-major blocks as one 2np-row operand: rows [0, np)
// the forward term P_l, rows [np, 2np) the adjoint term Pbar_{l+1}.

// Tile of a product with t64 tiles of 64 x 64 (or 4 t64 of 32 x 32). Both take
// Gauss's three real products. 64 x 64 tiles run with eight waves of 32 x 16
// (90 VGPRs, 41 KB of LDS: two workgroups per CU): 84.7 TF/s algorithmic
// (63.5 TF/s of MFMA, 81 % of peak) at N = 4096, the rate that 128 x 128 tiles
// reached there with one workgroup per CU, and 831 us against 1103 us at
// N = 2048. 32 x 32 tiles (four waves of 16 x 16) reach 70 TF/s but fill the
// chip earlier: 425 us against 471 us at N = 1536, 80 against 91 us at 768, 13
// against 31 us at 256. Time per k in rounds of 256 workgroups, fitted on
// N = 256 .. 4096: 0.102 us a round (0.12 us for a single one) with 64 x 64
// tiles, 0.045 us and 0.029 us for each further round with 32 x 32 tiles.
inline bool take_tile64(long t64, long t32) {
  const long r64 = (t64 + 255) / 256, r32 = (t32 + 255) / 256;
  const double c64 = r64 == 1 ? 0.12 : 0.102 * (double)r64;
  const double c32 = 0.045 + 0.029 * (double)(r32 - 1);
  return c64 <= c32;
}

// Products of mrows x ncols (multiples of 16) per batch member that fit one
// round of one workgroup per CU in blocks of 16 x 16 or 32 x 16 share their
// reduction between waves instead of taking tiles: 16 rows first (N = 512: 128 rows
// 9.4 us, 13.1 us in blocks of 32, 23.7 us in 32 x 32 tiles), 32 while those fit
// (256 rows 13.4, 16.8 and 24.1 us). Beyond one round tiles are as good or better
// (N = 512, 512 rows: 24.5 us in each form; N = 768, 768 rows: 76 us in tiles, 81).
inline int split_rows(long m16, long n16, long batch) {
  if (m16 * n16 * batch <= 256) return 16;
  return (m16 + 1) / 2 * n16 * batch <= 256 ? 32 : 0;
}

template <int FM, bool CONJ_A, bool CONJ_B, int LB, class Epi>
hipError_t launch_split(const Operands& op, int mrows, int ncols, int batch, Epi epi,
                        hipStream_t s) {
  hipLaunchKernelGGL((zgemm_split_kernel<FM, 8, CONJ_A, CONJ_B, LB, false, Epi>),
                     dim3(ncols / 16, (mrows + 16 * FM - 1) / (16 * FM), batch), dim3(512), 0, s,
                     op, epi);
  return hipGetLastError();
}

// Few rows of A: 1, 2, 4, 8 or 16 of them on the vector units, 32, 48 or 64 on
// the matrix cores, in blocks of 16 rows or two once those take more than one
// round (N = 1536, 64 rows: 34 us against 45 us; N = 4096: 186 against 247 us; 32 x 32
// tiles 66 and 190 us). 16 rows as two blocks of 8: 14 us at N = 1024 (17 us on the
// matrix cores), equal at 2048.
template <class Epi>
hipError_t launch_few(const Operands& op, int mrows, int ncols, Epi epi, hipStream_t s) {
  const dim3 gs(ncols / 4, mrows > 8 ? mrows / 8 : 1);
  switch (mrows) {
    case 1: hipLaunchKernelGGL((zgemm_few_states_kernel<1, Epi>), gs, dim3(256), 0, s, op, epi); break;
    case 2: hipLaunchKernelGGL((zgemm_few_states_kernel<2, Epi>), gs, dim3(256), 0, s, op, epi); break;
    case 4: hipLaunchKernelGGL((zgemm_few_states_kernel<4, Epi>), gs, dim3(256), 0, s, op, epi); break;
    case 8:
    case 16: hipLaunchKernelGGL((zgemm_few_states_kernel<8, Epi>), gs, dim3(256), 0, s, op, epi); break;
    case 32:
    case 48:
    case 64:  // (48 rows: the second block's upper half is scratch rows below 64)
      return split_rows(mrows / 16, ncols / 16, 1) == 16
                 ? launch_split<1, false, false, B_ROWS>(op, mrows, ncols, 1, epi, s)
                 : launch_split<2, false, false, B_ROWS>(op, mrows, ncols, 1, epi, s);
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// C_z(m, n) over mrows x ncols (multiples of 64) for `batch` operand pairs.
template <bool CONJ_A, bool CONJ_B, int LB = B_ROWS, class Epi>
hipError_t launch_gemm(const Operands& op0, int mrows, int ncols, int batch, Epi epi,
                       hipStream_t s) {
  if (ncols % 64 != 0 || op0.kdim % 64 != 0 || batch < 1 || batch > 65535)
    return hipErrorInvalidValue;
  if constexpr (!CONJ_A && !CONJ_B && LB == B_ROWS)
    if (op0.few) return batch == 1 ? launch_few(op0, mrows, ncols, epi, s) : hipErrorInvalidValue;
  if (mrows % 64 != 0) return hipErrorInvalidValue;
  switch (op0.tiles ? 0 : split_rows(mrows / 16, ncols / 16, batch)) {
    case 16: return launch_split<1, CONJ_A, CONJ_B, LB>(op0, mrows, ncols, batch, epi, s);
    case 32: return launch_split<2, CONJ_A, CONJ_B, LB>(op0, mrows, ncols, batch, epi, s);
  }
  Operands op = op0;
  const long t64 = (long)(mrows / 64) * (ncols / 64) * batch;
  if (take_tile64(t64, 4 * t64)) {
    op.tiles_m = mrows / 64;
    op.tiles_n = ncols / 64;
    hipLaunchKernelGGL((zgemm_nt_f64_kernel<64, 64, 8, 2, 4, CONJ_A, CONJ_B, LB, false, 4,
                                            Epi>),
                       dim3(grid_rows(op.tiles_m) * op.tiles_n, batch), dim3(512), 0, s, op, epi);
  } else {
    op.tiles_m = mrows / 32;
    op.tiles_n = ncols / 32;
    hipLaunchKernelGGL((zgemm_nt_f64_kernel<32, 32, 16, 2, 2, CONJ_A, CONJ_B, LB, false, 1,
                                            Epi>),
                       dim3(grid_rows(op.tiles_m) * op.tiles_n, batch), dim3(256), 0, s, op, epi);
  }
  return hipGetLastError();
}

// The same for a Hermitian np x np result: the tiles on and above the diagonal
// (at N = 4096 3.82 ms against 6.49 ms for all tiles).
template <bool CONJ_A, bool CONJ_B, class Epi>
hipError_t launch_gemm_herm(const Operands& op0, int np, int batch, Epi epi, hipStream_t s) {
  if (np % 64 != 0 || op0.kdim % 16 != 0 || batch < 1 || batch > 65535)
    return hipErrorInvalidValue;
  const long a = np / 64, b = np / 32, c = np / 16;
  const long t64 = a * (a + 1) / 2, t32 = b * (b + 1) / 2, t16 = c * (c + 1) / 2;
  Operands op = op0;
  if (t16 * batch <= 256)
    hipLaunchKernelGGL((zgemm_split_kernel<1, 8, CONJ_A, CONJ_B, B_ROWS, true, Epi>),
                       dim3(t16, 1, batch), dim3(512), 0, s, op0, epi);
  else if (take_tile64(t64 * batch, t32 * batch)) {
    op.tiles_n = (int)a;
    hipLaunchKernelGGL((zgemm_nt_f64_kernel<64, 64, 8, 2, 4, CONJ_A, CONJ_B, B_ROWS, true, 4,
                                            Epi>),
                       dim3(tri_grid((int)a), batch), dim3(512), 0, s, op, epi);
  } else {
    op.tiles_n = (int)b;
    hipLaunchKernelGGL((zgemm_nt_f64_kernel<32, 32, 16, 2, 2, CONJ_A, CONJ_B, B_ROWS, true, 1,
                                            Epi>),
                       dim3(tri_grid((int)b), batch), dim3(256), 0, s, op, epi);
  }
  return hipGetLastError();
}

// ---- O(N^2) helpers ----------------------------------------------------------------------------

// Ht_z = (sum_j w_j(k) M_j - beta) / dE for the step k of every batch member z,
// two elements of a row per thread. Bound by HBM (or L2 for the small batched
// sizes): the planes of the operators in use are read once per member, Ht is
// written once. Operators whose weight vanishes over the whole drive (the
// commutator of a commutator-free scheme) are not in the list.
__global__ __launch_bounds__(256) void heff_kernel(HeffSum h, const double* __restrict__ w, int t,
                                                   double beta, double inv_dE, long n, long ld,
                                                   double* __restrict__ out, long bs) {
  const int z = blockIdx.y;
  const long k = (long)z * h.len0 + (z < h.rem ? z : h.rem) + t;
  const double* wk = w ? w + k * h.stride : nullptr;
  const long plane = ld * ld;
  double* o = out + z * bs;
  const long half = ld / 2, total = ld * half;  // padding included: zero in the operators
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < total;
       e += (long)gridDim.x * blockDim.x) {
    const long i = e / half, c = 2 * (e - i * half), idx = i * ld + c;
    double r0 = 0.0, r1 = 0.0, i0 = 0.0, i1 = 0.0;
    for (int j = 0; j < h.count; ++j) {
      const double wj = wk ? wk[h.slot[j]] : h.w[j];
      const d2 a = *reinterpret_cast<const d2*>(h.re[j] + idx);
      const d2 b = *reinterpret_cast<const d2*>(h.im[j] + idx);
      r0 = fma(wj, a[0], r0);
      r1 = fma(wj, a[1], r1);
      i0 = fma(wj, b[0], i0);
      i1 = fma(wj, b[1], i1);
    }
    if (i == c && i < n) r0 -= beta;
    if (i == c + 1 && i < n) r1 -= beta;
    *reinterpret_cast<d2*>(o + idx) = d2{r0 * inv_dE, r1 * inv_dE};
    *reinterpret_cast<d2*>(o + plane + idx) = d2{i0 * inv_dE, i1 * inv_dE};
  }
}

// Q_q = sum_{l=0..s} g_ql T_l for q < J, elementwise (T_0 = 1 on the n x n
// block); a Q may take the place of a T. Each T is read and each Q written once,
// padding included (the buffer of a Q may have held anything there).
__global__ __launch_bounds__(256) void poly_combine_kernel(PolyCombine p, long n, long ld, long bs) {
  const long plane = ld * ld;
  const long zo = blockIdx.y * bs;
  const long half = ld / 2, total = ld * half;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < total;
       e += (long)gridDim.x * blockDim.x) {
    const long i = e / half, c = 2 * (e - i * half), idx = zo + i * ld + c;
    d2 qr[kPolyMaxBlocks], qi[kPolyMaxBlocks];
#pragma unroll
    for (int q = 0; q < kPolyMaxBlocks; ++q) {
      const double d0 = i == c && i < n ? 1.0 : 0.0, d1 = i == c + 1 && i < n ? 1.0 : 0.0;
      qr[q] = d2{p.gr[q][0] * d0, p.gr[q][0] * d1};
      qi[q] = d2{p.gi[q][0] * d0, p.gi[q][0] * d1};
    }
    for (int l = 1; l <= p.s; ++l) {
      const d2 a = *reinterpret_cast<const d2*>(p.t[l - 1] + idx);
      const d2 b = *reinterpret_cast<const d2*>(p.t[l - 1] + plane + idx);
#pragma unroll
      for (int q = 0; q < kPolyMaxBlocks; ++q) {
        const double gr = p.gr[q][l], gi = p.gi[q][l];
        qr[q] += gr * a - gi * b;
        qi[q] += gr * b + gi * a;
      }
    }
#pragma unroll
    for (int q = 0; q < kPolyMaxBlocks; ++q)
      if (q < p.J) {
        *reinterpret_cast<d2*>(p.q[q] + idx) = qr[q];
        *reinterpret_cast<d2*>(p.q[q] + plane + idx) = qi[q];
      }
  }
}

// A <- (A + A^dagger) / 2 in place, by pairs of 32 x 32 tiles through LDS.
__global__ __launch_bounds__(256) void hermitian_part_kernel(double* __restrict__ a, long np,
                                                             long bs) {
  __shared__ double ur[32][33], ui[32][33], lr[32][33], li[32][33];
  if (blockIdx.x < blockIdx.y) return;
  double* const re = a + blockIdx.z * bs;
  double* const im = re + np * np;
  const long bi = blockIdx.y * 32L, bj = blockIdx.x * 32L;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8 threads
  for (int r = ty; r < 32; r += 8) {
    ur[r][tx] = re[(bi + r) * np + bj + tx];
    ui[r][tx] = im[(bi + r) * np + bj + tx];
    lr[r][tx] = re[(bj + r) * np + bi + tx];
    li[r][tx] = im[(bj + r) * np + bi + tx];
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    re[(bi + r) * np + bj + tx] = 0.5 * (ur[r][tx] + lr[tx][r]);
    im[(bi + r) * np + bj + tx] = 0.5 * (ui[r][tx] - li[tx][r]);
    if (bi != bj) {
      re[(bj + r) * np + bi + tx] = 0.5 * (lr[r][tx] + ur[tx][r]);
      im[(bj + r) * np + bi + tx] = 0.5 * (li[r][tx] - ui[tx][r]);
    }
  }
}

// out[count * k_z + j] += Re Tr(A_z B_j) for Hermitian B_j = planes at b_re + j *
// plane, b_im + j * plane; k_z as in heff_kernel, `stride` sums per step.
__global__ __launch_bounds__(256) void trace_dot_kernel(const double* __restrict__ a, long plane,
                                                        long bs, const double* __restrict__ b_re,
                                                        const double* __restrict__ b_im, int count,
                                                        int stride, int len0, int rem, int t,
                                                        double* __restrict__ out) {
  const int z = blockIdx.y, j = blockIdx.z;
  const long k = (long)z * len0 + (z < rem ? z : rem) + t;
  const double* ar = a + z * bs;
  const double* br = b_re + j * plane;
  const double* bi = b_im + j * plane;
  double s = 0.0;
  for (long e = 2 * (blockIdx.x * 256L + threadIdx.x); e < plane; e += 512L * gridDim.x) {
    const d2 x = *reinterpret_cast<const d2*>(ar + e), y = *reinterpret_cast<const d2*>(ar + plane + e);
    const d2 p = *reinterpret_cast<const d2*>(br + e), q = *reinterpret_cast<const d2*>(bi + e);
    s = fma(x[0], p[0], s);
    s = fma(x[1], p[1], s);
    s = fma(y[0], q[0], s);
    s = fma(y[1], q[1], s);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) atomicAdd(out + stride * k + j, s);
}

// dst = conj(src) on planar pairs.
__global__ void conj_planar_kernel(const double* __restrict__ src, long plane,
                                   double* __restrict__ dst) {
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < plane;
       e += (long)gridDim.x * blockDim.x) {
    dst[e] = src[e];
    dst[plane + e] = -src[plane + e];
  }
}

__global__ void pack_planar_kernel(const double2* __restrict__ src, long rows, long cols,
                                   long ld_src, double* __restrict__ re, double* __restrict__ im,
                                   long ld) {
  const long total = rows * cols;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < total;
       e += (long)gridDim.x * blockDim.x) {
    const long i = e / cols, j = e % cols;
    const double2 v = src[i * ld_src + j];
    re[i * ld + j] = v.x;
    im[i * ld + j] = v.y;
  }
}

// 32 x 32 tiles through LDS: planes(j, i) = src(i, j), zero outside the source.
template <class C>  // double2 (complex128) or float2 (complex64) source elements
__global__ void pack_planar_t_kernel(const C* __restrict__ src, long rows, long cols,
                                     long ld_src, double* __restrict__ re,
                                     double* __restrict__ im, long ld) {
  __shared__ double tr[32][33], ti[32][33];
  const long i0 = blockIdx.x * 32L, j0 = blockIdx.y * 32L;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 256 threads: ty 0..7
  for (int r = ty; r < 32; r += 8) {
    const long i = i0 + r, j = j0 + tx;
    double vr = 0.0, vi = 0.0;
    if (i < rows && j < cols) {
      const C v = src[i * ld_src + j];
      vr = v.x;
      vi = v.y;
    }
    tr[r][tx] = vr;
    ti[r][tx] = vi;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const long j = j0 + r, i = i0 + tx;
    if (i < ld) {
      re[j * ld + i] = tr[tx][r];
      im[j * ld + i] = ti[tx][r];
    }
  }
}

// dst(i, j) = planes(j, i).
template <class C>  // double2 (complex128) or float2 (complex64) destination elements
__global__ void unpack_planar_t_kernel(const double* __restrict__ re,
                                       const double* __restrict__ im, long ld, long rows,
                                       long cols, C* __restrict__ dst, long ld_dst) {
  __shared__ double tr[32][33], ti[32][33];
  const long j0 = blockIdx.y * 32L, i0 = blockIdx.x * 32L;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int r = ty; r < 32; r += 8) {
    const long j = j0 + r, i = i0 + tx;
    if (j < cols && i < rows) {
      tr[r][tx] = re[j * ld + i];
      ti[r][tx] = im[j * ld + i];
    }
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const long i = i0 + r, j = j0 + tx;
    if (i < rows && j < cols) {
      C v;
      v.x = tr[tx][r];
      v.y = ti[tx][r];
      dst[i * ld_dst + j] = v;
    }
  }
}

__global__ void identity_rows_kernel(double* __restrict__ re, double* __restrict__ im, long n,
                                     long m, long ld) {
  const long total = m * ld;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < total;
       e += (long)gridDim.x * blockDim.x) {
    const long j = e / ld, i = e % ld;
    re[e] = (i == j && j < n) ? 1.0 : 0.0;
    im[e] = 0.0;
  }
}

// dst = d * src on count elements of planar complex arrays.
__global__ void scale_planar_kernel(const double* __restrict__ sr, const double* __restrict__ si,
                                    double dr, double di, double* __restrict__ tr,
                                    double* __restrict__ ti, long count) {
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < count;
       e += (long)gridDim.x * blockDim.x) {
    const double xr = sr[e], xi = si[e];
    tr[e] = dr * xr - di * xi;
    ti[e] = dr * xi + di * xr;
  }
}

// ---- Lanczos ---------------------------------------------------------------------------------
// Per operator: 5 complex vectors (A q of this and the last step, three q's in
// rotation), then alpha, beta and the number of alphas once it is final.

// Sum over the workgroup's NT threads, the same value in each.
template <int NT>
__device__ __forceinline__ double wg_sum(double v, double* red) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  __syncthreads();  // (red may hold the last call's)
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  v = 0.0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) v += red[w];
  return v;
}

// End of step j - 1 and the product of step j in one launch: every workgroup
// forms alpha, w - alpha q - beta q', its norm and the next q by itself (the
// same sums in the same order, so they all stop alike), a thread keeping its EPT
// elements of q in registers, and then takes `rows` rows of A q. What it costs
// is the launch and the reductions, 5 to 6 us at N = 199 for both operators of a
// cover, against 18 us per operator with the vectors on the host (two copies, a
// product and a wait): both covers of the 199-state model in 1.3 ms instead of
// 7.2 ms. EPT = 0 (longer vectors): q comes from lanczos_update_kernel's launch.
template <int EPT>
__global__ __launch_bounds__(256) void lanczos_step_kernel(LanczosBatch b, int j, int ksteps,
                                                           int rows) {
  constexpr int NT = 256, RC = 4;
  __shared__ double red[NT / 64];
  __shared__ double rrow[NT / 64][2 * RC];
  const int t = threadIdx.x;
  const long n = b.n;
  double* st = b.state + blockIdx.y * b.stride;
  double* alpha = st + 10 * n;
  double* beta = alpha + ksteps;
  double* count = beta + ksteps;
  if (*count != 0.0) return;
  auto vec = [&](int i) { return reinterpret_cast<d2*>(st) + (long)i * n; };
  d2 q[EPT > 0 ? EPT : 1];
  const d2* qm = vec(2 + j % 3);
  if constexpr (EPT > 0) {
    if (j == 0) {
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const long k = t + (long)e * NT;
        q[e] = k < n ? qm[k] : d2{0.0, 0.0};
      }
    } else {
      const d2* w = vec((j - 1) & 1);
      const d2* q1 = vec(2 + (j - 1) % 3);
      const d2* q2 = vec(2 + (j + 1) % 3);
      const double bp = j >= 2 ? beta[j - 2] : 0.0;
      d2 p1[EPT];
      double a = 0.0, b2 = 0.0;
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const long k = t + (long)e * NT;
        q[e] = k < n ? w[k] : d2{0.0, 0.0};
        p1[e] = k < n ? q1[k] : d2{0.0, 0.0};
        a += p1[e][0] * q[e][0] + p1[e][1] * q[e][1];
      }
      a = wg_sum<NT>(a, red);
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const long k = t + (long)e * NT;
        q[e] -= a * p1[e];
        if (j >= 2 && k < n) q[e] -= bp * q2[k];
        b2 += q[e][0] * q[e][0] + q[e][1] * q[e][1];
      }
      const double bn = sqrt(wg_sum<NT>(b2, red));
      const bool stop = j == ksteps || bn <= 1e-13 * (fabs(a) + bp + 1e-300);
      if (blockIdx.x == 0 && t == 0) {
        alpha[j - 1] = a;
        if (stop)
          *count = j;
        else
          beta[j - 1] = bn;
      }
      if (stop) return;
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const long k = t + (long)e * NT;
        q[e] /= bn;
        if (blockIdx.x == 0 && k < n) vec(2 + j % 3)[k] = q[e];
      }
    }
  }
  const double* ar = b.re[blockIdx.y];
  const double* ai = b.im[blockIdx.y];
  d2* y = vec(j & 1);
  const long r1 = min(n, (blockIdx.x + 1L) * rows);
  for (long r0 = (long)blockIdx.x * rows; r0 < r1; r0 += RC) {
    double c[2 * RC];
#pragma unroll
    for (int v = 0; v < 2 * RC; ++v) c[v] = 0.0;
    auto add = [&](long k, d2 x) {
#pragma unroll
      for (int r = 0; r < RC; ++r) {
        const long o = min(r0 + r, n - 1) * b.ld + k;
        const double re = ar[o], im = ai[o];
        c[2 * r] += re * x[0] - im * x[1];
        c[2 * r + 1] += re * x[1] + im * x[0];
      }
    };
    if constexpr (EPT > 0) {
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const long k = t + (long)e * NT;
        if (k < n) add(k, q[e]);
      }
    } else {
      for (long k = t; k < n; k += NT) add(k, qm[k]);
    }
    lane_sums<2 * RC, 32>(c, t & 63);  // value v in the lanes 8 v ..
    __syncthreads();                   // (rrow may hold the last rows')
    if ((t & 7) == 0) rrow[t >> 6][(t & 63) >> 3] = c[0];
    __syncthreads();
    if (t < RC && r0 + t < r1) {
      d2 s{0.0, 0.0};
#pragma unroll
      for (int w = 0; w < NT / 64; ++w) s += d2{rrow[w][2 * t], rrow[w][2 * t + 1]};
      y[r0 + t] = s;
    }
  }
}

// The end of step j - 1 (see lanczos_step_kernel) for vectors of any length, one
// workgroup per operator.
__global__ __launch_bounds__(1024) void lanczos_update_kernel(LanczosBatch b, int j, int ksteps) {
  constexpr int NT = 1024;
  __shared__ double red[NT / 64];
  const long n = b.n;
  double* st = b.state + blockIdx.x * b.stride;
  double* alpha = st + 10 * n;
  double* beta = alpha + ksteps;
  double* count = beta + ksteps;
  if (*count != 0.0) return;
  auto vec = [&](int i) { return reinterpret_cast<d2*>(st) + (long)i * n; };
  d2* w = vec((j - 1) & 1);
  const d2* q1 = vec(2 + (j - 1) % 3);
  const d2* q2 = vec(2 + (j + 1) % 3);
  const double bp = j >= 2 ? beta[j - 2] : 0.0;
  double a = 0.0, b2 = 0.0;
  for (long k = threadIdx.x; k < n; k += NT) a += q1[k][0] * w[k][0] + q1[k][1] * w[k][1];
  a = wg_sum<NT>(a, red);
  for (long k = threadIdx.x; k < n; k += NT) {
    d2 v = w[k] - a * q1[k];
    if (j >= 2) v -= bp * q2[k];
    w[k] = v;
    b2 += v[0] * v[0] + v[1] * v[1];
  }
  const double bn = sqrt(wg_sum<NT>(b2, red));
  const bool stop = j == ksteps || bn <= 1e-13 * (fabs(a) + bp + 1e-300);
  if (threadIdx.x == 0) {
    alpha[j - 1] = a;
    if (stop)
      *count = j;
    else
      beta[j - 1] = bn;
  }
  if (stop) return;
  for (long k = threadIdx.x; k < n; k += NT) vec(2 + j % 3)[k] = w[k] / bn;
}

// H0 = diag(e) into zeroed planes of row stride ld.
__global__ void diag_planar_kernel(const double* __restrict__ e, long n, long ld,
                                   double* __restrict__ re) {
  const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (i < n) re[i * ld + i] = e[i];
}

// B = s i [diag(e), Q] elementwise: B_ij = s i (e_i - e_j) Q_ij for i, j < n.
__global__ void diag_commutator_kernel(const double* __restrict__ e, long n, long ld,
                                       const double* __restrict__ qr,
                                       const double* __restrict__ qi, double s,
                                       double* __restrict__ br, double* __restrict__ bi) {
  const long total = n * n;
  for (long t = blockIdx.x * (long)blockDim.x + threadIdx.x; t < total;
       t += (long)gridDim.x * blockDim.x) {
    const long i = t / n, j = t % n, idx = i * ld + j;
    const double d = s * (e[i] - e[j]);
    const double xr = qr[idx], xi = qi[idx];
    br[idx] = -d * xi;
    bi[idx] = d * xr;
  }
}

// out = sum_j w_j M_j elementwise over planar matrices (the per-step part of
// the sixth-order effective Hamiltonian).
__global__ void weighted_sum_kernel(WeightedSum ws, long total, double* __restrict__ outr,
                                    double* __restrict__ outi) {
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < total;
       e += (long)gridDim.x * blockDim.x) {
    double sr = 0.0, si = 0.0;
    for (int j = 0; j < ws.count; ++j) {
      sr = fma(ws.w[j], ws.re[j][e], sr);
      si = fma(ws.w[j], ws.im[j][e], si);
    }
    outr[e] = sr;
    outi[e] = si;
  }
}

// Energy expectation of state rows (state-major planes, row m = state m):
// avg[m] += w * sum_i Re(conj(x_mi) y_mi) / sum_i |x_mi|^2 with y = H x in
// the same layout; one workgroup per state, i < n.
__global__ void energy_rows_kernel(const double* __restrict__ xr, const double* __restrict__ xi,
                                   const double* __restrict__ yr, const double* __restrict__ yi,
                                   long n, long ld, double w, double* __restrict__ avg) {
  __shared__ double sn[256], sd[256];
  const long m = blockIdx.x;
  double num = 0.0, den = 0.0;
  for (long i = threadIdx.x; i < n; i += blockDim.x) {
    const long e = m * ld + i;
    const double a = xr[e], b = xi[e];
    num += a * yr[e] + b * yi[e];
    den += a * a + b * b;
  }
  sn[threadIdx.x] = num;
  sd[threadIdx.x] = den;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      sn[threadIdx.x] += sn[threadIdx.x + o];
      sd[threadIdx.x] += sd[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) avg[m] += w * sn[0] / sd[0];
}

__global__ void fill_zero_kernel(double* __restrict__ p, long count) {
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < count;
       e += (long)gridDim.x * blockDim.x)
    p[e] = 0.0;
}

// ---------------------------------------------------------------------------------------
// Whole chain for N <= 64 in one launch. The columns of U_T are independent
// propagations (Sec. 5: the identity is split into blocks of columns), so each
// workgroup takes 16 states (rows of the state-major block) through its steps
// on its own. A build splits the chain into gridDim.y segments of consecutive
// steps, each propagating the identity (N / 16 CUs alone would work otherwise:
// 2274 us per 100-step build in one segment); the segments' operators are multiplied up
// afterwards. Per step a workgroup forms Ht_k = (H0 + a_k V + b_k K - beta) / dE in
// LDS, runs the L Chebyshev terms with its 16 x 64 block of P_{l-1}, P_l in
// LDS, keeps its share of the sum Y of the terms from P_1 on in registers (the large one,
// c_0 X, is added once, last), and ends the step with X_k = exp(-i beta h) (c_0 X + Y) in LDS
// (the phase in two parts: one part would be off alike in every step). One barrier per term, none between
// workgroups; the only HBM traffic is the operators (L2-resident, 192 KB) and
// the block of X read once and written once.
// Wave j computes output columns i = 16 j .. 16 j + 15 of each product
// C(s, i) = sum_k P(s, k) Ht(i, k) with four real products per k-step on the
// 16x16x4 FP64 matrix cores; lane l then owns states 4 r + l / 16 and column
// 16 j + l % 16 of every term, so P_{l+1} overwrites P_{l-1} element by
// element in place.
// ---------------------------------------------------------------------------------------
constexpr int kSmallN = 64, kSmallS = 16, kSmallLd = 65;  // padded LDS rows: no bank conflicts

__global__ __launch_bounds__(256) void small_chain_kernel(SmallChain c) {
  __shared__ double hs[2][kSmallN * kSmallLd];            // Ht re, im
  __shared__ double ps[2][2][kSmallS * kSmallLd];         // two P buffers [buf][re, im]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int s0 = blockIdx.x * kSmallS;                    // first state of this workgroup
  const int n = c.n;
  const long ld = c.ld;
  // this segment's steps; segments other than a single one start from the identity
  const int seg = blockIdx.y;
  const int k_lo = c.k0 + seg * c.len0 + (seg < c.rem ? seg : c.rem);
  const int k_hi = gridDim.y > 1 ? k_lo + c.len0 + (seg < c.rem ? 1 : 0) : c.k1;
  double* const xre = c.xr + seg * c.bs;
  double* const xim = c.xi + seg * c.bs;
  // the block of X (rows s0 .. s0 + 15 of the state-major planes) into buffer 0
  for (int e = tid; e < kSmallS * kSmallN; e += 256) {
    const int s = e / kSmallN, k = e % kSmallN;
    const bool one = s0 + s == k && k < n;
    ps[0][0][s * kSmallLd + k] =
        gridDim.y > 1 ? (one ? 1.0 : 0.0) : xre[(long)(s0 + s) * ld + k];
    ps[0][1][s * kSmallLd + k] = gridDim.y > 1 ? 0.0 : xim[(long)(s0 + s) * ld + k];
  }
  const int ci = 16 * wave + (lane & 15);  // output column i of this lane
  const int kq = lane >> 4;                // k within a 4-step of the matrix cores
  const int L = c.L;
  int cur = 0;                             // buffer holding X_k (then P_l)
  for (int k = k_lo; k < k_hi; ++k) {
    const double a = c.ab[2 * k], b = c.ab[2 * k + 1];
    __syncthreads();  // the previous step's last writes; Ht no longer read
    for (int e = tid; e < kSmallN * kSmallN; e += 256) {
      const int i = e / kSmallN, kk = e % kSmallN;
      double re = 0.0, im = 0.0;
      if (i < n && kk < n) {
        const long g = (long)i * ld + kk;
        re = c.h0r[g] + a * c.vr[g] + b * c.kr[g];
        im = c.h0i[g] + a * c.vi[g] + b * c.ki[g];
        if (i == kk) re -= c.beta;
        re *= c.inv_dE;
        im *= c.inv_dE;
      }
      hs[0][i * kSmallLd + kk] = re;
      hs[1][i * kSmallLd + kk] = im;
    }
    __syncthreads();
    double yr[4], yi[4], x0r[4], x0i[4];
    const int prv = cur ^ 1;  // P_{l-1} buffer (P_0 = X stays in `cur` for the first term)
    for (int l = 0; l < L; ++l) {
      // acc = Ht P_l for this lane's four (state, column) pairs; P_l in buffer `src`
      const int src = (l == 0) ? cur : ((l & 1) ? prv : cur);
      const double* pr = ps[src][0];
      const double* pi = ps[src][1];
      d4 accR = d4{0, 0, 0, 0}, accI = d4{0, 0, 0, 0};
#pragma unroll
      for (int k4 = 0; k4 < kSmallN; k4 += 4) {
        const int kk = k4 + kq;
        const double ar = pr[(lane & 15) * kSmallLd + kk], ai = pi[(lane & 15) * kSmallLd + kk];
        const double br = hs[0][ci * kSmallLd + kk], bi = hs[1][ci * kSmallLd + kk];
        accR = mfma_f64(ar, br, accR);
        accR = mfma_f64(-ai, bi, accR);
        accI = mfma_f64(ar, bi, accI);
        accI = mfma_f64(ai, br, accI);
      }
      // term l + 1 from acc: P_1 = acc, P_{l+1} = 2 acc - P_{l-1}; the old
      // P_{l-1} (or X) sits where P_{l+1} goes, read and written by this lane only
      const int dst = (l == 0) ? prv : ((l & 1) ? cur : prv);
      const double cr = c.coef[2 * (l + 1)], cim = c.coef[2 * (l + 1) + 1];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = 4 * r + kq;
        const int idx = s * kSmallLd + ci;
        double vr, vi;
        if (l == 0) {
          vr = accR[r];
          vi = accI[r];
          const double xr = ps[cur][0][idx], xi = ps[cur][1][idx];
          x0r[r] = xr;
          x0i[r] = xi;
          yr[r] = yi[r] = 0.0;
        } else {
          vr = 2.0 * accR[r] - ps[dst][0][idx];
          vi = 2.0 * accI[r] - ps[dst][1][idx];
        }
        yr[r] += cr * vr - cim * vi;
        yi[r] += cr * vi + cim * vr;
        if (l + 1 < L) {
          ps[dst][0][idx] = vr;
          ps[dst][1][idx] = vi;
        }
      }
      if (l + 1 < L) __syncthreads();  // P_{l+1} complete before the next product reads it
    }
    // X_k = ph Y into the buffer the last product did not read: every wave must
    // be done with that product first
    const int last_src = (L == 1) ? cur : (((L - 1) & 1) ? prv : cur);
    const int xb = last_src ^ 1;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int idx = (4 * r + kq) * kSmallLd + ci;
      const double sr = c.coef[0] * x0r[r] - c.coef[1] * x0i[r] + yr[r];
      const double si = c.coef[0] * x0i[r] + c.coef[1] * x0r[r] + yi[r];
      ps[xb][0][idx] = fma(c.phr, sr, fma(-c.phi, si, c.phr_lo * sr - c.phi_lo * si));
      ps[xb][1][idx] = fma(c.phr, si, fma(c.phi, sr, c.phr_lo * si + c.phi_lo * sr));
    }
    cur = xb;
  }
  __syncthreads();
  for (int e = tid; e < kSmallS * kSmallN; e += 256) {
    const int s = e / kSmallN, k = e % kSmallN;
    xre[(long)(s0 + s) * ld + k] = ps[cur][0][s * kSmallLd + k];
    xim[(long)(s0 + s) * ld + k] = ps[cur][1][s * kSmallLd + k];
  }
}

inline unsigned grid_for(long total, int block) {
  long g = (total + block - 1) / block;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (unsigned)g;
}

// dst(j, i) = src(i, j) (+ d on the diagonal of the n x n block) through 32 x 32 LDS tiles
// (one padding column).
__global__ __launch_bounds__(256) void transpose_planar_kernel(const double* __restrict__ sr,
                                                               const double* __restrict__ si,
                                                               double* __restrict__ dr,
                                                               double* __restrict__ di, long np,
                                                               long bs, long n, double d_re,
                                                               double d_im) {
  __shared__ double tr[32][33], ti[32][33];
  sr += blockIdx.z * bs;
  si += blockIdx.z * bs;
  dr += blockIdx.z * bs;
  di += blockIdx.z * bs;
  const long bi = blockIdx.y * 32L, bj = blockIdx.x * 32L;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8 threads
  for (int r = ty; r < 32; r += 8) {
    tr[r][tx] = sr[(bi + r) * np + bj + tx];
    ti[r][tx] = si[(bi + r) * np + bj + tx];
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const bool diag = bj + r == bi + tx && bj + r < n;
    dr[(bj + r) * np + bi + tx] = tr[tx][r] + (diag ? d_re : 0.0);
    di[(bj + r) * np + bi + tx] = ti[tx][r] + (diag ? d_im : 0.0);
  }
}

}  // namespace

hipError_t launch_cheb_f64(const ChebTerm& t, int mrows, int np, hipStream_t s) {
  Operands op{t.a_re, t.a_im, t.b_re, t.b_im, np, np, 0, 0, 0, 0, mrows <= 64 && mrows < np, t.tiles};
  switch (t.kind) {
    case CHEB_FIRST:
      return launch_gemm<false, false>(op, mrows, np, 1, EpiCheb<CHEB_FIRST>{t, np}, s);
    case CHEB_FIRST_LAST:
      return launch_gemm<false, false>(op, mrows, np, 1, EpiCheb<CHEB_FIRST_LAST>{t, np}, s);
    case CHEB_MID:
      return launch_gemm<false, false>(op, mrows, np, 1, EpiCheb<CHEB_MID>{t, np}, s);
    case CHEB_LAST:
      return launch_gemm<false, false>(op, mrows, np, 1, EpiCheb<CHEB_LAST>{t, np}, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_adj_step(const double* ar, const double* ai, int mrows, const double* htr,
                           const double* hti, double* sr, double* si, const double* lr,
                           const double* li, double dr, double di, double fac, int row_off, int np,
                           hipStream_t s) {
  Operands op{ar, ai, htr, hti, np, np, 0, 0, 0, 0};
  EpiAdjStep e{sr, si, lr, li, dr, di, fac, np, row_off};
  return launch_gemm<false, false>(op, mrows, np, 1, e, s);
}

hipError_t launch_adj_dot(const double* pr, const double* pi, const double* dr_, const double* di_,
                          int ncols, const double* pbr, const double* pbi, double w, double* out,
                          int np, hipStream_t s) {
  Operands op{pr, pi, dr_, di_, np, np, 0, 0, 0, 0};
  EpiAdjDot e{pbr, pbi, out, np, w};
  return launch_gemm<false, false>(op, np, ncols, 1, e, s);
}

hipError_t launch_zgemm_nt_f64(const double* ar, const double* ai, bool conj_a, const double* br,
                               const double* bi, bool conj_b, double* cr, double* ci, int mrows,
                               int ncols, int kdim, int ld, double alr, double ali, double ber,
                               double bei, hipStream_t s) {
  Operands op{ar, ai, br, bi, ld, kdim, 0, 0, 0, 0, mrows <= 64 && mrows < ncols};
  EpiStore e{cr, ci, ld, alr, ali, ber, bei};
  if (conj_a && conj_b) return launch_gemm<true, true>(op, mrows, ncols, 1, e, s);
  if (conj_a) return launch_gemm<true, false>(op, mrows, ncols, 1, e, s);
  if (conj_b) return launch_gemm<false, true>(op, mrows, ncols, 1, e, s);
  return launch_gemm<false, false>(op, mrows, ncols, 1, e, s);
}

hipError_t launch_unitarity_f64(const double* xr, const double* xi, int n, int np, double* out,
                                hipStream_t s) {
  Operands op{xr, xi, xr, xi, np, np, 0, 0, 0, 0};
  EpiUnitarity e{n, out};
  return launch_gemm_herm<true, false>(op, np, 1, e, s);
}

hipError_t launch_pack_planar(const void* src, long rows, long cols, long ld_src, double* re,
                              double* im, long ld, hipStream_t s) {
  hipLaunchKernelGGL(pack_planar_kernel, dim3(grid_for(rows * cols, 256)), dim3(256), 0, s,
                     reinterpret_cast<const double2*>(src), rows, cols, ld_src, re, im, ld);
  return hipGetLastError();
}

hipError_t launch_pack_planar_t(const void* src, long rows, long cols, long ld_src, double* re,
                                double* im, long ld, long mrows, bool c64, hipStream_t s) {
  if (mrows % 32 != 0 || ld % 32 != 0) return hipErrorInvalidValue;
  dim3 grid((unsigned)(ld / 32), (unsigned)(mrows / 32));
  if (c64)
    hipLaunchKernelGGL(pack_planar_t_kernel<float2>, grid, dim3(256), 0, s,
                       reinterpret_cast<const float2*>(src), rows, cols, ld_src, re, im, ld);
  else
    hipLaunchKernelGGL(pack_planar_t_kernel<double2>, grid, dim3(256), 0, s,
                       reinterpret_cast<const double2*>(src), rows, cols, ld_src, re, im, ld);
  return hipGetLastError();
}

hipError_t launch_unpack_planar_t(const double* re, const double* im, long ld, long rows,
                                  long cols, void* dst, long ld_dst, bool c64, hipStream_t s) {
  dim3 grid((unsigned)((rows + 31) / 32), (unsigned)((cols + 31) / 32));
  if (c64)
    hipLaunchKernelGGL(unpack_planar_t_kernel<float2>, grid, dim3(256), 0, s, re, im, ld, rows,
                       cols, reinterpret_cast<float2*>(dst), ld_dst);
  else
    hipLaunchKernelGGL(unpack_planar_t_kernel<double2>, grid, dim3(256), 0, s, re, im, ld, rows,
                       cols, reinterpret_cast<double2*>(dst), ld_dst);
  return hipGetLastError();
}

hipError_t launch_identity_rows(double* re, double* im, long n, long m, long ld, hipStream_t s) {
  hipLaunchKernelGGL(identity_rows_kernel, dim3(grid_for(m * ld, 256)), dim3(256), 0, s, re, im,
                     n, m, ld);
  return hipGetLastError();
}

hipError_t launch_heff_f64(const HeffSum& h, const double* w, int t, int batch, double beta,
                           double dE, long n, long ld, double* out, long bs, hipStream_t s) {
  if (h.count < 1 || h.count > kHeffTerms || batch < 1 || batch > 65535 || ld % 2 != 0 ||
      (!w && batch != 1))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(heff_kernel, dim3(grid_for(ld * (ld / 2), 256), batch), dim3(256), 0, s, h, w,
                     t, beta, 1.0 / dE, n, ld, out, bs);
  return hipGetLastError();
}

hipError_t launch_poly_t(const double* ta, const double* tb, const double* s1, double f1,
                         const double* s2, double f2, double* out, int np, long bs, int batch,
                         hipStream_t s) {
  const long plane = (long)np * np;
  // T_b(k, c) = conj(T_b(c, k))
  Operands op{ta, ta + plane, tb, tb + plane, np, np, 0, 0, bs, bs};
  return launch_gemm_herm<false, true>(op, np, batch, EpiPolyT{out, s1, s2, np, plane, bs, f1, f2}, s);
}

hipError_t launch_poly_combine(const PolyCombine& p, long n, long ld, long bs, int batch,
                               hipStream_t s) {
  if (p.s < 1 || p.s > kPolyMaxS || p.J < 1 || p.J > kPolyMaxBlocks || batch < 1 || batch > 65535)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(poly_combine_kernel, dim3(grid_for(ld * (ld / 2), 256), batch), dim3(256), 0,
                     s, p, n, ld, bs);
  return hipGetLastError();
}

hipError_t launch_poly_block(const double* a, long a_bs, const double* b, long b_bs, bool b_herm,
                             double f, double fa, const double* sub, double fs, bool add,
                             double* out, long o_bs, int np, int batch, hipStream_t s) {
  const long plane = (long)np * np;
  Operands op{a, a + plane, b, b + plane, np, np, 0, 0, a_bs, b_bs};
  const EpiPolyBlock e{out, a, sub, np, plane, o_bs, a_bs, f, fa, fs, add};
  // (A B)(m, c) = sum_k A(m, k) B(k, c), B(k, c) = conj(B(c, k)) when Hermitian
  return b_herm ? launch_gemm<false, true>(op, np, np, batch, e, s)
                : launch_gemm<false, false, B_TRANS>(op, np, np, batch, e, s);
}

hipError_t launch_hermitian_part(double* a, int np, long bs, int batch, hipStream_t s) {
  if (np < 32 || np % 32 != 0 || np / 32 > 65535 || batch < 1 || batch > 65535)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(hermitian_part_kernel,
                     dim3((unsigned)(np / 32), (unsigned)(np / 32), (unsigned)batch), dim3(256), 0,
                     s, a, np, bs);
  return hipGetLastError();
}

hipError_t launch_trace_dot(const double* a, int np, long bs, int batch, const double* b_re,
                            const double* b_im, int count, int stride, int len0, int rem, int t,
                            double* out, hipStream_t s) {
  const long plane = (long)np * np;
  if (np % 2 != 0 || batch < 1 || batch > 65535 || count < 1) return hipErrorInvalidValue;
  const unsigned gx = (unsigned)std::min<long>(64, (plane / 2 + 255) / 256);
  hipLaunchKernelGGL(trace_dot_kernel, dim3(gx, batch, count), dim3(256), 0, s, a, plane, bs, b_re,
                     b_im, count, stride, len0, rem, t, out);
  return hipGetLastError();
}

hipError_t launch_conj_planar(const double* src, int np, double* dst, hipStream_t s) {
  const long plane = (long)np * np;
  hipLaunchKernelGGL(conj_planar_kernel, dim3(grid_for(plane, 256)), dim3(256), 0, s, src, plane,
                     dst);
  return hipGetLastError();
}

hipError_t launch_poly_apply(const double* x, long x_bs, const double* e, long e_bs, int e_layout,
                             const PolyScalar& c0, const double* base, long base_bs, double* out,
                             long o_bs, int mrows, int np, int batch, hipStream_t s) {
  const long plane = (long)np * np;
  Operands op{x, x + plane, e, e + plane, np, np, 0, 0, x_bs, e_bs, mrows <= 64 && mrows < np};
  const EpiPolyApply epi{out, base, np, plane, o_bs, base_bs, c0};
  switch (e_layout) {
    case POLY_OPERATOR: return launch_gemm<false, false>(op, mrows, np, batch, epi, s);
    case POLY_STATES: return launch_gemm<false, false, B_TRANS>(op, mrows, np, batch, epi, s);
    case POLY_STATES_SHIFTED:
      if (base != x || base_bs != x_bs) return hipErrorInvalidValue;
      op.sr = c0.r;
      op.si = c0.i;
      return launch_gemm<false, false, B_SHIFTED>(op, mrows, np, batch, epi, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_scale_planar(const double* sr, const double* si, double dr, double di,
                               double* tr, double* ti, long count, hipStream_t s) {
  hipLaunchKernelGGL(scale_planar_kernel, dim3(grid_for(count, 256)), dim3(256), 0, s, sr, si, dr,
                     di, tr, ti, count);
  return hipGetLastError();
}

hipError_t launch_lanczos_step(const LanczosBatch& b, int j, int ksteps, hipStream_t s) {
  if (b.n < 1 || b.ld < b.n || b.count < 1 || b.count > kLanczosOps || j < 0 || j > ksteps)
    return hipErrorInvalidValue;
  if (j > 0 && b.n > 4096)
    hipLaunchKernelGGL(lanczos_update_kernel, dim3(b.count), dim3(1024), 0, s, b, j, ksteps);
  // one row per workgroup until they fill the chip twice, then blocks of four
  const long per = (b.n * b.count + 511) / 512;
  const int rows = per == 1 ? 1 : (int)((per + 3) / 4 * 4);
  // (the end of the last step needs no product)
  const dim3 grid(j == ksteps ? 1 : (unsigned)((b.n + rows - 1) / rows), b.count);
  if (b.n <= 256)
    hipLaunchKernelGGL(lanczos_step_kernel<1>, grid, dim3(256), 0, s, b, j, ksteps, rows);
  else if (b.n <= 1024)
    hipLaunchKernelGGL(lanczos_step_kernel<4>, grid, dim3(256), 0, s, b, j, ksteps, rows);
  else if (b.n <= 4096)
    hipLaunchKernelGGL(lanczos_step_kernel<16>, grid, dim3(256), 0, s, b, j, ksteps, rows);
  else if (j < ksteps)
    hipLaunchKernelGGL(lanczos_step_kernel<0>, grid, dim3(256), 0, s, b, j, ksteps, rows);
  return hipGetLastError();
}

hipError_t launch_energy_rows(const double* xr, const double* xi, const double* yr,
                              const double* yi, long rows, long n, long ld, double w, double* avg,
                              hipStream_t s) {
  if (rows < 1 || n < 1 || ld < n || rows > 0x7fffffffL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(energy_rows_kernel, dim3((unsigned)rows), dim3(256), 0, s, xr, xi, yr, yi, n,
                     ld, w, avg);
  return hipGetLastError();
}

hipError_t launch_diag_planar(const double* e, long n, long ld, double* re, hipStream_t s) {
  if (n < 1 || ld < n) return hipErrorInvalidValue;
  hipLaunchKernelGGL(diag_planar_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, e, n,
                     ld, re);
  return hipGetLastError();
}

hipError_t launch_diag_commutator(const double* e, long n, long ld, const double* qr,
                                  const double* qi, double sgn, double* br, double* bi,
                                  hipStream_t s) {
  if (n < 1 || ld < n) return hipErrorInvalidValue;
  hipLaunchKernelGGL(diag_commutator_kernel, dim3(grid_for(n * n, 256)), dim3(256), 0, s, e, n,
                     ld, qr, qi, sgn, br, bi);
  return hipGetLastError();
}

long small_chain_max_n() { return kSmallN; }

hipError_t launch_small_chain(const SmallChain& c, int mrows, int nseg, hipStream_t s) {
  if (nseg < 1 || nseg > 65535 ||
      (nseg > 1 && (long)nseg * c.len0 + c.rem != (long)c.k1 - c.k0))
    return hipErrorInvalidValue;
  if (c.ld != kSmallN || mrows < kSmallS || mrows % kSmallS || mrows > kSmallN || c.n > kSmallN ||
      c.L < 1 || c.k0 < 0 || c.k1 < c.k0)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(small_chain_kernel, dim3(mrows / kSmallS, nseg), dim3(256), 0, s, c);
  return hipGetLastError();
}

hipError_t launch_fill_zero(double* p, long count, hipStream_t s) {
  if (count < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for(count, 256)), dim3(256), 0, s, p, count);
  return hipGetLastError();
}

hipError_t launch_weighted_sum(const WeightedSum& ws, long total, double* outr, double* outi,
                               hipStream_t s) {
  if (ws.count < 1 || ws.count > kMaxSumTerms || total < 1) return hipErrorInvalidValue;
  for (int j = 0; j < ws.count; ++j)
    if (!ws.re[j] || !ws.im[j]) return hipErrorInvalidValue;
  hipLaunchKernelGGL(weighted_sum_kernel, dim3(grid_for(total, 256)), dim3(256), 0, s, ws, total,
                     outr, outi);
  return hipGetLastError();
}

hipError_t launch_transpose_planar(const double* sr, const double* si, double* dr, double* di,
                                   long np, long bs, int batch, hipStream_t s, long n, double d_re,
                                   double d_im) {
  if (np < 32 || np % 32 != 0 || np / 32 > 65535 || batch < 1 || batch > 65535)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(transpose_planar_kernel,
                     dim3((unsigned)(np / 32), (unsigned)(np / 32), (unsigned)batch), dim3(256), 0,
                     s, sr, si, dr, di, np, bs, n, d_re, d_im);
  return hipGetLastError();
}

}  // namespace fq
