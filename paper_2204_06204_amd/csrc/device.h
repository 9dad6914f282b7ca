// Device helpers: deterministic FP64 reductions, SIMP scaling, node loads
// and the element product in the sum/difference basis.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace fbto {

// --------------------------------------------------------------------------
// FP64 reductions with a fixed summation order (deterministic run to run).
// --------------------------------------------------------------------------
// Wave-wide sum / max of a double with DPP lane moves (no LDS traffic):
// xor-1 and xor-2 within quads, mirrors within 8 and 16 lanes, then the
// row broadcasts fold the four 16-lane rows into lane 63, which is read
// back as a wave-uniform value.  The order of operations is fixed.
// DPP and readlane read all 64 lanes whatever the execution mask, so every
// kernel that reduces this way is launched with whole waves (a partial last
// wave would mix in the stale registers of its missing lanes).
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_move(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  const int rlo = __builtin_amdgcn_update_dpp(0, lo, CTRL, ROWMASK, 0xf, false);
  const int rhi = __builtin_amdgcn_update_dpp(0, hi, CTRL, ROWMASK, 0xf, false);
  return __hiloint2double(rhi, rlo);
}
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_move<0xB1, 0xf>(v);    // quad_perm [1,0,3,2]
  v += dpp_move<0x4E, 0xf>(v);    // quad_perm [2,3,0,1]
  v += dpp_move<0x141, 0xf>(v);   // row_half_mirror
  v += dpp_move<0x140, 0xf>(v);   // row_mirror: every lane holds its row's sum
  v += dpp_move<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp_move<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, dpp_move<0xB1, 0xf>(v));
  v = fmax(v, dpp_move<0x4E, 0xf>(v));
  v = fmax(v, dpp_move<0x141, 0xf>(v));
  v = fmax(v, dpp_move<0x140, 0xf>(v));
  // rows not written by a broadcast receive 0 from dpp_move; max with a
  // non-negative or -inf identity needs the real value, so fold explicitly
  const double b15 = dpp_move<0x142, 0xa>(v);
  v = ((__lane_id() >> 4) & 1) ? fmax(v, b15) : v;
  const double b31 = dpp_move<0x143, 0xc>(v);
  v = (__lane_id() >= 32) ? fmax(v, b31) : v;
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
  return __hiloint2double(hi, lo);
}

// Reduce NV values over the block: entry i is a sum, or a max when bit i of
// MAXMASK is set.  The result is returned to every thread.
template <int NV, unsigned MAXMASK>
__device__ __forceinline__ void block_reduce(double (&v)[NV]) {
  __shared__ double sh[NV][16];
  const int nthr = blockDim.x * blockDim.y * blockDim.z;
  const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
  const int lane = tid & 63, w = tid >> 6, nw = (nthr + 63) >> 6;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const double x = ((MAXMASK >> i) & 1u) ? wave_max(v[i]) : wave_sum(v[i]);
    if (lane == 0) sh[i][w] = x;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    double acc = sh[i][0];
    for (int k = 1; k < nw; ++k) acc = ((MAXMASK >> i) & 1u) ? fmax(acc, sh[i][k]) : acc + sh[i][k];
    v[i] = acc;
  }
  __syncthreads();
}

// The same for a block of NTHR threads (a multiple of 64) through LDS: the
// values are stored, then 16 lanes per value fold a strided sixteenth of the
// block's entries each and a row-wise DPP butterfly joins the 16 lanes.
// Every thread does about NV + NTHR / 16 operations, against some 20 per
// value and wave for the DPP reduction of every value above.  The order of
// operations is fixed.  lds: reduce_lds_words values of LDS.  A kernel that
// reduces more than once can hand every call the same ones (an array declared
// in here would be a further one for each), with a barrier before a call if
// other threads may still read what lies there.
template <int NV, int NTHR>
__host__ __device__ constexpr int reduce_lds_words() { return NV * (NTHR + 1); }
template <int NV, unsigned MAXMASK, int NTHR>
__device__ __forceinline__ void block_reduce_lds(double (&v)[NV], double* lds) {
  static_assert(NTHR % 64 == 0 && NTHR <= 1024, "whole waves");
  constexpr int SEG = NTHR / 16;
  double* const res = lds + NV * NTHR;
  const int tid = threadIdx.x;
#pragma unroll
  for (int i = 0; i < NV; ++i) lds[i * NTHR + tid] = v[i];
  __syncthreads();
  for (int t = tid; t < NV * 16; t += NTHR) {  // rows of 16 lanes: one value each
    const int i = t >> 4, l = t & 15;
    const bool is_max = (MAXMASK >> i) & 1u;
    double acc = lds[i * NTHR + l];
#pragma unroll
    for (int j = 1; j < SEG; ++j) {
      const double x = lds[i * NTHR + l + 16 * j];
      acc = is_max ? fmax(acc, x) : acc + x;
    }
    const double a1 = dpp_move<0xB1, 0xf>(acc);   // quad_perm [1,0,3,2]
    acc = is_max ? fmax(acc, a1) : acc + a1;
    const double a2 = dpp_move<0x4E, 0xf>(acc);   // quad_perm [2,3,0,1]
    acc = is_max ? fmax(acc, a2) : acc + a2;
    const double a3 = dpp_move<0x141, 0xf>(acc);  // row_half_mirror
    acc = is_max ? fmax(acc, a3) : acc + a3;
    const double a4 = dpp_move<0x140, 0xf>(acc);  // row_mirror: every lane holds the row's result
    acc = is_max ? fmax(acc, a4) : acc + a4;
    if (l == 0) res[i] = acc;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = res[i];
}
template <int NV, unsigned MAXMASK, int NTHR>
__device__ __forceinline__ void block_reduce_lds(double (&v)[NV]) {
  __shared__ double lds[reduce_lds_words<NV, NTHR>()];
  block_reduce_lds<NV, MAXMASK, NTHR>(v, lds);
}

// Reduce NV arrays of per-block partials (entry i: n[i] values at src[i];
// sum, or max where bit i of MAXMASK is set).  Every block computes the same
// result in the same order; the producing kernel has finished, so plain
// loads see its stores.  Each round loads two entries per thread of every
// array before folding any, so that the arrays cost one memory latency per
// round, not one each.
template <int NV, unsigned MAXMASK>
__device__ __forceinline__ void fold_parts(double (&v)[NV], const double* const (&src)[NV], const int (&n)[NV]) {
  const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
  const int nthr = blockDim.x * blockDim.y * blockDim.z;
  int nmax = 0;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    nmax = n[i] > nmax ? n[i] : nmax;
    v[i] = ((MAXMASK >> i) & 1u) ? -INFINITY : 0.0;
  }
  for (int k = tid; k - tid < nmax; k += 2 * nthr) {
    double x[NV][2];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const double id = ((MAXMASK >> i) & 1u) ? -INFINITY : 0.0;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int kk = k + u * nthr;
        x[i][u] = kk < n[i] ? src[i][kk] : id;
      }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int u = 0; u < 2; ++u) v[i] = ((MAXMASK >> i) & 1u) ? fmax(v[i], x[i][u]) : v[i] + x[i][u];
  }
}
template <int NV, unsigned MAXMASK, int NTHR = 0>
__device__ __forceinline__ void reduce_parts(double (&v)[NV], const double* const (&src)[NV],
                                             const int (&n)[NV]) {
  fold_parts<NV, MAXMASK>(v, src, n);
  if constexpr (NTHR > 0) block_reduce_lds<NV, MAXMASK, NTHR>(v);
  else block_reduce<NV, MAXMASK>(v);
}
template <int NV, unsigned MAXMASK, int NTHR>
__device__ __forceinline__ void reduce_parts(double (&v)[NV], const double* const (&src)[NV], const int (&n)[NV],
                                             double* lds) {
  fold_parts<NV, MAXMASK>(v, src, n);
  block_reduce_lds<NV, MAXMASK, NTHR>(v, lds);
}

// Block-reduce NV values and let thread 0 store them as this block's
// partials: entry i goes to dst[i][block].  NTHR > 0: the block has NTHR
// threads, reduced through LDS.
template <int NV>
__device__ __forceinline__ void store_parts(const double (&v)[NV], double* const (&dst)[NV], int block) {
  const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
  if (tid == 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) dst[i][block] = v[i];
  }
}
template <int NV, unsigned MAXMASK, int NTHR = 0>
__device__ __forceinline__ void write_parts(double (&v)[NV], double* const (&dst)[NV], int block) {
  if constexpr (NTHR > 0) block_reduce_lds<NV, MAXMASK, NTHR>(v);
  else block_reduce<NV, MAXMASK>(v);
  store_parts(v, dst, block);
}
template <int NV, unsigned MAXMASK, int NTHR>
__device__ __forceinline__ void write_parts(double (&v)[NV], double* const (&dst)[NV], int block, double* lds) {
  block_reduce_lds<NV, MAXMASK, NTHR>(v, lds);
  store_parts(v, dst, block);
}

// Scalar recurrence of MINRES pass itn >= 1 (see k_minres), from ||R2||^2 and, with
// `lanczos`, the partials <R1, R2> and <Y, R2> of its product; ks is the state
// that pass itn - 1 left.  Every block runs it on the same reduced values in
// the same order; the lead thread stores the next state.
constexpr double kTinyNorm = 1e-30;  // a norm below this is zero (FP32 reciprocals stay finite)
struct MinresCoef {
  double s, c1, as;                        // y = s Y - c1 R1 - as R2
  double inv_oldb, wc1, wc2, inv_gamma;    // w = (R1 inv_oldb - wc1 W2 - wc2 W) inv_gamma
  double phi;                              // x += damp phi w
};
__device__ __forceinline__ MinresCoef minres_scalars(int itn, bool lanczos, double nrm2, double r12, double yr2,
                                                     const double (&ks)[7], double* next, bool lead) {
  MinresCoef q;
  const double beta = sqrt(fmax(nrm2, 0.0));
  double oldb = 0.0, alfa_prev = 0.0, dbar = 0.0, epsln = 0.0, phibar = beta, cs = -1.0, sn = 0.0;
  if (itn >= 2) {
    oldb = ks[0];
    alfa_prev = ks[1];
    dbar = ks[2];
    epsln = ks[3];
    phibar = ks[4];
    cs = ks[5];
    sn = ks[6];
  }
  // Givens rotation of iteration itn - 1
  double oldeps = 0.0, delta = 0.0, gamma = 1.0, phi = 0.0;
  if (itn >= 2) {
    oldeps = epsln;
    delta = cs * dbar + sn * alfa_prev;
    const double gbar = sn * dbar - cs * alfa_prev;
    epsln = sn * beta;
    dbar = -cs * beta;
    gamma = fmax(sqrt(gbar * gbar + beta * beta), 1e-300);
    cs = gbar / gamma;
    sn = beta / gamma;
    phi = cs * phibar;
    phibar = sn * phibar;
  }
  // Lanczos step of iteration itn.  Norms below kTinyNorm mean the Krylov
  // space is exhausted (the residual is zero to rounding): the reciprocals are
  // then taken as 0, so every further vector and update is 0 rather than 0 *
  // inf in FP32.
  const double s = beta > kTinyNorm ? 1.0 / beta : 0.0;
  const double c1 = (itn >= 2 && oldb > kTinyNorm) ? beta / oldb : 0.0;
  const double alfa = lanczos ? s * (s * yr2 - c1 * r12) : 0.0;
  if (lead) {
    next[0] = beta;
    next[1] = alfa;
    next[2] = dbar;
    next[3] = epsln;
    next[4] = phibar;
    next[5] = cs;
    next[6] = sn;
  }
  q.s = s;
  q.c1 = c1;
  q.as = alfa * s;
  q.inv_oldb = oldb > kTinyNorm ? 1.0 / oldb : 0.0;
  q.wc1 = oldeps;
  q.wc2 = delta;
  q.inv_gamma = gamma > kTinyNorm ? 1.0 / gamma : 0.0;
  q.phi = phi;
  return q;
}

// q = n / d for 0 <= n < 2^31 with rd = 1.0 / d: the FP64 product is within
// 2^-21 of n / d, so one correction step makes the quotient exact.
__device__ __forceinline__ int fdiv(int n, int d, double rd) {
  int q = (int)((double)n * rd);
  const int r = n - q * d;
  q += (r >= d) ? 1 : 0;
  q -= (r < 0) ? 1 : 0;
  return q;
}

// --------------------------------------------------------------------------
// SIMP scaling s = rho_min + (1 - rho_min) rho^p and ds/drho.
// --------------------------------------------------------------------------
// General exponents: FP64 goes through pow() in a separate function, so that
// the cubic case (the common SIMP exponent) keeps the hot loops free of its
// code; FP32 takes rho^e = 2^(e log2 rho) from the hardware's base-2
// exponential and logarithm (a few ulp, no call: a call inside the z-march
// makes the compiler keep its live scalar registers in vector lanes).
__device__ __noinline__ double simp_pow(double rho, double e) { return pow(rho, e); }

template <typename T>
__device__ __forceinline__ T simp_pow_t(T rho, double e) {
  if constexpr (sizeof(T) == 4) {
    if (!(rho > 0.0f)) return rho == 0.0f ? (e == 0.0 ? 1.0f : 0.0f) : __builtin_nanf("");
    return __builtin_amdgcn_exp2f((float)e * __builtin_amdgcn_logf(rho));
  } else {
    return simp_pow(rho, e);
  }
}

template <typename T>
__device__ __forceinline__ T simp_s(T rho, const Simp& sp) {
  const T rm = (T)sp.rho_min;
  T pw;
  if (sp.cubic) pw = rho * rho * rho;
  else pw = simp_pow_t<T>(rho, sp.penal);
  return rm + ((T)1 - rm) * pw;
}
template <typename T>
__device__ __forceinline__ T simp_ds(T rho, const Simp& sp) {
  const T rm = (T)sp.rho_min;
  T pw;
  if (sp.cubic) pw = rho * rho;
  else pw = simp_pow_t<T>(rho, sp.penal - 1.0);
  return (T)sp.penal * ((T)1 - rm) * pw;
}

// --------------------------------------------------------------------------
// Element product in the sum/difference basis (45 nonzeros instead of the
// dense 24 x 24): analysis butterflies, sparse modal KE.
// --------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void analysis8(T (&v)[8]) {
#pragma unroll
  for (int bit = 1; bit < 8; bit <<= 1) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i & bit) continue;
      const T lo = v[i], hi = v[i | bit];
      v[i] = lo + hi;
      v[i | bit] = hi - lo;
    }
  }
}
// z = KE_modal c  (component-major c[3][8], z[3][8]; mode 0 carries no energy).
// The modes fall into groups that couple only within themselves (see Modal):
// a common term and one product per member, 14 additions and 26 products (as
// 15 multiply-adds and 11 multiplications), where the matrix entry by entry
// takes 21 multiplications and 24 multiply-adds.
template <typename T>
__device__ __forceinline__ void modal_ke(const T (&c)[3][8], const Modal<T>& km, T (&z)[3][8]) {
  z[0][0] = z[1][0] = z[2][0] = (T)0;
  // normal strains, mode i of component i
  const T tn = km.l0 * ((c[0][1] + c[1][2]) + c[2][4]);
  // the modes of the other two axes
  const T tt = km.m1 * ((c[0][6] + c[1][5]) + c[2][3]);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    z[i][1 << i] = km.m8 * c[i][1 << i] + tn;
    z[i][7 ^ (1 << i)] = km.m1 * c[i][7 ^ (1 << i)] + tt;
    z[i][7] = km.d3 * c[i][7];
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int i = k == 0 ? 1 : 0, j = k == 2 ? 1 : 2;  // the other two axes
    // shear strain of axes i and j
    z[i][1 << j] = z[j][1 << i] = km.m0 * (c[i][1 << j] + c[j][1 << i]);
    // normal strains of i and j varying along k
    const int qi = (1 << i) | (1 << k), qj = (1 << j) | (1 << k);
    const T tk = km.l1 * (c[i][qi] + c[j][qj]);
    z[i][qi] = km.m0 * c[i][qi] + tk;
    z[j][qj] = km.m0 * c[j][qj] + tk;
  }
}

// le^T KE ue  (FP64 accumulation of the final dot)
template <typename T>
__device__ __forceinline__ double elem_bilinear(const T (&le)[8][3], const T (&ue)[8][3],
                                                const Modal<T>& km) {
  T cu[3][8], cl[3][8], z[3][8];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
#pragma unroll
    for (int a = 0; a < 8; ++a) { cu[i][a] = ue[a][i]; cl[i][a] = le[a][i]; }
    analysis8(cu[i]);
    analysis8(cl[i]);
  }
  modal_ke(cu, km, z);
  double acc = 0.0;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
#pragma unroll
    for (int q = 1; q < 8; ++q) acc += (double)cl[i][q] * (double)z[i][q];
  }
  return acc;
}

}  // namespace fbto
