// Plane (2D) variant of the hot path: the unit-square bilinear quadrilateral
// (Q4, plane stress) on a regular nx x ny grid -- the paper's own setting
// (Sec. 4.3 regular-grid discretisation, Sec. 5 experiments) -- and the
// separable Gaussian density filter of its experiments (Sec. 5, filter
// paragraph; Remark on modifiers, Sec. 3).
//
// Layout: node n = i + (nx + 1) j, DOF 2 n + c, element e = ex + nx ey,
// element-local node a = ax + 2 ay.  Multi-RHS vectors are [nrhs][2N].
//
// The plane grids of the paper (at most 192 x 576 elements, 0.9 MB per FP32
// vector) sit in the L2 and Infinity caches, so these kernels gather
// directly from global memory: one node (apply) or element (sensitivity)
// per thread, its 3 x 3 node neighbourhood read through L1/L2; the MINRES step
// (k_plane_minres) stages tiles in LDS.  The
// reductions use the per-block partial slots of the 3D path, with the same
// meaning, so the CG, MINRES, projection and finishing kernels serve both.
#include <hip/hip_runtime.h>

#include <cmath>

#include "device.h"
#include "internal.h"

namespace fbto {

namespace {
constexpr int kPlaneBlock = 256;

enum { PL_APPLY = 0, PL_RESID = 1, PL_CG = 2, PL_LZ = 3 };

template <typename T>
struct PlaneArgs {
  int nx, ny;
  int64_t N, ndof;
  const T* rho;
  const T* u;          // input vector
  T* y;                // output: K u, or r = f - K u (RESID: may be NULL)
  const T* f;          // RESID
  int parts;           // RESID: leave the partials of the residual
  const T* invD;       // CG: the preconditioner
  T* invD_out;         // RESID (optional): form the Jacobi diagonal and store its inverse, and z = D^-1 r
  T* z;                // RESID, with invD_out
  const uint8_t* mask; // bit c: DOF c of the node fixed
  Q4<T> ke;
  double ke_diag;
  Simp sp;
  double* P;
  int maxp;
  Scalars* sc;
  int step;            // CG, LZ: the partials go to the set of parity step & 1
};

__device__ __forceinline__ double* pslot2(double* P, int slot, int r, int maxp) {
  return P + ((int64_t)slot * 4 + r) * maxp;
}

// y = K u at node (i, j) for NR vectors, gathered from the four elements
// around the node; fixed DOFs of the neighbours enter as zero.
template <typename T, int NR, int MODE>
__global__ void __launch_bounds__(kPlaneBlock) k_plane_apply(PlaneArgs<T> A, int rhs0) {
  constexpr int NP = MODE == PL_APPLY ? 1 : MODE == PL_RESID ? 4 * NR : 2 * NR;
  double part[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) part[i] = 0.0;
  const int nxn = A.nx + 1;
  for (int64_t nn = (int64_t)blockIdx.x * kPlaneBlock + threadIdx.x; nn < A.N;
       nn += (int64_t)gridDim.x * kPlaneBlock) {
    const int n = (int)nn;
    const int j = n / nxn, i = n - j * nxn;
    // masked values of the 3 x 3 node neighbourhood, [dy][dx][c]
    T un[NR][3][3][2];
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        const int ii = i + dx - 1, jj = j + dy - 1;
        const bool ok = ii >= 0 && ii <= A.nx && jj >= 0 && jj <= A.ny;
        const int m = ok ? ii + nxn * jj : n;
        const unsigned mv = ok ? A.mask[m] : 3u;
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const T v = A.u[(int64_t)(rhs0 + r) * A.ndof + 2 * m + c];
            un[r][dy][dx][c] = ((mv >> c) & 1u) ? (T)0 : v;
          }
      }
    // the four elements: (i - ax, j - ay), node local index a = ax + 2 ay
    T acc[NR][2];
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[r][0] = acc[r][1] = (T)0;
    T ssum = (T)0;
#pragma unroll
    for (int ay = 0; ay < 2; ++ay)
#pragma unroll
      for (int ax = 0; ax < 2; ++ax) {
        const int ex = i - ax, ey = j - ay;
        const bool ok = ex >= 0 && ex < A.nx && ey >= 0 && ey < A.ny;
        const T rv = A.rho[ok ? ex + A.nx * ey : 0];
        const T s = ok ? simp_s<T>(rv, A.sp) : (T)0;
        ssum += s;
        const int a = ax + 2 * ay;
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            T t = (T)0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
              const int bx = b & 1, by = b >> 1;
              // element node b is neighbourhood node (bx - ax + 1, by - ay + 1)
#pragma unroll
              for (int d = 0; d < 2; ++d) t += A.ke.k[2 * a + c][2 * b + d] * un[r][by - ay + 1][bx - ax + 1][d];
            }
            acc[r][c] += s * t;
          }
      }
    const unsigned m = A.mask[n];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int64_t o = (int64_t)(rhs0 + r) * A.ndof + 2 * (int64_t)n;
      T pv[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        pv[c] = A.u[o + c];  // the own value, unmasked
        if ((m >> c) & 1u) acc[r][c] = pv[c];  // identity row of a fixed DOF
      }
      if constexpr (MODE == PL_APPLY) {
#pragma unroll
        for (int c = 0; c < 2; ++c) A.y[o + c] = acc[r][c];
      } else if constexpr (MODE == PL_RESID) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const T fv = A.f[o + c];
          const T rv = fv - acc[r][c];
          if (A.y) A.y[o + c] = rv;
          T zv = (T)0;
          if (A.invD_out) {
            T d = (T)A.ke_diag * ssum;
            if ((m >> c) & 1u) d = (T)1;
            const T dl = d > (T)0 ? (T)1 / d : (T)0;
            if (r == 0) A.invD_out[2 * (int64_t)n + c] = dl;
            zv = dl * rv;
            A.z[o + c] = zv;
          }
          part[4 * r + 0] += (double)rv * (double)rv;
          part[4 * r + 1] = fmax(part[4 * r + 1], fabs((double)rv));
          part[4 * r + 2] += (double)fv * (double)fv;
          part[4 * r + 3] += (double)rv * (double)zv;
        }
      } else {  // PL_CG: p.s, s.D^-1 s; PL_LZ: y.u, u.u
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          A.y[o + c] = acc[r][c];
          part[2 * r] += (double)acc[r][c] * (double)pv[c];
          if constexpr (MODE == PL_CG)
            part[2 * r + 1] += (double)acc[r][c] * (double)(A.invD[2 * (int64_t)n + c] * acc[r][c]);
          else
            part[2 * r + 1] += (double)pv[c] * (double)pv[c];
        }
      }
    }
  }
  if constexpr (MODE == PL_CG || MODE == PL_LZ) {
    const int par = A.step & 1;
    double* dst[2 * NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      dst[2 * r + 0] = pslot2(A.P, P_PQ0 + par, rhs0 + r, A.maxp);
      dst[2 * r + 1] = pslot2(A.P, (MODE == PL_CG ? P_EP0 : P_RZ0) + par, rhs0 + r, A.maxp);
    }
    write_parts<2 * NR, 0u>(part, dst, blockIdx.x);
    // LZ: u.u is the norm's square of iteration `step` - 1 too
    if constexpr (MODE == PL_LZ)
      if (threadIdx.x == 0) pslot2(A.P, P_KRN0 + (par ^ 1), 0, A.maxp)[blockIdx.x] = part[1];
  }
  if constexpr (MODE == PL_RESID) {
    if (!A.parts) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) {  // a new solve starts from this residual
      for (int r = 0; r < NR; ++r) {
        A.sc->done[rhs0 + r] = 0.0;
        A.sc->status[rhs0 + r] = 0.0;
        A.sc->steps[rhs0 + r] = 0.0;
      }
    }
    double* dst[4 * NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      dst[4 * r + 0] = pslot2(A.P, P_RNF, rhs0 + r, A.maxp);
      dst[4 * r + 1] = pslot2(A.P, P_RIF, rhs0 + r, A.maxp);
      dst[4 * r + 2] = pslot2(A.P, P_FN, rhs0 + r, A.maxp);
      dst[4 * r + 3] = pslot2(A.P, P_RZ0, rhs0 + r, A.maxp);  // r.z and r.r of step 0
    }
    write_parts<4 * NR, 0x2222u>(part, dst, blockIdx.x);
    if (threadIdx.x == 0) {
#pragma unroll
      for (int r = 0; r < NR; ++r) pslot2(A.P, P_RN0, rhs0 + r, A.maxp)[blockIdx.x] = part[4 * r];
    }
  }
}

// The fused MINRES step of the Krylov low-level step: the vector pass of
// iteration t (see k_minres) and iteration t + 1's product K y of its new
// Lanczos vector y.  A block owns a tile of 32 x 8 nodes, one per thread; y is
// formed at them and (by the first 84 threads) at the ring of halo nodes around
// them, and staged in LDS masked; s_e of the tile's 33 x 9 elements is staged
// beside it.  Y, R1 and R2 are read at halo nodes too, so y goes to a third
// buffer R3 and the product to the other Y buffer.  As two kernels (vector
// pass, product) the step was bound by two launches, each waiting for the
// partials of the one before: 8.0 + 8.2 us at 576 x 192 FP64.  The loads of a
// block's first tile are issued before its prologue reduces the partials.
constexpr int kPmX = 32, kPmY = 8, kPmRing = 2 * (kPmX + 2) + 2 * kPmY;
static_assert(kPmX * kPmY == kPlaneBlock, "one node per thread");
template <typename T>
struct Vec2 {
  T v[2];
};
template <typename T>
struct PlaneMinresArgs {
  int nx, ny, tiles_x, ntiles;
  const T* rho;
  const T *Y, *R1, *R2, *W;
  T *R3, *W2, *x, *Ynext;
  const uint8_t* mask;
  Q4<T> ke;
  Simp sp;
  double* P;
  int maxp;
  Scalars* sc;
  int itn, n_apply, n_kr;
  double damp;
};

template <typename T>
__global__ void __launch_bounds__(kPlaneBlock) k_plane_minres(PlaneMinresArgs<T> A) {
  using V2 = Vec2<T>;
  constexpr int LX = kPmX + 2, LY = kPmY + 2;   // staged nodes
  constexpr int SX = kPmX + 1, SY = kPmY + 1;   // staged elements
  __shared__ T ys[LX * LY][2];
  __shared__ T ss[SX * SY];
  const int tid = threadIdx.x, tx = tid % kPmX, ty = tid / kPmX;
  const int nxn = A.nx + 1, itn = A.itn;
  // LDS position of the thread's ring node, if it has one, and of its second element
  const bool has_ring = tid < kPmRing;
  int rx, ry;
  if (tid < 2 * LX) {
    rx = tid < LX ? tid : tid - LX;
    ry = tid < LX ? 0 : LY - 1;
  } else {
    const int t = tid - 2 * LX;
    rx = t < kPmY ? 0 : LX - 1;
    ry = 1 + (t < kPmY ? t : t - kPmY);
  }
  const bool has_el = tid < kPmX + SY;
  const int fx = tid < SY ? kPmX : tid - SY, fy = tid < SY ? tid : kPmY;

  struct Node {
    V2 y, r1, r2;
    unsigned m;
    bool ok;
  };
  Node own, ring;
  V2 wv{}, w2v{}, xv{};
  T re[2];
  bool oke[2];
  int n = 0;
  auto load_node = [&](int i, int j, bool want, Node& q) -> int {
    q.ok = want && i >= 0 && i <= A.nx && j >= 0 && j <= A.ny;
    const int k = q.ok ? i + nxn * j : 0;
    q.y = reinterpret_cast<const V2*>(A.Y)[k];
    q.r1 = reinterpret_cast<const V2*>(A.R1)[k];
    q.r2 = reinterpret_cast<const V2*>(A.R2)[k];
    q.m = A.mask[k];
    return k;
  };
  auto load_elem = [&](int ex, int ey, bool want, T& r, bool& ok) {
    ok = want && ex >= 0 && ex < A.nx && ey >= 0 && ey < A.ny;
    r = A.rho[ok ? ex + A.nx * ey : 0];
  };
  auto load_tile = [&](int t) {
    const int x0 = (t % A.tiles_x) * kPmX, y0 = (t / A.tiles_x) * kPmY;
    n = load_node(x0 + tx, y0 + ty, true, own);
    load_node(x0 - 1 + rx, y0 - 1 + ry, has_ring, ring);
    load_elem(x0 - 1 + tx, y0 - 1 + ty, true, re[0], oke[0]);
    load_elem(x0 - 1 + fx, y0 - 1 + fy, has_el, re[1], oke[1]);
    wv = reinterpret_cast<const V2*>(A.W)[n];
    w2v = reinterpret_cast<const V2*>(A.W2)[n];
    xv = reinterpret_cast<const V2*>(A.x)[n];
  };
  load_tile(blockIdx.x);

  double ks[7], pv[3];
#pragma unroll
  for (int i = 0; i < 7; ++i) ks[i] = A.sc->kr[(itn + 1) & 1][i];
  {
    const double* src[3] = {pslot2(A.P, P_KRN0 + ((itn + 1) & 1), 0, A.maxp), pslot2(A.P, P_RZ0 + (itn & 1), 0, A.maxp),
                            pslot2(A.P, P_PQ0 + (itn & 1), 0, A.maxp)};
    const int cnt[3] = {A.n_kr, A.n_apply, A.n_apply};
    reduce_parts<3, 0u>(pv, src, cnt);
  }
  const MinresCoef q =
      minres_scalars(itn, true, pv[0], pv[1], pv[2], ks, A.sc->kr[itn & 1], blockIdx.x == 0 && tid == 0);
  const T s = (T)q.s, c1 = (T)q.c1, as = (T)q.as, inv_oldb = (T)q.inv_oldb;
  const T wc1 = (T)q.wc1, wc2 = (T)q.wc2, inv_gamma = (T)q.inv_gamma, step = (T)(A.damp * q.phi);

  double part[3] = {0.0, 0.0, 0.0};  // ||y||^2, <K y, y>, <R2, y>
  for (int t = blockIdx.x; t < A.ntiles; t += gridDim.x) {
    if (t != (int)blockIdx.x) {
      __syncthreads();  // the last tile's product has read the LDS
      load_tile(t);
    }
    T yo[2];  // the own node's y
    auto stage = [&](const Node& q, int li, T (&yn)[2]) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const T r1m = itn >= 2 ? q.r1.v[c] : (T)0;  // R1 holds no vector yet on the first iteration
        yn[c] = s * q.y.v[c] - c1 * r1m - as * q.r2.v[c];
        ys[li][c] = q.ok && !((q.m >> c) & 1u) ? yn[c] : (T)0;
      }
    };
    stage(own, tx + 1 + LX * (ty + 1), yo);
    if (has_ring) {
      T yr[2];
      stage(ring, rx + LX * ry, yr);
    }
    ss[tx + SX * ty] = oke[0] ? simp_s<T>(re[0], A.sp) : (T)0;
    if (has_el) ss[fx + SX * fy] = oke[1] ? simp_s<T>(re[1], A.sp) : (T)0;
    if (own.ok) {
      V2 wn, xn, yn;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const T wm = itn >= 3 ? wv.v[c] : (T)0, w2m = itn >= 4 ? w2v.v[c] : (T)0;  // zero before the first
        wn.v[c] = (own.r1.v[c] * inv_oldb - wc1 * w2m - wc2 * wm) * inv_gamma;
        xn.v[c] = xv.v[c] + step * wn.v[c];
        yn.v[c] = yo[c];
        part[0] += (double)yo[c] * (double)yo[c];
        part[2] += (double)own.r2.v[c] * (double)yo[c];
      }
      reinterpret_cast<V2*>(A.R3)[n] = yn;
      if (itn >= 2) {  // finishes iteration t - 1
        reinterpret_cast<V2*>(A.W2)[n] = wn;
        reinterpret_cast<V2*>(A.x)[n] = xn;
      }
    }
    __syncthreads();
    // K y at the own node from the four elements around it, in k_plane_apply's order
    T acc[2] = {(T)0, (T)0};
#pragma unroll
    for (int ay = 0; ay < 2; ++ay)
#pragma unroll
      for (int ax = 0; ax < 2; ++ax) {
        const T se = ss[tx + 1 - ax + SX * (ty + 1 - ay)];
        const int a = ax + 2 * ay;
        T tc[2] = {(T)0, (T)0};
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int bx = b & 1, by = b >> 1;
          const int li = tx + 1 + bx - ax + LX * (ty + 1 + by - ay);
#pragma unroll
          for (int d = 0; d < 2; ++d) {
            const T v = ys[li][d];
#pragma unroll
            for (int c = 0; c < 2; ++c) tc[c] += A.ke.k[2 * a + c][2 * b + d] * v;
          }
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[c] += se * tc[c];
      }
    if (own.ok) {
      V2 o;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        if ((own.m >> c) & 1u) acc[c] = yo[c];  // identity row of a fixed DOF
        o.v[c] = acc[c];
        part[1] += (double)acc[c] * (double)yo[c];
      }
      reinterpret_cast<V2*>(A.Ynext)[n] = o;
    }
  }
  double* dst[3] = {pslot2(A.P, P_KRN0 + (itn & 1), 0, A.maxp), pslot2(A.P, P_PQ0 + ((itn + 1) & 1), 0, A.maxp),
                    pslot2(A.P, P_RZ0 + ((itn + 1) & 1), 0, A.maxp)};
  write_parts<3, 0u>(part, dst, blockIdx.x);
}

// Jacobi diagonal: ke_diag * (sum of s over the node's elements), 1 at fixed DOFs.
template <typename T>
__global__ void __launch_bounds__(kPlaneBlock)
    k_plane_diag(int nx, int ny, int64_t N, const T* rho, T* invD, const uint8_t* mask, Simp sp, double ke_diag) {
  const int nxn = nx + 1;
  for (int64_t nn = (int64_t)blockIdx.x * kPlaneBlock + threadIdx.x; nn < N; nn += (int64_t)gridDim.x * kPlaneBlock) {
    const int n = (int)nn;
    const int j = n / nxn, i = n - j * nxn;
    T acc = (T)0;
#pragma unroll
    for (int dy = -1; dy <= 0; ++dy)
#pragma unroll
      for (int dx = -1; dx <= 0; ++dx) {
        const int ex = i + dx, ey = j + dy;
        const bool ok = ex >= 0 && ex < nx && ey >= 0 && ey < ny;
        const T rv = rho[ok ? ex + nx * ey : 0];
        acc += ok ? simp_s<T>(rv, sp) : (T)0;
      }
    const unsigned m = mask[n];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      T d = (T)ke_diag * acc;
      if ((m >> c) & 1u) d = (T)1;
      invD[2 * nn + c] = d > (T)0 ? (T)1 / d : (T)0;
    }
  }
}

// dobj_e = -ds_e sum_r lam_{r,e}^T KE u_{r,e} (times Hsi_e when given).
template <typename T>
__global__ void __launch_bounds__(kPlaneBlock)
    k_plane_sens(int nx, int ny, int64_t ndof, const T* rho, const T* u, const T* lam, int nrhs, T* dobj,
                 const uint8_t* mask, Q4<T> ke, Simp sp, const T* Hsi) {
  const int64_t E = (int64_t)nx * ny;
  const int nxn = nx + 1;
  for (int64_t ee = (int64_t)blockIdx.x * kPlaneBlock + threadIdx.x; ee < E; ee += (int64_t)gridDim.x * kPlaneBlock) {
    const int e = (int)ee;
    const int ey = e / nx, ex = e - ey * nx;
    double acc = 0.0;
    for (int R = 0; R < nrhs; ++R) {
      T ue[8], le[8];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int n = (ex + (a & 1)) + nxn * (ey + (a >> 1));
        const unsigned m = mask[n];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const T uv = u[R * ndof + 2 * n + c];
          const T lv = lam ? lam[R * ndof + 2 * n + c] : uv;
          ue[2 * a + c] = ((m >> c) & 1u) ? (T)0 : uv;
          le[2 * a + c] = ((m >> c) & 1u) ? (T)0 : lv;
        }
      }
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        T t = (T)0;
#pragma unroll
        for (int q = 0; q < 8; ++q) t += ke.k[p][q] * ue[q];
        acc += (double)le[p] * (double)t;
      }
    }
    double val = -(double)simp_ds<T>(rho[e], sp) * acc;
    if (Hsi) val *= (double)Hsi[e];
    dobj[e] = (T)val;
  }
}

// One output of a 1D pass of the separable Gaussian, at position pos of len:
//   sum_{|d| <= H, pos + d inside} g(d) x[d * stride]  (/ h if normalise),
// h the sum of g(d) over the offsets inside the grid; x is 0 outside it.  The
// taps are unrolled (weights read one by one cost a scalar load's latency each).
template <typename T, int H>
__device__ __forceinline__ T gauss_at(const T* x, int stride, int pos, int len, int normalise, const GaussW<T>& gw) {
  T acc = (T)0, h = (T)0;
#pragma unroll
  for (int d = -H; d <= H; ++d) {
    const T w = gw.w[d + H];
    acc += w * x[d * stride];
    h += pos + d >= 0 && pos + d < len ? w : (T)0;
  }
  return normalise ? acc / h : acc;
}

// Both passes (along `axis` first; 0: x, 1: y) on 32 x 8 tiles of outputs: the
// tile's values, times `pre` (1/Hs of the transpose) if given, are staged in LDS
// with H more on each side, and the first pass leaves its outputs there, halo
// rows or columns too.  want_sum: per-block partial sums of out into slot GSUM.
// Bound by launch and latency on the grids in use, so one launch instead of one
// per pass: an FP64 iteration at 576x192 284.9 -> 280.1 us (281.3 with the taps
// in a loop).
constexpr int kGaussTX = 32, kGaussTY = kPlaneBlock / kGaussTX;
template <typename T, int H>
__global__ void __launch_bounds__(kPlaneBlock)
    k_plane_gauss(int nx, int ny, int axis, const T* in, T* out, const T* pre, int normalise, GaussW<T> gw,
                   int want_sum, double* P, int maxp, int tiles_x, int ntiles) {
  constexpr int LX = kGaussTX + 2 * H, LY = kGaussTY + 2 * H;
  __shared__ T sa[LX * LY], sb[LX * LY];
  // the first pass's outputs: MX x MY of them from column and row ox, oy of the stage
  const int MX = axis == 0 ? kGaussTX : LX, MY = axis == 0 ? LY : kGaussTY;
  const int ox = axis == 0 ? H : 0, oy = axis == 0 ? 0 : H;
  const int tx = threadIdx.x % kGaussTX, ty = threadIdx.x / kGaussTX;
  static_assert(2 * H <= kGaussTX && 2 * H <= 2 * kGaussTY, "turns of the stage");
  double v[1] = {0.0};
  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int tj = t / tiles_x, x0 = (t - tj * tiles_x) * kGaussTX, y0 = tj * kGaussTY;
    // two rows of threads' turns at most along x, three along y
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int lx = tx + i * kGaussTX, ly = ty + j * kGaussTY, ex = x0 - H + lx, ey = y0 - H + ly;
        if (lx >= LX || ly >= LY) continue;
        T x = (T)0;
        if (ex >= 0 && ex < nx && ey >= 0 && ey < ny) {
          const int e = ey * nx + ex;
          x = pre ? in[e] * pre[e] : in[e];
        }
        sa[ly * LX + lx] = x;
      }
    __syncthreads();
    for (int my = ty; my < MY; my += kGaussTY)
      for (int mx = tx; mx < MX; mx += kGaussTX) {
        const int lx = ox + mx, ly = oy + my, ex = x0 - H + lx, ey = y0 - H + ly;
        T o = (T)0;
        if (ex >= 0 && ex < nx && ey >= 0 && ey < ny)
          o = gauss_at<T, H>(sa + ly * LX + lx, axis == 0 ? 1 : LX, axis == 0 ? ex : ey, axis == 0 ? nx : ny,
                             normalise, gw);
        sb[my * MX + mx] = o;
      }
    __syncthreads();
    const int ex = x0 + tx, ey = y0 + ty;
    if (ex < nx && ey < ny) {
      const T* x = sb + (axis == 0 ? (ty + H) * MX + tx : ty * MX + tx + H);
      const T o = gauss_at<T, H>(x, axis == 0 ? MX : 1, axis == 0 ? ey : ex, axis == 0 ? ny : nx, normalise, gw);
      out[ey * nx + ex] = o;
      v[0] += (double)o;
    }
  }
  if (want_sum) {
    double* dst[1] = {pslot2(P, P_GSUM, 0, maxp)};
    write_parts<1, 0u>(v, dst, blockIdx.x);
  }
}

// 1 / Hs_e = 1 / (h_x(ex) h_y(ey)): the 2D row sum of a separable window
// truncated at the grid's edges factors over the axes.
template <typename T>
__global__ void __launch_bounds__(kPlaneBlock) k_plane_hs(int nx, int ny, T* Hsi, GaussW<T> gw) {
  const int64_t E = (int64_t)nx * ny;
  for (int64_t ee = (int64_t)blockIdx.x * kPlaneBlock + threadIdx.x; ee < E; ee += (int64_t)gridDim.x * kPlaneBlock) {
    const int e = (int)ee;
    const int ey = e / nx, ex = e - ey * nx;
    double hx = 0.0, hy = 0.0;
    for (int d = -gw.half; d <= gw.half; ++d) {
      if (ex + d >= 0 && ex + d < nx) hx += (double)gw.w[d + gw.half];
      if (ey + d >= 0 && ey + d < ny) hy += (double)gw.w[d + gw.half];
    }
    Hsi[e] = (T)(1.0 / (hx * hy));
  }
}

int plane_blocks(int64_t n) {
  int64_t b = (n + kPlaneBlock - 1) / kPlaneBlock;
  if (b > kMaxVecBlocks) b = kMaxVecBlocks;
  if (b < 1) b = 1;
  return (int)b;
}

template <typename T> const Q4<T>& q4_of(fbto_grid_s* g);
template <> const Q4<double>& q4_of<double>(fbto_grid_s* g) { return g->q4_64; }
template <> const Q4<float>& q4_of<float>(fbto_grid_s* g) { return g->q4_32; }
template <typename T> GaussW<T> gauss_of(fbto_grid_s* g);
template <> GaussW<double> gauss_of<double>(fbto_grid_s* g) { return g->gauss64; }
template <> GaussW<float> gauss_of<float>(fbto_grid_s* g) { return g->gauss32; }

template <typename T>
PlaneArgs<T> plane_args(fbto_grid_s* g) {
  PlaneArgs<T> A{};
  A.nx = g->geo.nx;
  A.ny = g->geo.ny;
  A.N = g->geo.N;
  A.ndof = g->geo.ndof;
  A.mask = g->mask;
  A.ke = q4_of<T>(g);
  A.ke_diag = g->ke_diag;
  A.sp = g->simp;
  A.P = g->partials;
  A.maxp = g->max_partials;
  A.sc = g->sc;
  return A;
}

template <typename T, int MODE>
hipError_t plane_launch(fbto_grid_s* g, const PlaneArgs<T>& A, int nrhs, hipStream_t st, int* nb_out) {
  const int nb = plane_blocks(g->geo.N);
  if (nb > g->max_partials) return hipErrorInvalidValue;
  for (int r0 = 0; r0 < nrhs;) {
    const int left = nrhs - r0;
    if (left >= 2 && MODE != PL_APPLY) {
      hipLaunchKernelGGL((k_plane_apply<T, 2, MODE>), dim3(nb), dim3(kPlaneBlock), 0, st, A, r0);
      r0 += 2;
    } else {
      hipLaunchKernelGGL((k_plane_apply<T, 1, MODE>), dim3(nb), dim3(kPlaneBlock), 0, st, A, r0);
      r0 += 1;
    }
  }
  if (nb_out) *nb_out = nb;
  return hipGetLastError();
}
}  // namespace

template <typename T>
hipError_t plane_apply(fbto_grid_s* g, const T* rho, const T* u, T* y, int nrhs, hipStream_t st) {
  PlaneArgs<T> A = plane_args<T>(g);
  A.rho = rho;
  A.u = u;
  A.y = y;
  return plane_launch<T, PL_APPLY>(g, A, nrhs, st, nullptr);
}

template <typename T>
hipError_t plane_resid(fbto_grid_s* g, const T* rho, const T* u, const T* f, T* r, T* invD_out, T* z, int parts,
                       int nrhs, hipStream_t st, int* nb_out) {
  PlaneArgs<T> A = plane_args<T>(g);
  A.rho = rho;
  A.u = u;
  A.y = r;
  A.f = f;
  A.parts = parts;
  A.invD_out = invD_out;
  A.z = z;
  return plane_launch<T, PL_RESID>(g, A, nrhs, st, nb_out);
}

template <typename T>
hipError_t plane_apply_cg(fbto_grid_s* g, const T* rho, const T* p, const T* invD, T* s, int nrhs, int step,
                          hipStream_t st, int* nb_out) {
  PlaneArgs<T> A = plane_args<T>(g);
  A.rho = rho;
  A.u = p;
  A.invD = invD;
  A.y = s;
  A.step = step;
  return plane_launch<T, PL_CG>(g, A, nrhs, st, nb_out);
}

template <typename T>
hipError_t plane_apply_lanczos(fbto_grid_s* g, const T* rho, const T* u, T* y, int step, hipStream_t st, int* nb_out) {
  PlaneArgs<T> A = plane_args<T>(g);
  A.rho = rho;
  A.u = u;
  A.y = y;
  A.step = step;
  return plane_launch<T, PL_LZ>(g, A, 1, st, nb_out);
}

template <typename T>
hipError_t plane_minres_fused(fbto_grid_s* g, const T* rho, int itn, const T* Y, const T* R1, const T* R2, T* R3,
                              const T* W, T* W2, T* x, T* Ynext, int n_apply, int n_kr, double damp, hipStream_t st,
                              int* nb_out) {
  PlaneMinresArgs<T> A{};
  A.nx = g->geo.nx;
  A.ny = g->geo.ny;
  A.tiles_x = (g->geo.nxn + kPmX - 1) / kPmX;
  const int64_t ntiles = (int64_t)A.tiles_x * ((g->geo.ny + kPmY) / kPmY);  // ny + 1 rows of nodes
  if (ntiles > INT32_MAX || n_apply > g->max_partials || n_kr > g->max_partials) return hipErrorInvalidValue;
  A.ntiles = (int)ntiles;
  A.rho = rho;
  A.Y = Y; A.R1 = R1; A.R2 = R2; A.W = W;
  A.R3 = R3; A.W2 = W2; A.x = x; A.Ynext = Ynext;
  A.mask = g->mask;
  A.ke = q4_of<T>(g);
  A.sp = g->simp;
  A.P = g->partials;
  A.maxp = g->max_partials;
  A.sc = g->sc;
  A.itn = itn;
  A.n_apply = n_apply;
  A.n_kr = n_kr;
  A.damp = damp;
  const int nb = (int)(ntiles < g->max_partials ? ntiles : g->max_partials);
  if (nb_out) *nb_out = nb;
  hipLaunchKernelGGL((k_plane_minres<T>), dim3(nb), dim3(kPlaneBlock), 0, st, A);
  return hipGetLastError();
}

template <typename T>
hipError_t plane_diag(fbto_grid_s* g, const T* rho, T* invD, hipStream_t st) {
  hipLaunchKernelGGL((k_plane_diag<T>), dim3(plane_blocks(g->geo.N)), dim3(kPlaneBlock), 0, st, g->geo.nx,
                     g->geo.ny, g->geo.N, rho, invD, g->mask, g->simp, g->ke_diag);
  return hipGetLastError();
}

template <typename T>
hipError_t plane_sens(fbto_grid_s* g, const T* rho, const T* u, const T* lam, int nrhs, T* dobj, const T* Hsi,
                      hipStream_t st) {
  hipLaunchKernelGGL((k_plane_sens<T>), dim3(plane_blocks(g->geo.E)), dim3(kPlaneBlock), 0, st, g->geo.nx,
                     g->geo.ny, g->geo.ndof, rho, u, lam, nrhs, dobj, g->mask, q4_of<T>(g), g->simp, Hsi);
  return hipGetLastError();
}

template <typename T, int H>
void launch_gauss(int half, int grid, hipStream_t st, int nx, int ny, int kind, const T* in, T* out, const T* Hsi,
                  const GaussW<T>& gw, int want_sum, fbto_grid_s* g, int tiles_x, int ntiles) {
  if constexpr (H < kGaussMaxHalf) {
    if (half > H)
      return launch_gauss<T, H + 1>(half, grid, st, nx, ny, kind, in, out, Hsi, gw, want_sum, g, tiles_x, ntiles);
  }
  hipLaunchKernelGGL((k_plane_gauss<T, H>), dim3(grid), dim3(kPlaneBlock), 0, st, nx, ny, kind == 0 ? 0 : 1, in, out,
                     kind == 1 ? Hsi : (const T*)nullptr, kind == 0 ? 1 : 0, gw, want_sum, g->partials,
                     g->max_partials, tiles_x, ntiles);
}

// kind 0: out = (H in) / Hs (x pass, then y pass, each normalised);
// kind 1: out = H^T (in / Hs);  kind 2: out = H^T in (input already / Hs).
// in and out do not overlap.
template <typename T>
hipError_t plane_filter(fbto_grid_s* g, int kind, const T* in, T* out, const T* Hsi, int want_sum, hipStream_t st) {
  const int nx = g->geo.nx, ny = g->geo.ny;
  const int tiles_x = (nx + kGaussTX - 1) / kGaussTX;
  const int64_t ntiles = (int64_t)tiles_x * ((ny + kGaussTY - 1) / kGaussTY);
  const int grid = (int)std::min<int64_t>(ntiles, kMaxVecBlocks);
  if (want_sum) g->n_gsum = grid;
  launch_gauss<T, 0>(g->gauss64.half, grid, st, nx, ny, kind, in, out, Hsi, gauss_of<T>(g), want_sum, g, tiles_x,
                     (int)ntiles);
  return hipGetLastError();
}

template <typename T>
hipError_t plane_hs(fbto_grid_s* g, T* Hsi, hipStream_t st) {
  hipLaunchKernelGGL((k_plane_hs<T>), dim3(plane_blocks(g->geo.E)), dim3(kPlaneBlock), 0, st, g->geo.nx, g->geo.ny,
                     Hsi, gauss_of<T>(g));
  return hipGetLastError();
}

#define FBTO_PLANE_INST(T)                                                                                   \
  template hipError_t plane_apply<T>(fbto_grid_s*, const T*, const T*, T*, int, hipStream_t);                \
  template hipError_t plane_resid<T>(fbto_grid_s*, const T*, const T*, const T*, T*, T*, T*, int, int,       \
                                     hipStream_t, int*);                                                     \
  template hipError_t plane_apply_cg<T>(fbto_grid_s*, const T*, const T*, const T*, T*, int, int, hipStream_t, \
                                        int*);                                                               \
  template hipError_t plane_apply_lanczos<T>(fbto_grid_s*, const T*, const T*, T*, int, hipStream_t, int*);   \
  template hipError_t plane_minres_fused<T>(fbto_grid_s*, const T*, int, const T*, const T*, const T*, T*,   \
                                            const T*, T*, T*, T*, int, int, double, hipStream_t, int*);      \
  template hipError_t plane_diag<T>(fbto_grid_s*, const T*, T*, hipStream_t);                                \
  template hipError_t plane_sens<T>(fbto_grid_s*, const T*, const T*, const T*, int, T*, const T*,           \
                                    hipStream_t);                                                            \
  template hipError_t plane_filter<T>(fbto_grid_s*, int, const T*, T*, const T*, int, hipStream_t);          \
  template hipError_t plane_hs<T>(fbto_grid_s*, T*, hipStream_t);

FBTO_PLANE_INST(double)
FBTO_PLANE_INST(float)

}  // namespace fbto
