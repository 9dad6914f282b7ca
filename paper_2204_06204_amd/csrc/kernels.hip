// HIP kernels of the matrix-free SIMP hot path for gfx950 (MI355X).
//
// K(rho) u = sum_e s_e P_e^T KE P_e u on a structured hex8 grid
// (Sec. 3 and the regular-grid product of Sec. 4.3), the Jacobi-PCG low-level
// refinement (Alg. 1 / 3 low-level line with a Jacobi preconditioner,
// Sec. 4.1), the sensitivity of Sec. 3, the linear density filter (Remark on
// modifiers, Sec. 3) and the projection onto the volume-constrained box
// (Sec. 4.2, Eq. piecewiseLinearEQ).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstdio>
#include <type_traits>

#include "device.h"
#include "internal.h"

namespace fbto {

namespace {

constexpr int kVecBlock = 256;


template <typename T> const Modal<T>& modal_of(fbto_grid_s* g);
template <> const Modal<double>& modal_of<double>(fbto_grid_s* g) { return g->km64; }
template <> const Modal<float>& modal_of<float>(fbto_grid_s* g) { return g->km32; }
template <typename T> const T* spring_k_of(fbto_grid_s* g);
template <> const double* spring_k_of<double>(fbto_grid_s* g) { return g->spring_k64; }
template <> const float* spring_k_of<float>(fbto_grid_s* g) { return g->spring_k32; }
template <typename T> const T* stencil_w_of(fbto_grid_s* g);
template <> const double* stencil_w_of<double>(fbto_grid_s* g) { return g->stencil_w64; }
template <> const float* stencil_w_of<float>(fbto_grid_s* g) { return g->stencil_w32; }
template <typename T> Vecs& vecs_of(fbto_grid_s* g);
template <> Vecs& vecs_of<double>(fbto_grid_s* g) { return g->v64; }
template <> Vecs& vecs_of<float>(fbto_grid_s* g) { return g->v32; }

}  // namespace

// Grid of the vector kernels: at least 4 entries per thread, at most
// kMaxVecBlocks blocks (the number of partials a consumer reduces).
int vec_blocks(int64_t n) {
  int64_t b = (n + 4 * kVecBlock - 1) / (4 * kVecBlock);
  if (b > kMaxVecBlocks) b = kMaxVecBlocks;
  if (b < 1) b = 1;
  return (int)b;
}

__device__ __forceinline__ const double* pslot(const double* P, int slot, int r, int maxp) {
  return P + ((int64_t)slot * 4 + r) * maxp;
}
__device__ __forceinline__ double* pslot(double* P, int slot, int r, int maxp) {
  return P + ((int64_t)slot * 4 + r) * maxp;
}

// Grid for element / node kernels without partials: one entry per thread.
static int flat_grid(int64_t n) {
  return (int)std::max<int64_t>(1, std::min<int64_t>((n + kVecBlock - 1) / kVecBlock, 1 << 20));
}

// ===========================================================================
// apply_K: z-marching tiles in the sum/difference basis.
//
// A block owns a BX x BY tile of element columns (a runtime shape fitted to
// the grid) and a slab of node planes.  Thread (tx, ty) owns element column
// (ex, ey) = (x0 + tx, y0 + ty), x0 = bx (BX - 1) - 1, y0 = by (BY - 1) - 1,
// and writes node (ex, ey) of every plane of the slab when tx, ty >= 1:
// column and row 0 are the halo shared with the neighbouring tiles.
//
// Per element layer ez:
//   - every node of plane ez + 2 is read from HBM once per tile (the own
//     node, plus the far column and row of the tile by the first BX + BY + 1
//     threads), masked and staged in LDS one layer ahead of its use;
//   - the thread turns the upper face of its element into face modes
//     (x, then y butterflies); the lower face's modes are the upper face's
//     of the layer below, kept in registers;
//   - z butterflies give 8 modes x 3 components; the modal KE (45 entries)
//     times s_e; inverse z butterflies split the result into a lower-face
//     and an upper-face part.  The upper part is carried to the next layer in
//     modal form and added to that layer's lower part before the inverse x/y
//     butterflies, so each face is transformed once in each direction;
//   - the four corner values of plane ez are summed over the four element
//     columns around each node through LDS, in a fixed order.
// Node and corner buffers are double-buffered: one barrier per layer.
// Tiles overlap by one element column / row and slabs by one element layer,
// so there are no atomics and the result is bitwise reproducible.
//
// Modes:
//   APPLY  y = K u
//   RESID  r = f - K u (to y, if given), with the partials of r.r, max|r|,
//          f.f on request; the start of a CG solve also forms the Jacobi
//          diagonal, stores its inverse (one value per node) and z = D^-1 r,
//          with the partials of r.z
//   CG     y = s = K p with the partials of p.s and s.D^-1 s (the product of
//          the first CG step)
//   LZ     y = K u with the partials of u.u and y.u (the first product of the
//          Krylov update)
//   CGF    one fused CG step: the vector update of step k is done where each
//          node is staged (r' = r - alpha s, p' = D^-1 r' + beta p,
//          x' = x + alpha p), the owner of the node stores x', r', p' into the
//          output set, and the product is s' = K p' (step k + 1's) with its
//          partials.  Input and output sets are distinct buffers: halo nodes
//          of a tile are read by its neighbours while their owner writes the
//          update.  On large grids the iterate is updated every second step,
//          by two directions at once (XU).
//   MRF    the fused MINRES step of the Krylov low-level step (one RHS):
//          the vector pass of iteration t (see k_minres) done where each
//          node is staged, and iteration t + 1's product K y of the new
//          Lanczos vector y in the same pass.  Y, R1, R2 are read at halo
//          nodes too, so y goes to a third buffer R3 and the product to the
//          other Y buffer.  On large grids every second pass leaves the
//          direction and the iterate to the next one, which forms two
//          directions (XU): the Lanczos vector it lacks is still in the buffer
//          that R3 goes to, and two passes read W, W2, x and that vector and
//          write W, W2 and x, where a direction per pass takes ten accesses.
//          FP32 256x128x128 118 -> 105 us per Krylov degree, 128x64x64 21.5 ->
//          20.3 us; FP64 233 -> 208 and 31.7 -> 29.5 us.
// ===========================================================================
enum { MODE_APPLY = 0, MODE_RESID = 1, MODE_CG = 2, MODE_CGF = 3, MODE_SENSF = 4, MODE_MRF = 5, MODE_LZ = 6 };
static_assert(MODE_LZ < kApplyModes, "a tile choice per mode");
constexpr int kApplyMaxThreads = 512;
constexpr int kApplyMaxBlocks = 8192;
constexpr int kMaxP = kApplyMaxBlocks;  // partials per slot of a voxel grid

// Bits 3 R + 1 for R < nr: the |r|_inf entries (max-reduced) of the
// per-RHS triples (sum of squares, |r|_inf, another sum) that the residual
// and finishing reductions lay out.
constexpr unsigned rinf_mask(int nr) {
  unsigned m = 0u;
  for (int R = 0; R < nr; ++R) m |= 1u << (3 * R + 1);
  return m;
}

template <typename T>
struct ApplyArgs {
  Geo g;
  const T* rho;
  const T* u;          // input vector
  T* y;
  const T* f;          // RESID
  int parts;           // RESID: leave the partials of the residual
  T* z;                // RESID (optional): z = D^-1 r, with the Jacobi diagonal formed here
  // The inverse Jacobi diagonal (RESID stores it, CG and CGF read it).  Every
  // diagonal entry of KE is the same number, so without springs a node has one
  // value for its DOFs but the fixed ones, whose 1 is seen from the mask (DN =
  // 1); with springs a value per DOF is kept (DN = 3).
  T* dinv_out;         // RESID (optional, with z)
  int dn_out;          // RESID: 1 or 3 values per node
  double ke_diag;      // diagonal entry of KE (with z)
  const T* dinv;
  const uint8_t* mask; // bits 0-2: fixed DOFs of the node; bit 3: the node has a spring
  Modal<T> km;
  Simp sp;
  int nspring;
  const int64_t* sdof;
  const T* sk;
  int bx, by;          // tile of bx * by element columns (threads = (bx + 1) * (by + 1), one per node column)
  int tiles_x, tiles_y, slabs, dz, nblocks, per_xcd;
  uint32_t inv_tx, inv_ty;  // floor(2^32 / tiles) + 1 (0: one tile), for div_small
  float inv_tw;             // 1 / threads per tile row
  double* P;           // partial slots, of kMaxP values per RHS
  const Scalars* sc;
  int step;            // CG, CGF: step k; CG writes, CGF reads the partial set of parity k & 1
  // CGF and SENSF
  const T *xi, *ri, *pi, *si;        // step k's x, r, p, s
  T *xo, *ro, *po;                   // step k + 1's x, r, p (s goes to y)
  int n_gam, n_apply, n_fn;          // partial counts of step k's r.z, of its product, and of f.f
  double rtol;
  // SENSF only (last CG step fused with the sensitivity)
  T* dobj;                           // [E] -ds_e x_e^T KE x_e (times Hsi_e)
  const T* Hsi;                      // [E] 1/Hs_e, or NULL
  const T* fvec;                     // loads, for f . x (NULL: not formed)
  // MRF only (fused MINRES step; `step` is the iteration t, A.y the product)
  const T *mY, *mR1, *mR2, *mW;      // K R2 of iteration t, Lanczos vectors t - 1 and t, direction t - 2
  T *mR3, *mW2, *mx;                 // new Lanczos vector; direction t - 3 in, t - 1 out; iterate
  T* mWo;                            // XU 2: mW, written (direction t - 1; mW2 gets t - 2)
  int n_kr;                          // partial count of ||R2||^2
  double damp;                       // step size of the low-level step
};

// n / d by the multiplicative inverse inv = floor(2^32 / d) + 1 (0 for d = 1):
// exact while n d < 2^32 (block numbers and tile counts, at most 2^13 each).
// A kernel's first loads wait for its address arithmetic, 2 of the 9 us of a
// small grid's step.  With these instead of integer divisions and constant slot
// strides an FP32 CG step went from 11.1 to 10.5 us at 64x32x32 and from 19.1
// to 18.5 us at 128x64x64, K u there from 11.6 to 11.0 us.
__device__ __forceinline__ uint32_t div_small(uint32_t n, uint32_t inv) { return inv ? __umulhi(n, inv) : n; }
static uint32_t inv_small(int d) { return d == 1 ? 0u : (uint32_t)(((uint64_t)1 << 32) / (uint64_t)d + 1); }
static_assert((int64_t)kApplyMaxBlocks * kApplyMaxBlocks < ((int64_t)1 << 32), "div_small is exact");

// Step coefficients of the CG recurrence for one RHS from gamma = r.z,
// delta = p.s, eps = s.D^-1 s (s = K p), r.r and f.f of step k (identical in
// every block):
//   alpha = gamma / delta,   beta = (alpha^2 eps - gamma) / gamma.
// The numerator of beta is r'.D^-1 r' of r' = r - alpha s expanded with
// r.D^-1 s = z.s = p.s (conjugate directions), so one reduction phase serves
// a step; gamma itself is always summed from r and z, so its rounding is not
// carried from step to step.  A numerator that rounds below zero (r' is zero
// to rounding) restarts from z'.  A solved, converged or broken-down RHS gets
// alpha = beta = 0.  The lead thread records the flags and the step count.
__device__ __forceinline__ void cg_coefficients(double gam, double del, double eps, double rr, double ff, int R,
                                                int par, double rtol, Scalars* sc, bool lead, double& alpha,
                                                double& beta) {
  const double rn = sqrt(rr), fn = sqrt(ff);
  bool done = sc->done[R] != 0.0 || (rtol > 0.0 && rn <= rtol * fn);
  double status = 0.0;
  alpha = 0.0;
  beta = 0.0;
  if (!done) {
    if (gam == 0.0 && isfinite(del)) {
      done = true;
    } else if (del > 0.0 && isfinite(del) && isfinite(gam) && isfinite(eps)) {
      alpha = gam / del;
      beta = fmax((alpha * alpha * eps - gam) / gam, 0.0);
    } else {
      status = isfinite(del) && isfinite(gam) && isfinite(eps) ? (double)FBTO_ERR_BREAKDOWN
                                                                : (double)FBTO_ERR_NONFINITE;
      done = true;
    }
  }
  if (lead) {
    if (done) sc->done[R] = 1.0;
    if (status != 0.0) sc->status[R] = status;
    if (alpha != 0.0) sc->steps[R] += 1.0;
    sc->alpha[par][R] = alpha;
  }
}

// Face modes of one face: u[a][c] at local node a = ax + 2 ay -> F[q][c],
// bit 0 / 1 of q set for the difference mode along x / y.
template <typename T>
__device__ __forceinline__ void face_modes(const T (&u)[4][3], T (&F)[4][3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const T s0 = u[0][c] + u[1][c], d0 = u[1][c] - u[0][c];
    const T s1 = u[2][c] + u[3][c], d1 = u[3][c] - u[2][c];
    F[0][c] = s0 + s1;
    F[1][c] = d0 + d1;
    F[2][c] = s1 - s0;
    F[3][c] = d1 - d0;
  }
}
// Transpose of face_modes.
template <typename T>
__device__ __forceinline__ void face_values(const T (&F)[4][3], T (&u)[4][3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const T v0 = F[0][c] - F[1][c], v1 = F[0][c] + F[1][c];
    const T v2 = F[2][c] - F[3][c], v3 = F[2][c] + F[3][c];
    u[0][c] = v0 - v2;
    u[2][c] = v0 + v2;
    u[1][c] = v1 - v3;
    u[3][c] = v1 + v3;
  }
}

// One element (one RHS): face modes of its lower and upper face, scale s.
// `carry` holds the modal upper-face result of the element below on entry
// and this element's on exit; `out` receives the values at the 4 nodes of
// the lower face (both elements' contributions).
template <typename T>
__device__ __forceinline__ void layer_product(const T (&Flo)[4][3], const T (&Fup)[4][3], T s,
                                              const Modal<T>& km, T (&carry)[4][3],
                                              T (&out)[4][3]) {
  T c[3][8], z[3][8];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    c[i][0] = (T)0;  // the all-sum mode (translation) carries no energy
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q) c[i][q] = Flo[q][i] + Fup[q][i];
      c[i][q + 4] = Fup[q][i] - Flo[q][i];
    }
  }
  modal_ke(c, km, z);
  // scaled by s here, where half of the products join an addition
  T lo[4][3];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const T zl = q ? z[i][q] - z[i][q + 4] : -z[i][4], zu = q ? z[i][q] + z[i][q + 4] : z[i][4];
      lo[q][i] = s * zl + carry[q][i];
      carry[q][i] = s * zu;
    }
  face_values(lo, out);
}

template <typename T>
struct ApplyStage {
  T v[2][3];
  unsigned m[2];
};

// Loads of one node plane for the fused CG step (one RHS).
template <typename T, int DN>
struct FusedStage {
  T x[3], q[3];                 // owned node only: x, step k - 1's p
  T r[3], s[3], p[3], d[DN];
  unsigned m;
};

// Loads of one node plane for the fused MINRES step.
template <typename T>
struct MinresStage {
  T w[3], w2[3], x[3], v[3];    // owned node only; v: Lanczos vector t - 2
  T y[3], r1[3], r2[3];
  unsigned m;
};

// Buffer access of the z-march kernels.  A resource spans 2^31 - 1 bytes
// from its base; kOOR, and kOOR plus the 8 and 16 bytes of an FP64 triple's
// later values, lie beyond it, so an access there loads 0 or is dropped
// without a cache request.
constexpr uint32_t kOOR = 0x80000000u;
// Thread layout of a z-march variant.  Node layout: one thread per node
// column of the tile ((bx + 1) (by + 1) threads), each staging one node per
// plane; the fused steps take it (fewer memory instructions per node; their
// staging does the CG or MINRES vector update too).  Element layout: one
// thread per element column (bx by threads), the tile's far column and row
// staged by a second slot of threads 0 .. bx + by; the plain product, the
// residual and the step-0 product take it (fewer threads for the same
// elements, measured faster for them).
template <int MODE>
constexpr bool node_layout() { return MODE == MODE_CGF || MODE == MODE_MRF || MODE == MODE_SENSF; }
// threads of a z-march block for a tile of bx x by element columns
template <int MODE>
constexpr int zmarch_threads(int bx, int by) {
  return ((node_layout<MODE>() ? (bx + 1) * (by + 1) : bx * by) + 63) / 64 * 64;
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t zrsrc(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, 0x7FFFFFFF, 0x00020000);
}
typedef float zf3 __attribute__((ext_vector_type(3)));
typedef unsigned zu3 __attribute__((ext_vector_type(3)));
typedef unsigned zu2 __attribute__((ext_vector_type(2)));
typedef unsigned zu4 __attribute__((ext_vector_type(4)));
typedef double zd2 __attribute__((ext_vector_type(2)));
// voff: the lane's byte offset (a node or element column, or kOOR); soff: the
// plane's, the same for the block, added by the load itself.  Stores add it in
// a vector register: with a scalar offset the compiler takes a store of three
// or four words to be safe from the next instruction's write to its data
// registers, and single nodes of the FP32 residual were then stored wrong now
// and then.
template <typename T>
__device__ __forceinline__ void zload3(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff, T (&v)[3]) {
  if constexpr (sizeof(T) == 4) {
    const zf3 t = __builtin_bit_cast(zf3, __builtin_amdgcn_raw_buffer_load_b96(rs, voff, soff, 0));
    v[0] = t.x;
    v[1] = t.y;
    v[2] = t.z;
  } else {
    const zd2 t = __builtin_bit_cast(zd2, __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 0));
    v[0] = t.x;
    v[1] = t.y;
    v[2] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rs, voff + 16u, soff, 0));
  }
}
template <typename T>
__device__ __forceinline__ void zstore3(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff, const T (&v)[3]) {
  if constexpr (sizeof(T) == 4) {
    zu3 t;
    t.x = __builtin_bit_cast(unsigned, v[0]);
    t.y = __builtin_bit_cast(unsigned, v[1]);
    t.z = __builtin_bit_cast(unsigned, v[2]);
    __builtin_amdgcn_raw_buffer_store_b96(t, rs, voff + soff, 0, 0);
  } else {
    const zd2 t = {v[0], v[1]};
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(zu4, t), rs, voff + soff, 0, 0);
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(zu2, v[2]), rs, voff + soff + 16u, 0, 0);
  }
}
template <typename T>
__device__ __forceinline__ T zload1(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff) {
  if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, 0));
  else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, 0));
}
template <typename T>
__device__ __forceinline__ void zstore1(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff, T v) {
  if constexpr (sizeof(T) == 4)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, voff + soff, 0, 0);
  else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(zu2, v), rs, voff + soff, 0, 0);
}
// v, or 0 where bit c of the mask byte m is set, by bit operations (two per
// 32 bits; a compare and a select take three).
template <typename T>
__device__ __forceinline__ T zmasked(unsigned m, int c, T v) {
  const int keep = __builtin_amdgcn_sbfe((int)~m, c, 1);  // all ones where the bit is clear
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_bit_cast(int, v) & keep);
  } else {
    return __hiloint2double(__double2hiint(v) & keep, __double2loint(v) & keep);
  }
}

// Wave priority around the plane loads of a z-march layer (FP32 only): the
// loads then go out ahead of the element products of the other waves on the
// SIMD.  Measured: FP32 fused steps 1.5-2.5% and the FP32 apply up to 2%
// faster; the FP64 fused CG step at 256x128x128 ran 14% slower with it, so
// FP64 keeps the default priority.
template <typename T>
__device__ __forceinline__ void loads_priority(bool raise) {
  if constexpr (sizeof(T) == 4) {
    if (raise) __builtin_amdgcn_s_setprio(2);
    else __builtin_amdgcn_s_setprio(0);
  }
}

// A value that is the same in every lane of the wave, kept in a scalar
// register (FP32; FP64 values stay in vector registers).
template <typename T>
__device__ __forceinline__ T wave_uniform(T v) {
  if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
  else return v;
}

// Waves per SIMD the register allocation of a z-march variant must allow:
// three for the FP32 fused steps (at most 168 VGPRs; they take 114 to 135),
// which run many blocks per CU on large grids; the others are left to the
// compiler.
template <typename T, int MODE>
constexpr int apply_min_waves() {
  return (sizeof(T) == 4 && (MODE == MODE_CGF || MODE == MODE_MRF)) ? 3 : 1;
}

// RR (fused CG step): form r.r for the tolerance test; solves of a fixed
// step count (rtol = 0) read no r.r and run the variant without it.
// DN (CG, CGF): values of the inverse diagonal per node.
// XU (fused CG and MINRES steps): updates of the iterate.  1: x += alpha_k p_k;
// 0: none, it is left to the next step; 2: x += alpha_{k-1} p_{k-1} + alpha_k
// p_k, with p_{k-1} read from the buffer that p_{k+1} goes to, before it is
// stored.  The operations and their order are the same; two steps read x and
// p_{k-1} and write x once instead of reading and writing x twice, half a vector
// less per step.
template <typename T, int MODE, bool RR = true, int DN = 1, int XU = 1>
__global__ void __launch_bounds__(kApplyMaxThreads) __attribute__((amdgpu_waves_per_eu(apply_min_waves<T, MODE>())))
    k_apply(ApplyArgs<T> A) {
  extern __shared__ __align__(16) unsigned char apply_smem[];
  const int b = blockIdx.x;
  const int lb = (b & 7) * A.per_xcd + (b >> 3);  // XCD-aware: neighbours share an L2
  if (lb >= A.nblocks) return;                    // whole block
  const int rhs0 = blockIdx.y;                    // the load case
  double* const parts = A.P + rhs0 * kMaxP;       // its partials
  const Geo G = A.g;
  const int BX = A.bx, BY = A.by;
  constexpr bool NL = node_layout<MODE>();
  constexpr int kSlots = NL ? 1 : 2;  // node columns a thread stages per plane
  const int NW = BX + 1;          // LDS node row
  const int NS = NW * (BY + 1);   // LDS nodes per plane
  const int TW = NL ? NW : BX;    // threads per tile row
  const int TS = NL ? NS : BX * BY;  // threads with a node (node layout) or an element (element layout)
  // a node's three values and a thread's nine corner values lie together:
  // odd strides of 3 and 9 values (no bank conflicts), few wide LDS
  // instructions, and immediate offsets instead of an address each
  T* nodes = reinterpret_cast<T*>(apply_smem);   // [2][NS][3]
  T* corners = nodes + 2 * 3 * NS;              // [2][TS][9]
  T* dcorn = corners + 2 * 9 * TS;              // [2][TS] density sums of the diagonal

  // Thread (tx, ty) of the tile computes element column (x0 + tx, y0 + ty)
  // for tx < BX, ty < BY and stages node (x0 + tx, y0 + ty).  In the node
  // layout the threads of the tile's far column and row (tx = BX or
  // ty = BY) stage those nodes and run the element code on neighbouring LDS
  // values; nothing reads what they produce.  In the element layout
  // threads 0 .. BX + BY stage them in a second slot.  The block is padded
  // to whole waves (the DPP reductions read every lane of a wave); padding
  // threads mirror thread 0 and store nothing.
  const int tid = threadIdx.x;
  const bool live = tid < TS;
  const int tl = live ? tid : 0;
  const int ty = (int)((tl + 0.5f) * A.inv_tw), tx = tl - ty * TW;  // exact: tl < 512
  const int t2 = (int)div_small(lb, A.inv_tx);
  const int bxi = lb - t2 * A.tiles_x;
  const int bz = (int)div_small(t2, A.inv_ty);
  const int byi = t2 - bz * A.tiles_y;
  const int x0 = bxi * (BX - 1) - 1, y0 = byi * (BY - 1) - 1;
  const int ex = x0 + tx, ey = y0 + ty;
  const int k0 = bz * A.dz;
  const int kend = min(k0 + A.dz, G.nz + 1);  // emitted planes [k0, kend)
  const int ez0 = k0 == 0 ? 0 : k0 - 1;        // first element layer (a halo layer if k0 > 0)
  const int plane = G.nxn * G.nyn;
  const bool elem_t = live && tx < BX && ty < BY;  // a thread with an element column
  const bool col_elem = elem_t && ex >= 0 && ex < G.nx && ey >= 0 && ey < G.ny;
  // nodes whose four element columns are all in the tile: their outputs
  const bool writer = live && tx >= 1 && ty >= 1 && tx < BX && ty < BY && ex <= G.nx && ey <= G.ny;

  // Node columns staged by this thread: slot 0 its own (ex, ey); in the
  // element layout slot 1 one node of the tile's far column / row (threads
  // 0 .. BX + BY).  Padding threads stage thread 0's node again (the same
  // value into the same LDS slot).
  // Every memory operation of the z-march is issued unconditionally (loads
  // and stores a thread does not need go out of range, see below).  With no
  // branch around them the compiler can
  // count the loads in flight and wait only for the ones it consumes, so
  // the planes prefetched for the next layers stay in flight.
  const bool has_extra = !NL && tid <= BX + BY;
  int li[2], gcol[2];
  li[0] = tx + NW * ty;
  gcol[0] = (ex >= 0 && ex <= G.nx && ey >= 0 && ey <= G.ny) ? ex + G.nxn * ey : -1;
  {
    const int lx = tid <= BY ? BX : tid - BY - 1;
    const int ly = tid <= BY ? tid : BY;
    const int i1 = x0 + lx, j1 = y0 + ly;
    li[1] = has_extra ? lx + NW * ly : li[0];  // the own node again: the same value, same thread
    gcol[1] = has_extra ? ((i1 >= 0 && i1 <= G.nx && j1 >= 0 && j1 <= G.ny) ? i1 + G.nxn * j1 : -1) : gcol[0];
  }

  // Memory access of the z-march.  Every array is addressed through a buffer
  // resource based at the block's first plane ez0, with 32-bit byte offsets
  // relative to it (the host keeps 3 b plane (dz + 3) < 2^31, b the value
  // size).  A lane whose node is not needed -- the far-node slot of a thread
  // without a far node, planes past the slab, values only the owner of a
  // node uses, outputs of a thread that owns none -- passes an out-of-range
  // offset: its load returns 0 and its store is dropped, without a cache
  // request, while every memory instruction is still issued unconditionally.
  const int64_t pbase = (int64_t)ez0 * plane;               // first node of plane ez0
  const int64_t vbase = (int64_t)rhs0 * G.ndof + 3 * pbase;  // its first value in RHS rhs0
  auto rsrc = [](const void* p) { return zrsrc(p); };
  auto vres = [&](const T* v) { return rsrc(v ? v + vbase : v); };  // [nrhs][3N]
  auto dres = [&](const T* v, int dn) { return rsrc(v ? v + dn * pbase : v); };  // [N][dn]
  // An access takes the byte offset of the lane's node column in its plane
  // (computed once; kOOR where the lane has none) and the plane's byte offset
  // in a scalar register: no vector arithmetic per access.
  // The small grids are bound by the instructions they issue: with this, the
  // node and corner layouts above and one select per partial an FP32 layer of
  // K u went from 270 to 237 vector instructions and one of the fused step from
  // 310 to 267, in 129 registers instead of 156 (215, 250 to 257 and 114 to 121
  // now, with the element product by strain groups).  K u at 256x128x128 51.5 ->
  // 49.0 us; FP32 outer iteration 208 -> 199 us at 128x64x64 and 120 -> 116 us at
  // 64x32x32; FP64 336 -> 325 us.
  const uint32_t vc1 = gcol[0] >= 0 ? (uint32_t)gcol[0] : kOOR;  // mask bytes
  const uint32_t vc3 = gcol[0] >= 0 ? (uint32_t)(3 * sizeof(T)) * (uint32_t)gcol[0] : kOOR;
  const uint32_t vx1 = has_extra && gcol[1] >= 0 ? (uint32_t)gcol[1] : kOOR;  // the far node
  const uint32_t vx3 = has_extra && gcol[1] >= 0 ? (uint32_t)(3 * sizeof(T)) * (uint32_t)gcol[1] : kOOR;
  const uint32_t vw3 = writer ? vc3 : kOOR;  // the node a thread owns
  const uint32_t vd = gcol[0] >= 0 ? (uint32_t)sizeof(T) * (uint32_t)gcol[0] : kOOR;  // values per node
  const uint32_t vwd = writer ? vd : kOOR;
  auto splane = [&](int k) -> uint32_t { return (uint32_t)(k - ez0) * (uint32_t)plane; };
  auto sd = [&](int k) -> uint32_t { return (uint32_t)sizeof(T) * splane(k); };
  auto s3 = [&](int k) -> uint32_t { return (uint32_t)(3 * sizeof(T)) * splane(k); };
  const __amdgpu_buffer_rsrc_t rs_m = rsrc(A.mask + pbase);
  auto bload3 = [](__amdgpu_buffer_rsrc_t rs, uint32_t vo, uint32_t so, T (&v)[3]) { zload3<T>(rs, vo, so, v); };
  auto bstore3 = [](__amdgpu_buffer_rsrc_t rs, uint32_t vo, uint32_t so, const T (&v)[3]) { zstore3<T>(rs, vo, so, v); };
  // the mask byte of a node (0 out of range, where the values load as 0 too)
  auto bmask = [&](uint32_t vo, uint32_t so) -> unsigned {
    return __builtin_amdgcn_raw_buffer_load_b8(rs_m, vo, so, 0);
  };

  // Planes past the slab's last one (kend) are staged but never read; their
  // loads are out of range.
  const __amdgpu_buffer_rsrc_t rs_u = vres(A.u);
  auto issue = [&](int k, ApplyStage<T>& S) {
    const bool kv = k >= 0 && k <= kend && k <= G.nz;  // planes the block reads
    const uint32_t so1 = kv ? splane(k) : 0u, so3 = (uint32_t)(3 * sizeof(T)) * so1;
#pragma unroll
    for (int sl = 0; sl < kSlots; ++sl) {
      const uint32_t o1 = kv ? (sl ? vx1 : vc1) : kOOR, o3 = kv ? (sl ? vx3 : vc3) : kOOR;
      S.m[sl] = bmask(o1, so1);
      bload3(rs_u, o3, so3, S.v[sl]);
    }
  };
  auto stage = [&](const ApplyStage<T>& S, int buf) {
    T* nb = nodes + buf * (3 * NS);
#pragma unroll
    for (int sl = 0; sl < kSlots; ++sl) {
      if (sl == 1 && !has_extra) continue;  // no far node: nothing staged
#pragma unroll
      for (int c = 0; c < 3; ++c) nb[3 * li[sl] + c] = zmasked(S.m[sl], c, S.v[sl][c]);
    }
  };
  // the lower-left node of the thread's element (node 0's for threads
  // without an element, whose face values nothing reads: their reads stay
  // inside the plane)
  const int lf = 3 * (elem_t ? li[0] : 0);
  auto read_face = [&](int buf, T (&F)[4][3]) {
    const T* nb = nodes + buf * (3 * NS) + lf;
    T u4[4][3];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int c = 0; c < 3; ++c) u4[a][c] = nb[3 * (a >> 1) * NW + 3 * (a & 1) + c];
    face_modes(u4, F);
  };
  // The density of the next layer is loaded raw and turned into s_e only
  // when it is used: consuming a load right after it was issued would make
  // the wave wait for every load issued before it (the counter is in order),
  // including the node planes prefetched for the next layers.
  const __amdgpu_buffer_rsrc_t rs_rho = rsrc(A.rho + (int64_t)G.nx * G.ny * ez0);
  const uint32_t ve = col_elem ? (uint32_t)sizeof(T) * (uint32_t)(ex + G.nx * ey) : kOOR;
  auto load_rho = [&](int ez) -> T {
    const bool el = ez >= 0 && ez < G.nz && ez < kend;  // element layers of this block
    const uint32_t so = el ? (uint32_t)sizeof(T) * (uint32_t)((ez - ez0) * (G.nx * G.ny)) : 0u;
    return zload1<T>(rs_rho, el ? ve : kOOR, so);
  };
  auto scale_of = [&](int ez, T rv) -> T {
    const bool el = col_elem && ez >= 0 && ez < G.nz;
    return el ? simp_s<T>(rv, A.sp) : (T)0;
  };

  constexpr int NP = MODE == MODE_APPLY ? 1 : 4;  // partial values per block
  double part[NP];
  // The thread's own sums of non-negative terms (r.r, r.z = sum r^2 / d,
  // f.f) and max|r| over its owned nodes, at most 3 (dz + 1) terms per RHS,
  // accumulate in T and join the FP64 partials before the block reduction;
  // sums with terms of either sign (p.s) stay FP64 throughout.
  //   RESID: r.r, max|r|, f.f, r.z   CGF: r.z, r.r   CG, CGF: s.D^-1 s (2)
  T tpart[4] = {(T)0, (T)0, (T)0, (T)0};
#pragma unroll
  for (int i = 0; i < NP; ++i) part[i] = 0.0;

  // fused CG step: coefficients of step k from its partials (every block;
  // called in the prologue, after the first planes' loads are issued, so
  // the two latencies overlap)
  T al = (T)0, be = (T)0, alq = (T)0;  // alq: step k - 1's alpha, if its update is pending
  auto cg_prologue = [&]() {
    const int par = A.step & 1;
    constexpr int NV = RR ? 5 : 3;
    double pre[NV];
    const double* src[NV];
    int cnt[NV];
    src[0] = pslot(parts, P_RZ0 + par, 0, kMaxP);
    src[1] = pslot(parts, P_PQ0 + par, 0, kMaxP);
    src[2] = pslot(parts, P_EP0 + par, 0, kMaxP);
    cnt[0] = A.n_gam;
    cnt[1] = cnt[2] = A.n_apply;
    if constexpr (RR) {
      src[3] = pslot(parts, P_RN0 + par, 0, kMaxP);
      src[4] = pslot(parts, P_FN, 0, kMaxP);
      cnt[3] = A.n_gam;
      cnt[4] = A.n_fn;
    }
    // step k - 1's alpha: the lead thread stores step k's beside it, by parity
    double aq = 0.0;
    if constexpr (XU == 2) aq = A.sc->alpha[par ^ 1][rhs0];
    reduce_parts<NV, 0u>(pre, src, cnt);
    double rr = 0.0, ff = 0.0;
    if constexpr (RR) {
      rr = pre[3];
      ff = pre[4];
    }
    double alpha, beta;
    cg_coefficients(pre[0], pre[1], pre[2], rr, ff, rhs0, par, RR ? A.rtol : 0.0, const_cast<Scalars*>(A.sc),
                    lb == 0 && tid == 0, alpha, beta);
    // the same value in every lane: kept in scalar registers
    al = wave_uniform((T)alpha);
    be = wave_uniform((T)beta);
    if constexpr (XU == 2) alq = wave_uniform((T)aq);
  };
  // fused CG step: loads of one plane, and the update at staging time.
  const __amdgpu_buffer_rsrc_t rs_r = vres(A.ri), rs_s = vres(A.si), rs_x = vres(A.xi), rs_p = vres(A.pi),
                               rs_d = dres(A.dinv, DN);
  // loads of the node's inverse diagonal (voffset: per node or per DOF), and
  // its value at each DOF.  One value per node where the fused step read
  // three is 8 (FP64: 16) of 108 (212) bytes per node.
  auto load_d = [&](uint32_t o1, uint32_t so1, uint32_t o3, uint32_t so3, T (&d)[DN]) {
    if constexpr (DN == 3) bload3(rs_d, o3, so3, d);
    else d[0] = zload1<T>(rs_d, o1, (uint32_t)sizeof(T) * so1);
  };
  auto dof_d = [](const T (&d)[DN], unsigned m, int c) -> T {
    if constexpr (DN == 3) return d[c];
    else return ((m >> c) & 1u) ? (T)1 : d[0];
  };
  const __amdgpu_buffer_rsrc_t rs_xo = vres(A.xo), rs_ro = vres(A.ro), rs_po = vres(A.po);
  auto issue_f = [&](int k, FusedStage<T, DN>& S) {
    const bool kv = k >= 0 && k <= kend && k <= G.nz;  // planes the block reads
    const bool own_plane = k >= k0 && k < kend;
    const uint32_t so1 = kv ? splane(k) : 0u, so3 = (uint32_t)(3 * sizeof(T)) * so1;
    const uint32_t o3 = kv ? vc3 : kOOR;
    S.m = bmask(kv ? vc1 : kOOR, so1);
    bload3(rs_r, o3, so3, S.r);
    bload3(rs_s, o3, so3, S.s);
    load_d(kv ? vd : kOOR, so1, o3, so3, S.d);
    bload3(rs_p, o3, so3, S.p);
    const uint32_t oo = kv && own_plane ? vw3 : kOOR;  // used by the owner only
    if constexpr (XU >= 1) bload3(rs_x, oo, so3, S.x);
    if constexpr (XU == 2) bload3(rs_po, oo, so3, S.q);
  };
  // zq: the node's p' (unmasked: the output of a fixed DOF); dq: its D^-1
  auto stage_f = [&](const FusedStage<T, DN>& S, int buf, int k, T (&zq)[3], T (&dq)[DN]) {
    T* nb = nodes + buf * (3 * NS) + 3 * li[0];
    const bool own_plane = k >= k0 && k < kend;
    // the owner's byte offset; other threads store out of range (dropped)
    const uint32_t o3 = own_plane ? vw3 : kOOR, so3 = own_plane ? s3(k) : 0u;
    T xn[3], rn[3], pn[3], rz = (T)0, rr = (T)0;
#pragma unroll
    for (int c = 0; c < DN; ++c) dq[c] = S.d[c];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      rn[c] = S.r[c] - al * S.s[c];
      const T zn = dof_d(S.d, S.m, c) * rn[c];
      pn[c] = zn + be * S.p[c];
      nb[c] = zmasked(S.m, c, pn[c]);
      zq[c] = pn[c];
      if constexpr (XU == 1) xn[c] = S.x[c] + al * S.p[c];
      if constexpr (XU == 2) xn[c] = (S.x[c] + alq * S.q[c]) + al * S.p[c];
      rz += rn[c] * zn;
      if constexpr (RR) rr += rn[c] * rn[c];
    }
    const bool owner = writer && own_plane;
    tpart[0] += owner ? rz : (T)0;                    // r.z
    if constexpr (RR) tpart[1] += owner ? rr : (T)0;  // r.r
    if constexpr (XU >= 1) bstore3(rs_xo, o3, so3, xn);
    bstore3(rs_ro, o3, so3, rn);
    bstore3(rs_po, o3, so3, pn);
  };

  // fused MINRES step: the scalar recurrence of iteration t (every block,
  // same order; block 0 keeps the state), as in k_minres
  T ms = (T)0, mc1 = (T)0, mas = (T)0, minvb = (T)0, mwc1 = (T)0, mwc2 = (T)0, minvg = (T)0, mstep = (T)0;
  T pinvb = (T)0, pwc1 = (T)0, pwc2 = (T)0, pinvg = (T)0, pstep = (T)0;  // XU 2: of iteration t - 2
  auto uniform = [](T v) -> T { return wave_uniform(v); };
  auto mrf_prologue = [&]() {
    const int itn = A.step;
    double v[3];
    const double* src[3] = {pslot(parts, P_KRN0 + ((itn - 1) & 1), 0, kMaxP), pslot(parts, P_RZ0 + (itn & 1), 0, kMaxP),
                            pslot(parts, P_PQ0 + (itn & 1), 0, kMaxP)};
    const int cnt[3] = {A.n_kr, A.n_apply, A.n_apply};
    reduce_parts<3, 0u>(v, src, cnt);
    Scalars* sc = const_cast<Scalars*>(A.sc);
    double ks[7];
#pragma unroll
    for (int i = 0; i < 7; ++i) ks[i] = sc->kr[(itn + 1) & 1][i];
    const MinresCoef q = minres_scalars(itn, true, v[0], v[1], v[2], ks, sc->kr[itn & 1], lb == 0 && tid == 0);
    ms = uniform((T)q.s);
    mc1 = uniform((T)q.c1);
    mas = uniform((T)q.as);
    minvb = uniform((T)q.inv_oldb);
    mwc1 = uniform((T)q.wc1);
    mwc2 = uniform((T)q.wc2);
    minvg = uniform((T)q.inv_gamma);
    mstep = uniform((T)(A.damp * q.phi));
    if constexpr (XU == 0) {  // left to the next pass
      if (lb == 0 && tid == 0) {
        sc->kr_pend[0] = q.inv_oldb;
        sc->kr_pend[1] = q.wc1;
        sc->kr_pend[2] = q.wc2;
        sc->kr_pend[3] = q.inv_gamma;
        sc->kr_pend[4] = q.phi;
      }
    }
    if constexpr (XU == 2) {
      pinvb = uniform((T)sc->kr_pend[0]);
      pwc1 = uniform((T)sc->kr_pend[1]);
      pwc2 = uniform((T)sc->kr_pend[2]);
      pinvg = uniform((T)sc->kr_pend[3]);
      pstep = uniform((T)(A.damp * sc->kr_pend[4]));
    }
  };
  // fused MINRES step (single vectors, rhs0 = 0): the memory access of the fused CG step
  const __amdgpu_buffer_rsrc_t rs_mY = vres(A.mY), rs_mR1 = vres(A.mR1), rs_mR2 = vres(A.mR2), rs_mW = vres(A.mW),
                               rs_mW2 = vres(A.mW2), rs_mx = vres(A.mx), rs_mR3 = vres(A.mR3), rs_mWo = vres(A.mWo);
  auto issue_m = [&](int k, MinresStage<T>& S) {
    const bool kv = k >= 0 && k <= kend && k <= G.nz;  // planes the block reads
    const bool own_plane = k >= k0 && k < kend;
    const uint32_t so1 = kv ? splane(k) : 0u, so3 = (uint32_t)(3 * sizeof(T)) * so1;
    const uint32_t o3 = kv ? vc3 : kOOR, oo = kv && own_plane ? vw3 : kOOR;
    S.m = bmask(kv ? vc1 : kOOR, so1);
    bload3(rs_mY, o3, so3, S.y);
    bload3(rs_mR1, o3, so3, S.r1);
    bload3(rs_mR2, o3, so3, S.r2);
    if constexpr (XU >= 1) {  // the iterate and the directions: owner only
      bload3(rs_mW, oo, so3, S.w);
      bload3(rs_mW2, oo, so3, S.w2);
      bload3(rs_mx, oo, so3, S.x);
    }
    if constexpr (XU == 2) bload3(rs_mR3, oo, so3, S.v);
  };
  auto stage_m = [&](const MinresStage<T>& S, int buf, int k, T (&zq)[3]) {
    T* nb = nodes + buf * (3 * NS) + 3 * li[0];
    const bool own_plane = k >= k0 && k < kend;
    const int itn = A.step;
    T yn[3], wn[3], wp[3], xn[3];
    double yy = 0.0, ry = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const T r1m = itn >= 2 ? S.r1[c] : (T)0;  // R1 holds no vector yet on the first iteration
      yn[c] = ms * S.y[c] - mc1 * r1m - mas * S.r2[c];
      nb[c] = zmasked(S.m, c, yn[c]);
      zq[c] = yn[c];  // unmasked: the output of a fixed DOF
      if constexpr (XU == 1) {
        const T wm = itn >= 3 ? S.w[c] : (T)0, w2m = itn >= 4 ? S.w2[c] : (T)0;
        wn[c] = (S.r1[c] * minvb - mwc1 * w2m - mwc2 * wm) * minvg;
        xn[c] = S.x[c] + mstep * wn[c];
      }
      if constexpr (XU == 2) {  // iterations t - 2 (wp), then t - 1
        const T wm = itn >= 4 ? S.w[c] : (T)0, w2m = itn >= 5 ? S.w2[c] : (T)0;
        wp[c] = (S.v[c] * pinvb - pwc1 * w2m - pwc2 * wm) * pinvg;
        wn[c] = (S.r1[c] * minvb - mwc1 * wm - mwc2 * wp[c]) * minvg;
        xn[c] = (S.x[c] + pstep * wp[c]) + mstep * wn[c];
      }
      yy += (double)yn[c] * (double)yn[c];
      ry += (double)S.r2[c] * (double)yn[c];
    }
    const bool owner = writer && own_plane;
    if constexpr (NP >= 3) {
      part[0] += owner ? yy : 0.0;  // ||y||^2
      part[2] += owner ? ry : 0.0;  // <R2, y>: R1.R2 of iteration t + 1
    }
    const uint32_t oo = own_plane ? vw3 : kOOR, so3 = own_plane ? s3(k) : 0u;
    bstore3(rs_mR3, oo, so3, yn);
    if (XU >= 1 && itn >= 2) {  // finishes iteration t - 1 (uniform)
      bstore3(rs_mW2, oo, so3, XU == 2 ? wp : wn);
      if constexpr (XU == 2) bstore3(rs_mWo, oo, so3, wn);
      bstore3(rs_mx, oo, so3, xn);
    }
  };

  // The element stiffness constants.  The FP32 fused steps keep them in
  // vector registers (copied once, here): in scalar registers they pushed
  // the kernel past the scalar register file, and the spilled values came
  // back by v_readlane in every layer.
  Modal<T> km = A.km;
  if constexpr (sizeof(T) == 4 && (MODE == MODE_CGF || MODE == MODE_MRF)) {
    float* q = reinterpret_cast<float*>(&km);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(Modal<T>) / sizeof(float)); ++i) {
      float v;
      asm volatile("v_mov_b32 %0, %1" : "=v"(v) : "s"(q[i]));
      q[i] = v;
    }
  }
  ApplyStage<T> S[2];
  FusedStage<T, DN> SF;
  MinresStage<T> SM;
  T F[2][4][3];
  T carry[4][3];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int c = 0; c < 3; ++c) carry[q][c] = (T)0;

  // prologue: planes ez0, ez0 + 1 staged (and, unfused, plane ez0 + 2 in flight)
  unsigned mq[2];  // mask of the own node, by parity of the plane from ez0
  T rq[2][3];  // its unmasked input value
  T dq[2][DN];     // CGF: its D^-1
  T rho_next;
  // residual and CG modes: values of the own node read only at its output
  // (RESID: f; CG: D^-1), loaded one layer ahead.  FP64 loads them at the output
  // instead: the queue would not fit its registers.
  constexpr bool kOwnQ = sizeof(T) == 4 && (MODE == MODE_RESID || MODE == MODE_CG);
  T oq[2][3];
  const __amdgpu_buffer_rsrc_t rs_f = vres(A.f), rs_y = vres(A.y), rs_z = vres(A.z);
  const __amdgpu_buffer_rsrc_t rs_do = dres(A.dinv_out, A.dn_out);
  auto load_own = [&](int k, T (&q)[3]) {
    const bool ok = k >= k0 && k < kend;  // planes this block outputs
    const uint32_t o3 = ok ? vw3 : kOOR, so3 = ok ? s3(k) : 0u;
    if constexpr (MODE == MODE_RESID) {
      bload3(rs_f, o3, so3, q);
    } else {
      T d[DN];
      load_d(ok ? vwd : kOOR, ok ? splane(k) : 0u, o3, so3, d);
#pragma unroll
      for (int c = 0; c < DN; ++c) q[c] = d[c];
    }
  };
  if constexpr (MODE == MODE_CGF) {
    FusedStage<T, DN> SF1;
    issue_f(ez0, SF);
    rho_next = load_rho(ez0);
    issue_f(ez0 + 1, SF1);
    cg_prologue();
    stage_f(SF, ez0 & 1, ez0, rq[0], dq[0]);
    mq[0] = SF.m;
    stage_f(SF1, (ez0 + 1) & 1, ez0 + 1, rq[1], dq[1]);
    mq[1] = SF1.m;
  } else if constexpr (MODE == MODE_MRF) {
    MinresStage<T> SM1;
    issue_m(ez0, SM);
    rho_next = load_rho(ez0);
    issue_m(ez0 + 1, SM1);
    mrf_prologue();
    stage_m(SM, ez0 & 1, ez0, rq[0]);
    mq[0] = SM.m;
    stage_m(SM1, (ez0 + 1) & 1, ez0 + 1, rq[1]);
    mq[1] = SM1.m;
  } else {
    issue(ez0, S[0]);
    issue(ez0 + 1, S[1]);
    stage(S[0], ez0 & 1);
    stage(S[1], (ez0 + 1) & 1);
    mq[0] = S[0].m[0];
    mq[1] = S[1].m[0];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      rq[0][c] = S[0].v[0][c];
      rq[1][c] = S[1].v[0][c];
    }
    // the density first, then the next plane: as in every layer, so that
    // the wait for the density leaves the plane's loads in flight
    rho_next = load_rho(ez0);
    if constexpr (kOwnQ) load_own(ez0, oq[0]);
    issue(ez0 + 2, S[0]);
  }
  // the three corner values of the neighbouring columns around the own node
  // (a thread that owns none reads its own slot)
  const int tl1 = writer ? tid - 1 : tl, tlb = writer ? tid - TW : tl, tlbb = writer ? tid - TW - 1 : tl;
  const int cr1 = 9 * tl1, crb = 9 * tlb + 3, crbb = 9 * tlbb + 6;
  T s_below = (T)0;  // s of the element below (diagonal of the residual mode)
  __syncthreads();
  read_face(ez0 & 1, F[0]);
  __syncthreads();  // the first layer restages the buffer of plane ez0

  auto layer = [&](auto parity, int ez) {
    constexpr int P = decltype(parity)::value;
    const T s = scale_of(ez, rho_next);
    rho_next = load_rho(ez + 1);
    if constexpr (kOwnQ) load_own(ez + 1, oq[P ^ 1]);
    loads_priority<T>(true);
    if constexpr (MODE == MODE_CGF) {
      issue_f(ez + 2, SF);
    } else if constexpr (MODE == MODE_MRF) {
      issue_m(ez + 2, SM);
    } else {
      issue(ez + 3, S[P ^ 1]);
    }
    loads_priority<T>(false);
    const T dcol = s_below + s;  // this column's share of the lower-face nodes' diagonal
    s_below = s;
    read_face((ez + 1) & 1, F[P ^ 1]);
    const bool emit = ez >= k0;  // uniform over the block
    T out[4][3];
    layer_product(F[P], F[P ^ 1], s, km, carry, out);
    const int cb = ez & 1;
    if (emit && live) {
#pragma unroll
      for (int a = 1; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 3; ++c) corners[(cb * TS + tid) * 9 + (a - 1) * 3 + c] = out[a][c];
      if constexpr (MODE == MODE_RESID) {
        if (A.z) dcorn[cb * TS + tid] = dcol;
      }
    }
    // the staged plane's values of the own node: into the slot that this
    // layer's output leaves
    T nq[3], nd[DN];
    unsigned nm;
    if constexpr (MODE == MODE_CGF) {
      stage_f(SF, ez & 1, ez + 2, nq, nd);
      nm = SF.m;
    } else if constexpr (MODE == MODE_MRF) {
      stage_m(SM, ez & 1, ez + 2, nq);
      nm = SM.m;
    } else {
      stage(S[P], ez & 1);
      nm = S[P].m[0];
#pragma unroll
      for (int c = 0; c < 3; ++c) nq[c] = S[P].v[0][c];
    }
    __syncthreads();
    {
      // every thread runs the output code; a thread that owns no output node
      // reads its own LDS slots, loads and stores out of range
      const bool wr = emit && writer;
      const uint32_t o3 = emit ? vw3 : kOOR, so3 = emit ? s3(ez) : 0u;
      const unsigned m = wr ? mq[P] : 0u;
      const T* cr = corners + cb * 9 * TS;
      T acc[3], pv[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        acc[c] = ((out[0][c] + cr[cr1 + c]) + cr[crb + c]) + cr[crbb + c];
        pv[c] = rq[P][c];  // the input value at this node, as staged
      }
      if (m) {  // springs, then identity rows of fixed DOFs (rare nodes)
        const int n = gcol[0] + ez * plane;
        if (m & 8u) {
          for (int sI = 0; sI < A.nspring; ++sI) {
            const int64_t d = A.sdof[sI] - (int64_t)3 * n;
#pragma unroll
            for (int c = 0; c < 3; ++c)
              if (d == c) acc[c] += A.sk[sI] * pv[c];
          }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c)
          if ((m >> c) & 1u) acc[c] = pv[c];
      }
      // partial sums count owned nodes only (a select: values of a thread
      // without an owned node may be anything, NaN included)
      auto own_only = [wr](double v) { return wr ? v : 0.0; };
      auto own_t = [wr](T v) { return wr ? v : (T)0; };
      if constexpr (MODE == MODE_RESID) {
        T fv[3], rv[3], zv[3] = {(T)0, (T)0, (T)0};
        if constexpr (kOwnQ) {
#pragma unroll
          for (int c = 0; c < 3; ++c) fv[c] = oq[P][c];
        } else {
          bload3(rs_f, o3, so3, fv);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) rv[c] = fv[c] - acc[c];
        if (A.z) {  // the start of a CG solve (uniform)
          // Jacobi diagonal: ke_diag * sum of s over the node's 8 elements,
          // one value (and one division) for the node's three DOFs
          const T d0 = (T)A.ke_diag * (((dcol + dcorn[cb * TS + tl1]) + dcorn[cb * TS + tlb]) + dcorn[cb * TS + tlbb]);
          const T dinv0 = d0 > (T)0 ? (T)1 / d0 : (T)0;
          T d[3] = {dinv0, dinv0, dinv0};
          if (m) {  // springs and fixed DOFs (rare nodes)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              T dc = d0;
              if (m & 8u)
                for (int sI = 0; sI < A.nspring; ++sI)
                  if (A.sdof[sI] == (int64_t)(3 * (gcol[0] + ez * plane) + c)) dc += A.sk[sI];
              if ((m >> c) & 1u) dc = (T)1;
              d[c] = dc > (T)0 ? (T)1 / dc : (T)0;
            }
          }
#pragma unroll
          for (int c = 0; c < 3; ++c) zv[c] = d[c] * rv[c];
          bstore3(rs_z, o3, so3, zv);
          if (A.dinv_out && rhs0 == 0) {  // the same for every RHS
            if (A.dn_out == 1) zstore1<T>(rs_do, emit ? vwd : kOOR, emit ? sd(ez) : 0u, dinv0);
            else bstore3(rs_do, o3, so3, d);
          }
        }
        bstore3(rs_y, A.y ? o3 : kOOR, so3, rv);
        T rr = (T)0, rm = (T)0, ff = (T)0, rz = (T)0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          rr += rv[c] * rv[c];
          rm = fmax(rm, fabs(rv[c]));
          ff += fv[c] * fv[c];
          rz += rv[c] * zv[c];
        }
        tpart[0] += own_t(rr);
        tpart[1] = fmax(tpart[1], own_t(rm));
        tpart[2] += own_t(ff);
        tpart[3] += own_t(rz);
      } else {
        bstore3(rs_y, o3, so3, acc);
        if constexpr (MODE == MODE_CG || MODE == MODE_LZ) {
          T q3[3];  // CG: D^-1
          if constexpr (MODE == MODE_CG) {
            T d[DN];
            if constexpr (kOwnQ) {
#pragma unroll
              for (int c = 0; c < DN; ++c) d[c] = oq[P][c];
            } else {
              load_d(emit ? vwd : kOOR, emit ? splane(ez) : 0u, o3, so3, d);
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) q3[c] = dof_d(d, m, c);
          }
          double yu = 0.0, uu = 0.0;
          T ss = (T)0;
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            yu += (double)acc[c] * (double)pv[c];
            if constexpr (MODE == MODE_CG) ss += acc[c] * (q3[c] * acc[c]);
            else uu += (double)pv[c] * (double)pv[c];
          }
          part[1] += own_only(yu);  // p.s / y.u
          if constexpr (MODE == MODE_CG) tpart[2] += own_t(ss);  // s.D^-1 s
          else part[0] += own_only(uu);                         // u.u
        }
        if constexpr (MODE == MODE_CGF || MODE == MODE_MRF) {
          double yu = 0.0;
#pragma unroll
          for (int c = 0; c < 3; ++c) yu += (double)acc[c] * (double)pv[c];
          part[1] += own_only(yu);  // p'.s' / <K y, y>
        }
        if constexpr (MODE == MODE_CGF) {
          T ss = (T)0;
#pragma unroll
          for (int c = 0; c < 3; ++c) ss += acc[c] * (dof_d(dq[P], m, c) * acc[c]);
          tpart[2] += own_t(ss);  // s'.D^-1 s'
        }
      }
    }
    mq[P] = nm;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      rq[P][c] = nq[c];
    }
    if constexpr (MODE == MODE_CGF) {
#pragma unroll
      for (int c = 0; c < DN; ++c) dq[P][c] = nd[c];
    }
  };
  for (int ez = ez0; ez < kend; ez += 2) {
    layer(std::integral_constant<int, 0>{}, ez);
    if (ez + 1 >= kend) break;
    layer(std::integral_constant<int, 1>{}, ez + 1);
  }

  if constexpr (MODE == MODE_CG || MODE == MODE_CGF || MODE == MODE_LZ) {
    // CG: step k's product -> set k & 1; CGF: step k + 1's -> set (k + 1) & 1;
    // LZ: iteration k's
    const int par = (MODE == MODE_CGF ? A.step + 1 : A.step) & 1;
    // CG: p.s, s.D^-1 s   CGF: also r.z (, r.r)   LZ: y.u, u.u
    constexpr int NV = MODE == MODE_CGF ? (RR ? 4 : 3) : 2;
    double* dst[NV];
    double v[NV];
    dst[0] = pslot(parts, P_PQ0 + par, 0, kMaxP);
    v[0] = part[1];
    if constexpr (MODE == MODE_LZ) {
      dst[1] = pslot(parts, P_RZ0 + par, 0, kMaxP);
      v[1] = part[0];
    } else {
      dst[1] = pslot(parts, P_EP0 + par, 0, kMaxP);
      v[1] = (double)tpart[2];
    }
    if constexpr (MODE == MODE_CGF) {
      dst[2] = pslot(parts, P_RZ0 + par, 0, kMaxP);
      v[2] = (double)tpart[0];
      if constexpr (RR) {
        dst[3] = pslot(parts, P_RN0 + par, 0, kMaxP);
        v[3] = (double)tpart[1];
      }
    }
    write_parts<NV, 0u>(v, dst, lb);
    // LZ: u.u is the norm's square of iteration `step` - 1 too (which had a launch of
    // its own: Alg. 3 iteration at 128x64x64 FP32 469.9 -> 464.8 us, plane 576x192
    // FP64 280.6 -> 276.6 us)
    if constexpr (MODE == MODE_LZ)
      if (tid == 0) pslot(parts, P_KRN0 + (par ^ 1), 0, kMaxP)[lb] = v[1];
  }
  if constexpr (MODE == MODE_MRF) {
    // ||y||^2 -> the norm slot of iteration t; <K y, y> and <R2, y> -> the
    // product partials of iteration t + 1
    const int itn = A.step;
    double v[3] = {part[0], part[1], part[2]};
    double* dst[3] = {pslot(parts, P_KRN0 + (itn & 1), 0, kMaxP), pslot(parts, P_PQ0 + ((itn + 1) & 1), 0, kMaxP),
                      pslot(parts, P_RZ0 + ((itn + 1) & 1), 0, kMaxP)};
    write_parts<3, 0u>(v, dst, lb);
  }
  if constexpr (MODE == MODE_RESID) {
    if (!A.parts) return;
    if (lb == 0 && tid == 0) {   // a new solve starts from this residual
      Scalars* sc = const_cast<Scalars*>(A.sc);
      sc->done[rhs0] = 0.0;
      sc->status[rhs0] = 0.0;
      sc->steps[rhs0] = 0.0;
    }
    double v[4];
    double* dst[4];
    for (int i = 0; i < 4; ++i) v[i] = (double)tpart[i];
    dst[0] = pslot(parts, P_RNF, 0, kMaxP);
    dst[1] = pslot(parts, P_RIF, 0, kMaxP);
    dst[2] = pslot(parts, P_FN, 0, kMaxP);
    dst[3] = pslot(parts, P_RZ0, 0, kMaxP);  // r.z and r.r of step 0
    write_parts<4, 0x2u>(v, dst, lb);
    if (tid == 0) pslot(parts, P_RN0, 0, kMaxP)[lb] = v[0];
  }
}

// ===========================================================================
// The last CG step of a solve fused with the sensitivity of Sec. 3 (one
// RHS).  On the tiling of k_apply, every staged node gets x' = x + alpha p;
// the owner of the node stores x', and forms r' = r - alpha s for the final
// residual norms and f . x'.
// Each element owned by the block gets
//   dobj_e = -ds_e x'_e^T KE x'_e  (times 1/Hs_e when given)
// from the face modes of its two faces.  Nothing is scattered back to the
// nodes, so there is no corner exchange; one barrier per layer guards the
// double-buffered node planes.
// ===========================================================================
template <typename T>
struct SensStage {
  T x[3], p[3];         // every staged node
  T r[3], s[3], f[3];   // owned node only
  unsigned m;
};

template <typename T>
__global__ void __launch_bounds__(kApplyMaxThreads)
    k_cg_sens(ApplyArgs<T> A) {
  extern __shared__ __align__(16) unsigned char apply_smem[];
  const int b = blockIdx.x;
  const int lb = (b & 7) * A.per_xcd + (b >> 3);
  if (lb >= A.nblocks) return;
  const Geo G = A.g;
  const int BX = A.bx, BY = A.by;
  const int NW = BX + 1;
  const int NS = NW * (BY + 1);
  T* nodes = reinterpret_cast<T*>(apply_smem);  // [2][NS][3]
  // one thread per node column of the tile (the node layout of k_apply)
  const int tid = threadIdx.x;
  const bool live = tid < NS;
  const int tl = live ? tid : 0;
  const int ty = (int)((tl + 0.5f) * A.inv_tw), tx = tl - ty * NW;  // exact: tl < 512
  const int t2 = (int)div_small(lb, A.inv_tx);
  const int bxi = lb - t2 * A.tiles_x;
  const int bz = (int)div_small(t2, A.inv_ty);
  const int byi = t2 - bz * A.tiles_y;
  const int x0 = bxi * (BX - 1) - 1, y0 = byi * (BY - 1) - 1;
  const int ex = x0 + tx, ey = y0 + ty;
  const int k0 = bz * A.dz;
  const int kend = min(k0 + A.dz, G.nz + 1);
  const int ez0 = k0 == 0 ? 0 : k0 - 1;
  const int elem_end = min(k0 + A.dz, G.nz);   // element layers [k0, elem_end) belong to this slab
  const int plane = G.nxn * G.nyn;
  const bool writer = live && tx >= 1 && ty >= 1 && tx < BX && ty < BY && ex <= G.nx && ey <= G.ny;
  const bool elem_owner = writer && ex < G.nx && ey < G.ny;
  // As in k_apply, the vectors are addressed through buffer resources based
  // at the block's first plane ez0: a plane past the slab or a thread that
  // owns no node gets an out-of-range offset, so its loads return 0 and its
  // stores are dropped, with no branch around them.
  const int li = 3 * tl;  // padding threads stage thread 0's node again (the same value into the same slot)
  const bool col = ex >= 0 && ex <= G.nx && ey >= 0 && ey <= G.ny;
  const uint32_t vc1 = col ? (uint32_t)(ex + G.nxn * ey) : kOOR;
  const uint32_t vc3 = col ? (uint32_t)(3 * sizeof(T)) * vc1 : kOOR;
  const uint32_t vw3 = writer ? vc3 : kOOR;  // the node a thread owns
  const uint32_t ve = elem_owner ? (uint32_t)sizeof(T) * (uint32_t)(ex + G.nx * ey) : kOOR;  // its element
  const int64_t pbase = (int64_t)ez0 * plane;  // first node of plane ez0
  auto vres = [&](const T* v) { return zrsrc(v ? v + 3 * pbase : v); };
  auto splane = [&](int k) -> uint32_t { return (uint32_t)(k - ez0) * (uint32_t)plane; };
  const __amdgpu_buffer_rsrc_t rs_m = zrsrc(A.mask + pbase), rs_x = vres(A.xi), rs_r = vres(A.ri),
                               rs_p = vres(A.pi), rs_s = vres(A.si), rs_f = vres(A.fvec), rs_xo = vres(A.xo);
  const int64_t ebase = (int64_t)ez0 * G.nx * G.ny;  // first element of layer ez0
  const __amdgpu_buffer_rsrc_t rs_rho = zrsrc(A.rho + ebase), rs_hs = zrsrc(A.Hsi ? A.Hsi + ebase : A.Hsi),
                               rs_do = zrsrc(A.dobj + ebase);

  // the step's alpha (every block, same order; called after the first
  // planes' loads are issued, so the two latencies overlap)
  T al = (T)0;
  auto coefficients = [&]() {
    const int par = A.step & 1;
    double pre[5];
    const double* src[5] = {pslot(A.P, P_RZ0 + par, 0, kMaxP), pslot(A.P, P_PQ0 + par, 0, kMaxP),
                            pslot(A.P, P_EP0 + par, 0, kMaxP), pslot(A.P, P_RN0 + par, 0, kMaxP),
                            pslot(A.P, P_FN, 0, kMaxP)};
    const bool tol = A.rtol > 0.0;  // r.r and f.f only for the tolerance test
    const int cnt[5] = {A.n_gam, A.n_apply, A.n_apply, tol ? A.n_gam : 0, tol ? A.n_fn : 0};
    reduce_parts<5, 0u>(pre, src, cnt);
    double alpha, beta;
    cg_coefficients(pre[0], pre[1], pre[2], pre[3], pre[4], 0, par, A.rtol, const_cast<Scalars*>(A.sc),
                    lb == 0 && tid == 0, alpha, beta);
    al = wave_uniform((T)alpha);
  };
  // r'.r', max|r'|, f.x', and the sum of the block's element sensitivities
  double part[4] = {0.0, 0.0, 0.0, 0.0};

  auto owns = [&](int k) { return k >= 0 && k <= G.nz && k >= k0 && k < kend; };  // the block's planes
  auto issue = [&](int k, SensStage<T>& S) {
    const bool kv = k >= 0 && k <= kend && k <= G.nz;  // planes past kend are never read
    const uint32_t so1 = kv ? splane(k) : 0u, so3 = (uint32_t)(3 * sizeof(T)) * so1;
    const uint32_t o3 = kv ? vc3 : kOOR, oo = owns(k) ? vw3 : kOOR;
    S.m = __builtin_amdgcn_raw_buffer_load_b8(rs_m, kv ? vc1 : kOOR, so1, 0);
    zload3<T>(rs_x, o3, so3, S.x);
    zload3<T>(rs_p, o3, so3, S.p);
    zload3<T>(rs_r, oo, so3, S.r);  // used by the owner only
    zload3<T>(rs_s, oo, so3, S.s);
    zload3<T>(rs_f, A.fvec ? oo : kOOR, so3, S.f);
  };
  auto stage = [&](const SensStage<T>& S, int buf, int k) {
    T* nb = nodes + buf * (3 * NS) + li;
    const bool ok = owns(k);
    T xn[3];
    double rr = 0.0, rm = 0.0, fx = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      xn[c] = S.x[c] + al * S.p[c];
      nb[c] = zmasked(S.m, c, xn[c]);
      const T rn = S.r[c] - al * S.s[c];
      rr += (double)rn * (double)rn;
      rm = fmax(rm, fabs((double)rn));
      fx += (double)S.f[c] * (double)xn[c];
    }
    zstore3<T>(rs_xo, ok ? vw3 : kOOR, ok ? (uint32_t)(3 * sizeof(T)) * splane(k) : 0u, xn);
    const bool own = ok && writer;
    part[0] += own ? rr : 0.0;
    part[1] = fmax(part[1], own ? rm : 0.0);
    part[2] += own ? fx : 0.0;
  };
  // the lower-left node of the thread's element (node 0's for threads
  // without an element: their reads stay inside the plane)
  const int lf = (live && tx < BX && ty < BY) ? li : 0;
  auto read_face = [&](int buf, T (&F)[4][3]) {
    const T* nb = nodes + buf * (3 * NS) + lf;
    T u4[4][3];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int c = 0; c < 3; ++c) u4[a][c] = nb[3 * (a >> 1) * NW + 3 * (a & 1) + c];
    face_modes(u4, F);
  };
  // scalar byte offset of an element layer; a layer that is not the block's is out of range
  auto eown = [&](int ez) { return ez >= k0 && ez < elem_end; };
  auto eso = [&](int ez) -> uint32_t {
    return eown(ez) ? (uint32_t)sizeof(T) * (uint32_t)((ez - ez0) * (G.nx * G.ny)) : 0u;
  };
  // density and 1/Hs of the element of a layer, loaded a layer ahead
  auto load_elem = [&](int ez, T (&v)[2]) {
    const uint32_t vo = eown(ez) ? ve : kOOR, so = eso(ez);
    v[0] = zload1<T>(rs_rho, vo, so);
    const T hv = zload1<T>(rs_hs, A.Hsi ? vo : kOOR, so);
    v[1] = A.Hsi ? hv : (T)1;
  };

  SensStage<T> S;
  T F[2][4][3];
  T ev[2][2];
  {
    SensStage<T> S1;
    issue(ez0, S);
    issue(ez0 + 1, S1);
    coefficients();
    stage(S, ez0 & 1, ez0);
    stage(S1, (ez0 + 1) & 1, ez0 + 1);
  }
  load_elem(ez0, ev[0]);
  __syncthreads();
  read_face(ez0 & 1, F[0]);
  __syncthreads();

  auto layer = [&](auto parity, int ez) {
    constexpr int P = decltype(parity)::value;
    load_elem(ez + 1, ev[P ^ 1]);
    loads_priority<T>(true);
    issue(ez + 2, S);
    loads_priority<T>(false);
    read_face((ez + 1) & 1, F[P ^ 1]);
    {
      T c[3][8], z[3][8];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        c[i][0] = (T)0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (q) c[i][q] = F[P][q][i] + F[P ^ 1][q][i];
          c[i][q + 4] = F[P ^ 1][q][i] - F[P][q][i];
        }
      }
      modal_ke(c, A.km, z);
      double en = 0.0;
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int q = 1; q < 8; ++q) en += (double)c[i][q] * (double)z[i][q];
      const double dc = -(double)simp_ds<T>(ev[P][0], A.sp) * en;  // d objective / d rho_e
      zstore1<T>(rs_do, eown(ez) ? ve : kOOR, eso(ez), (T)(dc * (double)ev[P][1]));
      // The filter weights are symmetric, so the filtered gradient
      // H^T (dc / Hs) sums to sum_e dc_e: its mean for the step, formed here.
      part[3] += (elem_owner && ez >= k0 && ez < elem_end) ? dc : 0.0;
    }
    stage(S, ez & 1, ez + 2);
    __syncthreads();
  };
  for (int ez = ez0; ez < kend; ez += 2) {
    layer(std::integral_constant<int, 0>{}, ez);
    if (ez + 1 >= kend) break;
    layer(std::integral_constant<int, 1>{}, ez + 1);
  }
  double* dst[4] = {pslot(A.P, P_RNF, 0, kMaxP), pslot(A.P, P_RIF, 0, kMaxP), pslot(A.P, P_DOT, 0, kMaxP),
                     pslot(A.P, P_GSUM, 0, kMaxP)};
  write_parts<4, 0x2u>(part, dst, lb);
}

template <typename T>
static size_t sens_lds_bytes(int bx, int by) {
  return sizeof(T) * (size_t)(2 * 3 * (bx + 1) * (by + 1));
}

template <typename T, int MODE>
static size_t apply_lds_bytes(int bx, int by) {
  const size_t ns = (size_t)(bx + 1) * (by + 1);                      // nodes per plane
  const size_t ts = node_layout<MODE>() ? ns : (size_t)bx * by;      // corner slots
  return sizeof(T) * (2 * 3 * ns + 2 * 9 * ts + 2 * ts);
}

// The z-march addresses each vector from the block's first plane with
// 32-bit byte offsets: its planes (dz + 3 at most: the slab, the halo layer
// below, the prefetched plane above) must span less than 2 GiB.
bool apply_offsets_fit(const Geo& G, int dz, size_t value_bytes) {
  return (int64_t)(3 * value_bytes) * G.nxn * G.nyn * (dz + 3) < ((int64_t)1 << 31);
}

// Tile of the fused steps on large grids (2^21 elements and more), where the
// memory path bounds them: blocks of 240 to 256 threads, two or three per CU.
// The cost of a choice is its rounds of resident blocks (the last one, partly
// filled, counts half and half its filling) times the planes that a block
// reads, times
//   - 1.55 with three blocks per CU: a round of three measured 1.55 times as
//     long as one of two (256x128x128 in one round of three 113 us a step,
//     320x160x160 in three of two 219 and two of three 226 us);
//   - the partial cache lines of a tile's rows, one line of 64 bytes per row.
// Against one fixed tile (27 x 8 columns, 33 layers), FP32 CG step: 320x160x160
// 251 -> 219 us, 230x130x150 140 -> 125 us, 220x115x115 (before: the model
// below) 88 -> 79 us; FP64 230x130x150 261 -> 245 us; 256x128x128 and
// 384x192x192 as before within 1%.
// No choice (the model below then takes the grid) where the shapes do not fit.
// Planes that fill less than half of their threads, FP32 CG step, these shapes
// against the model's: 1x1483x1483 519 and 192 us, 8x524x524 76 and 57 (0.40
// filled), 12x428x428 54 and 56 (0.58), 469x10x469 60 and 58 (0.75).  And fewer
// planes than the thinnest slab: 1048x1050x2 165 and 125 us, 396x397x14 53 and
// 48.
template <typename T, int MODE>
static TileChoice choose_large_tile(const Geo& G, int nrhs, int n_cu, int lds_per_cu) {
  constexpr int kMinDz = 16;
  static const int shapes[][2] = {{27, 8}, {31, 7}, {35, 6}, {24, 9}, {20, 11}, {18, 12}};
  TileChoice best{};
  if (G.nzn < kMinDz) return best;
  double best_cost = 1e300;
  for (const auto& sh : shapes) {
    const int bx = sh[0], by = sh[1], threads = zmarch_threads<MODE>(bx, by);
    const int tiles_x = (G.nxn + bx - 2) / (bx - 1), tiles_y = (G.nyn + by - 2) / (by - 1);
    const size_t need = apply_lds_bytes<T, MODE>(bx, by);
    if (need > kApplyMaxLds) continue;
    for (int cap = 2; cap <= 3; ++cap) {
      const size_t lds = std::max(need, (size_t)lds_for_block_cap(lds_per_cu, cap));
      int occ = 0;
      const hipError_t oe = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_apply<T, MODE>, threads, lds);
      if (oe != hipSuccess || occ < cap || lds > kApplyMaxLds) continue;
      for (int dz = kMinDz; dz <= std::min(49, G.nzn); ++dz) {
        const int slabs = (G.nzn + dz - 1) / dz;
        const int64_t nb = (int64_t)tiles_x * tiles_y * slabs;
        if (nb > kApplyMaxBlocks || !apply_offsets_fit(G, dz, sizeof(T))) continue;
        const double r = (double)nb * nrhs / ((double)cap * n_cu), full = std::floor(r), part = r - full;
        const double rounds = full + (part > 0.0 ? 0.5 + 0.5 * part : 0.0);
        const double cost = rounds * (dz + 3) * (cap == 3 ? 1.55 : 1.0) * (1.0 + 64.0 / (3 * sizeof(T)) / (bx + 1));
        if (cost < best_cost) {
          best_cost = cost;
          best = TileChoice{bx, by, dz, tiles_x, tiles_y, slabs, (int)nb, cap};
        }
      }
    }
  }
  const double threads = (double)best.tiles_x * best.tiles_y * (best.bx + 1) * (best.by + 1);
  return (double)G.nxn * G.nyn >= 0.5 * threads ? best : TileChoice{};
}

// The time of one layer of a round with w waves per CU, in wave-layers.  K u and
// the other element-layout kernels: w + 8 (K u at 256x128x128 FP32: 1.07 us per
// layer with 8 waves, 1.49 with 14, 1.58 with 16).  The fused steps in FP64: w +
// 3.9 (CG step at 64x32x32: 12.9 us in four layers of 4 waves, 13.9 in three of
// 8).  In FP32 a layer takes as long with 4 waves as with 8, and from there
// grows as w: at 97x53x41 five layers of 8 waves 13.8 us, seven of 4 15.2 us.
template <typename T, int MODE>
static double layer_cost(double w) {
  if (!node_layout<MODE>()) return w + 8.0;
  return sizeof(T) == 8 ? w + 3.9 : std::max(w, 8.0);
}

// Tile shape and slab depth for one apply variant.  The cost of a choice is the
// time of a layer (layer_cost) summed over the busiest CU's rounds of resident
// blocks, times the layers of a block (+ 2 for the prologue).  Rows count a
// little more the shorter they are (97x53x41, fused CG step with equal blocks:
// 13.8 us with 35 columns, 14.1 with 16, 14.4 with 10), up to the grid's own
// width (8x8x65000, FP32 MINRES pass: 195 us with 22 columns, 170 with 10).  Before, a layer cost
// max(w, 8) in every kernel: K u at 256x128x128 48 -> 39.6 us; FP64 CG step at
// 64x32x32 13.9 -> 13.1 us, at 180x90x90 87 -> 79 us.
template <typename T, int MODE>
static TileChoice choose_tile(const Geo& G, int nrhs, int n_cu, int lds_per_cu, int override_shape) {
  // fixed fields of a caller's override (FBTO_OPT_APPLY_TILE / _CGF_TILE)
  const int want_bx = override_shape & 0xff, want_by = (override_shape >> 8) & 0xff,
            want_dz = (override_shape >> 16) & 0xff;
  if constexpr (MODE == MODE_CGF || MODE == MODE_MRF) {
    if (override_shape == 0 && G.E >= ((int64_t)1 << 21)) {
      const TileChoice t = choose_large_tile<T, MODE>(G, nrhs, n_cu, lds_per_cu);
      if (t.nblocks) return t;
    }
  }
  TileChoice best{};
  double best_cost = 1e300;
  for (int bx = 8; bx <= 64; ++bx) {
    if (want_bx && bx != want_bx) continue;
    for (int by = 4; by <= 64; ++by) {
      if (want_by && by != want_by) continue;
      const int ts = node_layout<MODE>() ? (bx + 1) * (by + 1) : bx * by;  // threads
      // at most four waves: every layer ends at a block-wide barrier, and
      // blocks of up to one wave per SIMD measured fastest
      if (ts < 128 || ts > 256) continue;
      const size_t lds = MODE == MODE_SENSF ? sens_lds_bytes<T>(bx, by) : apply_lds_bytes<T, MODE>(bx, by);
      if (lds > kApplyMaxLds) continue;
      const int waves = (ts + 63) / 64;
      int occ = 0;
      hipError_t oe;
      if constexpr (MODE == MODE_SENSF)
        oe = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_cg_sens<T>, 64 * waves, lds);
      else
        oe = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_apply<T, MODE>, 64 * waves, lds);
      if (oe != hipSuccess || occ < 1) continue;
      const int tiles_x = (G.nxn + bx - 2) / (bx - 1);
      const int tiles_y = (G.nyn + by - 2) / (by - 1);
      for (int dz = 1; dz <= std::min(G.nzn, 64); ++dz) {
        if (want_dz && dz != want_dz) continue;
        // the planes a block reads, addressed by 32-bit byte offsets
        if (!apply_offsets_fit(G, dz, sizeof(T))) continue;
        const int slabs = (G.nzn + dz - 1) / dz;
        const int64_t nb = (int64_t)tiles_x * tiles_y * slabs;
        if (nb > kApplyMaxBlocks) continue;
        const int64_t per_cu = (nb * nrhs + n_cu - 1) / n_cu;
        const int64_t full = per_cu / occ, rem = per_cu % occ;
        // a block's waves go to the CU's four SIMDs; a count that does not
        // spread evenly (3, 5, 6, 7) leaves one SIMD with more work, as if
        // the block had the next multiple of four
        const double w = (waves == 1 || waves == 2 || waves == 4 || waves == 8) ? waves : (waves + 3) / 4 * 4;
        const double cost = (full * layer_cost<T, MODE>(occ * w) + (rem ? layer_cost<T, MODE>(rem * w) : 0.0)) *
                            (dz + 2.0) * (1.0 + 1.0 / std::min(bx + 1, G.nxn + 1));
        if (cost < best_cost) {
          best_cost = cost;
          best = TileChoice{bx, by, dz, tiles_x, tiles_y, slabs, (int)nb, (override_shape >> 24) & 0xf};
        }
      }
    }
  }
  return best;
}

template <typename T, int MODE, bool RR = true, int DN = 1, int XU = 1>
static hipError_t launch_apply_t(fbto_grid_s* g, const ApplyArgs<T>& A0, int nrhs, hipStream_t st, int* nb_out) {
  TileChoice& t = g->tiles[sizeof(T) == 8 ? 1 : 0][nrhs - 1][MODE];
  if (t.nblocks == 0) {
    t = choose_tile<T, MODE>(g->geo, nrhs, g->n_cu, g->lds_per_cu, g->tile_override[MODE == MODE_CGF ? 1 : 0]);
    if (t.nblocks == 0) return hipErrorInvalidConfiguration;
  }
  if (t.nblocks > g->max_partials) return hipErrorInvalidValue;
  if (nb_out) *nb_out = t.nblocks;
  ApplyArgs<T> A = A0;
  A.bx = t.bx;
  A.by = t.by;
  A.tiles_x = t.tiles_x;
  A.tiles_y = t.tiles_y;
  A.slabs = t.slabs;
  A.dz = t.dz;
  A.nblocks = t.nblocks;
  A.per_xcd = (t.nblocks + 7) / 8;
  A.inv_tx = inv_small(t.tiles_x);
  A.inv_ty = inv_small(t.tiles_y);
  A.inv_tw = 1.0f / (float)(node_layout<MODE>() ? t.bx + 1 : t.bx);
  const int grid = A.per_xcd * 8;
  size_t lds = apply_lds_bytes<T, MODE>(t.bx, t.by);
  if (t.cap) lds = std::max(lds, (size_t)lds_for_block_cap(g->lds_per_cu, t.cap));
  const int threads = zmarch_threads<MODE>(t.bx, t.by);  // whole waves
  hipLaunchKernelGGL((k_apply<T, MODE, RR, DN, XU>), dim3(grid, nrhs), dim3(threads), lds, st, A);
  return hipGetLastError();
}

template <typename T, int MODE, bool RR = true, int DN = 1, int XU = 1>
static hipError_t launch_apply_mode(fbto_grid_s* g, ApplyArgs<T> A, int nrhs, hipStream_t st, int* nb_out) {
  A.g = g->geo;
  A.mask = g->mask;
  A.km = modal_of<T>(g);
  A.sp = g->simp;
  A.nspring = g->n_springs;
  A.sdof = g->spring_dof;
  A.sk = spring_k_of<T>(g);
  A.P = g->partials;
  A.sc = g->sc;
  // One RHS per block (the per-RHS state of the z-march, two face-mode sets, the
  // modal carry and the staged loads, fills the register file), all of them in
  // one launch: on small grids a launch per load case left most CUs idle.
  // Three loads at 97x53x41, FP32: a CG step of all three 39 -> 18 us.
  if (g->max_partials != kApplyMaxBlocks || nrhs < 1 || nrhs > 4) return hipErrorInvalidValue;
  return launch_apply_t<T, MODE, RR, DN, XU>(g, A, nrhs, st, nb_out);
}

int apply_max_blocks(const Geo&, int) { return kApplyMaxBlocks; }

template <typename T>
hipError_t launch_apply(fbto_grid_s* g, const T* rho, const T* u, T* y, int nrhs, hipStream_t st) {
  if (g->dim == 2) return plane_apply<T>(g, rho, u, y, nrhs, st);
  ApplyArgs<T> A{};
  A.rho = rho;
  A.u = u;
  A.y = y;
  return launch_apply_mode<T, MODE_APPLY>(g, A, nrhs, st, nullptr);
}

template <typename T>
hipError_t launch_resid(fbto_grid_s* g, const T* rho, const T* u, const T* f, T* r, int parts, int nrhs,
                        hipStream_t st, int* nb_out) {
  if (g->dim == 2) return plane_resid<T>(g, rho, u, f, r, nullptr, nullptr, parts, nrhs, st, nb_out);
  ApplyArgs<T> A{};
  A.rho = rho;
  A.u = u;
  A.y = r;
  A.f = f;
  A.parts = parts;
  return launch_apply_mode<T, MODE_RESID>(g, A, nrhs, st, nb_out);
}

template <typename T>
hipError_t launch_resid_diag(fbto_grid_s* g, const T* rho, const T* u, const T* f, T* r, T* z, int nrhs,
                             hipStream_t st, int* nb_out) {
  Vecs& V = vecs_of<T>(g);
  if (g->dim == 2) return plane_resid<T>(g, rho, u, f, r, (T*)V.invD, z, 1, nrhs, st, nb_out);
  ApplyArgs<T> A{};
  A.rho = rho;
  A.u = u;
  A.y = r;
  A.f = f;
  A.parts = 1;
  A.dinv_out = (T*)V.invD;
  A.dn_out = g->n_springs > 0 ? 3 : 1;
  A.ke_diag = g->ke_diag;
  A.z = z;
  return launch_apply_mode<T, MODE_RESID>(g, A, nrhs, st, nb_out);
}

template <typename T>
hipError_t launch_apply_cg(fbto_grid_s* g, const T* rho, const T* p, T* s, int nrhs, int step, hipStream_t st,
                           int* nb_out) {
  Vecs& V = vecs_of<T>(g);
  if (g->dim == 2) return plane_apply_cg<T>(g, rho, p, (const T*)V.invD, s, nrhs, step, st, nb_out);
  ApplyArgs<T> A{};
  A.rho = rho;
  A.u = p;
  A.dinv = (const T*)V.invD;
  A.y = s;
  A.step = step;
  return g->n_springs > 0 ? launch_apply_mode<T, MODE_CG, true, 3>(g, A, nrhs, st, nb_out)
                          : launch_apply_mode<T, MODE_CG, true, 1>(g, A, nrhs, st, nb_out);
}

template <typename T>
hipError_t launch_apply_lanczos(fbto_grid_s* g, const T* rho, const T* u, T* y, int step, hipStream_t st,
                                int* nb_out) {
  if (g->dim == 2) return plane_apply_lanczos<T>(g, rho, u, y, step, st, nb_out);
  ApplyArgs<T> A{};
  A.rho = rho;
  A.u = u;
  A.y = y;
  A.step = step;
  return launch_apply_mode<T, MODE_LZ>(g, A, 1, st, nb_out);
}

template <typename T>
hipError_t launch_cg_sens(fbto_grid_s* g, const T* rho, const CgSet<T>& in, T* x, const T* f, T* dobj, const T* Hsi,
                          int step, const CgCnt& cn, double rtol, hipStream_t st, int* nb_out) {
  TileChoice& t = g->tiles[sizeof(T) == 8 ? 1 : 0][0][MODE_SENSF];
  if (t.nblocks == 0) {
    t = choose_tile<T, MODE_SENSF>(g->geo, 1, g->n_cu, g->lds_per_cu, g->tile_override[0]);
    if (t.nblocks == 0) return hipErrorInvalidConfiguration;
  }
  if (t.nblocks > g->max_partials || g->max_partials != kApplyMaxBlocks) return hipErrorInvalidValue;
  if (nb_out) *nb_out = t.nblocks;
  ApplyArgs<T> A{};
  A.g = g->geo;
  A.mask = g->mask;
  A.km = modal_of<T>(g);
  A.sp = g->simp;
  A.P = g->partials;
  A.sc = g->sc;
  A.rho = rho;
  A.xi = in.x; A.ri = in.r; A.pi = in.p; A.si = in.s;
  A.xo = x;
  A.dobj = dobj;
  A.Hsi = Hsi;
  A.fvec = f;
  A.step = step;
  A.n_gam = cn.gam;
  A.n_apply = cn.apply;
  A.n_fn = cn.fn;
  A.rtol = rtol;
  A.bx = t.bx;
  A.by = t.by;
  A.tiles_x = t.tiles_x;
  A.tiles_y = t.tiles_y;
  A.slabs = t.slabs;
  A.dz = t.dz;
  A.nblocks = t.nblocks;
  A.per_xcd = (t.nblocks + 7) / 8;
  A.inv_tx = inv_small(t.tiles_x);
  A.inv_ty = inv_small(t.tiles_y);
  A.inv_tw = 1.0f / (float)(t.bx + 1);
  const int grid = A.per_xcd * 8;
  const int threads = zmarch_threads<MODE_SENSF>(t.bx, t.by);
  size_t lds = sens_lds_bytes<T>(t.bx, t.by);
  if (t.cap) lds = std::max(lds, (size_t)lds_for_block_cap(g->lds_per_cu, t.cap));
  hipLaunchKernelGGL((k_cg_sens<T>), dim3(grid), dim3(threads), lds, st, A);
  return hipGetLastError();
}

// Grids whose iterate is updated every second step: 2^19 elements and more,
// without springs (CG).  Single and paired, in us per step:
//   FP32 CG   64x32x32 8.43, 8.42   64^3 12.6, 12.3   128x64x64 16.9, 16.4   128^3 41.3, 39.8
//   FP64 CG   64x32x32 10.4, 10.3   64^3 17.9, 17.4   128x64x64 26.4, 25.4   128^3 112, 106
//   FP32 MRF  64x32x32 9.45, 9.27   64^3 14.0, 13.4   128x64x64 19.8, 18.1   128^3 48.9, 44.5
//   FP64 MRF  64x32x32 11.1, 10.5   64^3 19.9, 18.8   128x64x64 29.4, 26.8   128^3 130, 110
// Two kernels in turn cost nothing that these show; where the rule's line lies
// every one of them gains 3% or more.  Below 2^16 elements CG gains nothing (-1 to
// +2%), and a whole 16x8x8 FP64 iteration measured 2% slower.
bool cg_pairs_updates(const fbto_grid_s* g) { return minres_pairs_updates(g) && g->n_springs == 0; }
bool minres_pairs_updates(const fbto_grid_s* g) { return g->dim == 3 && g->geo.E >= ((int64_t)1 << 19); }

template <typename T>
hipError_t launch_cg_fused(fbto_grid_s* g, const T* rho, const CgSet<T>& in, const CgSet<T>& out, int nrhs, int step,
                           int x_updates, const CgCnt& cn, double rtol, hipStream_t st, int* nb_out) {
  ApplyArgs<T> A{};
  A.rho = rho;
  A.y = out.s;
  A.dinv = (const T*)vecs_of<T>(g).invD;
  A.step = step;
  A.xi = in.x; A.ri = in.r; A.pi = in.p; A.si = in.s;
  A.xo = out.x; A.ro = out.r; A.po = out.p;
  A.n_gam = cn.gam;
  A.n_apply = cn.apply;
  A.n_fn = cn.fn;
  A.rtol = rtol;
  // r.r only for the tolerance test
  if (g->n_springs > 0) {
    if (x_updates != 1) return hipErrorInvalidValue;
    return rtol > 0.0 ? launch_apply_mode<T, MODE_CGF, true, 3, 1>(g, A, nrhs, st, nb_out)
                      : launch_apply_mode<T, MODE_CGF, false, 3, 1>(g, A, nrhs, st, nb_out);
  }
  auto run = [&](auto xu) {
    constexpr int XU = decltype(xu)::value;
    return rtol > 0.0 ? launch_apply_mode<T, MODE_CGF, true, 1, XU>(g, A, nrhs, st, nb_out)
                      : launch_apply_mode<T, MODE_CGF, false, 1, XU>(g, A, nrhs, st, nb_out);
  };
  switch (x_updates) {
    case 0: return run(std::integral_constant<int, 0>{});
    case 1: return run(std::integral_constant<int, 1>{});
    default: return run(std::integral_constant<int, 2>{});
  }
}

template <typename T>
hipError_t launch_minres_fused(fbto_grid_s* g, const T* rho, int itn, const T* Y, const T* R1, const T* R2, T* R3,
                               T* W, T* W2, T* x, T* Ynext, int n_apply, int n_kr, double damp, int x_updates,
                               hipStream_t st, int* nb_out) {
  if (g->dim == 2) {
    if (x_updates != 1) return hipErrorInvalidValue;
    return plane_minres_fused<T>(g, rho, itn, Y, R1, R2, R3, W, W2, x, Ynext, n_apply, n_kr, damp, st, nb_out);
  }
  ApplyArgs<T> A{};
  A.rho = rho;
  A.y = Ynext;
  A.step = itn;
  A.mY = Y; A.mR1 = R1; A.mR2 = R2; A.mW = W;
  A.mR3 = R3; A.mW2 = W2; A.mx = x; A.mWo = W;
  A.n_apply = n_apply;
  A.n_kr = n_kr;
  A.damp = damp;
  switch (x_updates) {
    case 0: return launch_apply_mode<T, MODE_MRF, true, 1, 0>(g, A, 1, st, nb_out);
    case 1: return launch_apply_mode<T, MODE_MRF, true, 1, 1>(g, A, 1, st, nb_out);
    default: return launch_apply_mode<T, MODE_MRF, true, 1, 2>(g, A, 1, st, nb_out);
  }
}

// ===========================================================================
// Jacobi diagonal: D = ke_diag * sum_{e at node} s_e (+ springs), 1 on fixed
// DOFs; stores its inverse per DOF.  Every diagonal entry of the unit-cube
// hex8 KE is the same number, so one sum per node serves all 3 DOFs.
// ===========================================================================
template <typename T>
__global__ void __launch_bounds__(kVecBlock)
    k_diag(Geo G, const T* rho, T* invD, const uint8_t* mask, Simp sp, double ke_diag, int nspring,
           const int64_t* sdof, const T* sk) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= (int)G.N) return;
  const int row = fdiv(n, G.nxn, G.rnxn);
  const int i = n - row * G.nxn;
  const int k = fdiv(row, G.nyn, G.rnyn);
  const int j = row - k * G.nyn;
  T acc = (T)0;
#pragma unroll
  for (int dz = -1; dz <= 0; ++dz)
#pragma unroll
    for (int dy = -1; dy <= 0; ++dy)
#pragma unroll
      for (int dx = -1; dx <= 0; ++dx) {
        const int ex = i + dx, ey = j + dy, ez = k + dz;
        const bool ok = ex >= 0 && ex < G.nx && ey >= 0 && ey < G.ny && ez >= 0 && ez < G.nz;
        const T rv = rho[ok ? ex + G.nx * (ey + G.ny * ez) : 0];
        acc += ok ? simp_s<T>(rv, sp) : (T)0;
      }
  const unsigned m = mask[n];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    T d = (T)ke_diag * acc;
    for (int s = 0; s < nspring; ++s)
      if (sdof[s] == 3 * (int64_t)n + c) d += sk[s];
    if ((m >> c) & 1u) d = (T)1;
    invD[3 * n + c] = d > (T)0 ? (T)1 / d : (T)0;
  }
}

template <typename T>
hipError_t launch_diag(fbto_grid_s* g, const T* rho, T* invD, hipStream_t st) {
  if (g->dim == 2) return plane_diag<T>(g, rho, invD, st);
  hipLaunchKernelGGL((k_diag<T>), dim3(flat_grid(g->geo.N)), dim3(kVecBlock), 0, st, g->geo, rho, invD,
                     g->mask, g->simp, g->ke_diag, g->n_springs, g->spring_dof, spring_k_of<T>(g));
  return hipGetLastError();
}

// ===========================================================================
// Jacobi-PCG with one reduction phase per step.  With s = K p (whose product
// leaves the partials of delta = p.s and eps = s.D^-1 s) and gamma = r.z:
//   alpha = gamma / delta,  beta = (alpha^2 eps - gamma) / gamma,
//   x += alpha p,  r -= alpha s,  z = D^-1 r,  p = z + beta p
// (cg_coefficients).  In exact arithmetic the iterates are those of the
// textbook recurrence, and in floating point nearly so: s is the product
// itself, not a recurrence for it, so the residual follows f - K x as closely
// as the textbook's.  Against the recurrence of Chronopoulos and Gear
// (w = K z, s = w + beta s) a step carries one vector less (nine accesses
// instead of eleven).  beta's numerator is a difference of two sums, which loses
// digits where the residual falls fast; the error against FP64 is no larger for
// it (FP32 solves from zero to 24 steps on six grids, 8 to 16 inputs each: 0.94
// to 1.00 times that of the other recurrence, geometric means; whole outer
// iterations 0.92 to 1.06 times, within their spread).  The scalars are reduced
// from the partials in every block's prologue; convergence and breakdown are
// decided identically in every block.
// ===========================================================================

// One vector update, step k (plane grids; also the last step of a solve
// whose sensitivity is not fused).  LAST: x and the final residual norms
// only; r, p and z are not needed again.
template <typename T, int NR, bool LAST>
__global__ void __launch_bounds__(kVecBlock)
    k_cg_step(int64_t ndof, const T* x_in, T* x, T* r, const T* s, T* p, const T* invD, const T* f, double* P,
              int maxp, CgCnt cn, int step, double rtol, Scalars* sc) {
  // first chunk of this thread's vector entries is loaded before the prologue
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t i_first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  // entries per thread and chunk: fewer with more load cases, so that the
  // chunk stays in registers
  constexpr int kU = NR <= 2 ? 8 : 4;
  T sv[kU][NR], pv[kU][NR], xv[kU][NR], rv[kU][NR], dv[kU];
  bool ok[kU];
  auto load_chunk = [&](int64_t i0) {
#pragma unroll
    for (int k = 0; k < kU; ++k) {
      const int64_t i = i0 + k * stride;
      ok[k] = i < ndof;
      const int64_t ii = ok[k] ? i : 0;
      if constexpr (!LAST) dv[k] = invD[ii];
#pragma unroll
      for (int R = 0; R < NR; ++R) {
        const int64_t o = R * ndof + ii;
        rv[k][R] = r[o];
        sv[k][R] = s[o];
        xv[k][R] = x_in[o];
        pv[k][R] = p[o];
      }
    }
  };
  if (i_first < ndof) load_chunk(i_first);

  double pre[5 * NR];
  const int par = step & 1;
  {
    const double* src[5 * NR];
    int cnt[5 * NR];
    const bool tol = rtol > 0.0;  // r.r and f.f only for the tolerance test
#pragma unroll
    for (int R = 0; R < NR; ++R) {
      src[5 * R + 0] = pslot(P, P_RZ0 + par, R, maxp);
      src[5 * R + 1] = pslot(P, P_PQ0 + par, R, maxp);
      src[5 * R + 2] = pslot(P, P_EP0 + par, R, maxp);
      src[5 * R + 3] = pslot(P, P_RN0 + par, R, maxp);
      src[5 * R + 4] = pslot(P, P_FN, R, maxp);
      cnt[5 * R + 0] = cn.gam;
      cnt[5 * R + 1] = cn.apply;
      cnt[5 * R + 2] = cn.apply;
      cnt[5 * R + 3] = tol ? cn.gam : 0;
      cnt[5 * R + 4] = tol ? cn.fn : 0;
    }
    reduce_parts<5 * NR, 0u, kVecBlock>(pre, src, cnt);
  }
  T al[NR], be[NR];
  const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
#pragma unroll
  for (int R = 0; R < NR; ++R) {
    double alpha, beta;
    cg_coefficients(pre[5 * R], pre[5 * R + 1], pre[5 * R + 2], pre[5 * R + 3], pre[5 * R + 4], R, par, rtol, sc,
                    lead, alpha, beta);
    al[R] = (T)alpha;
    be[R] = (T)beta;
  }

  // LAST: r.r, max|r| per RHS, f.x; otherwise r.z, r.r per RHS
  double v[2 * NR + 1];
#pragma unroll
  for (int i = 0; i < 2 * NR + 1; ++i) v[i] = 0.0;
  for (int64_t i0 = i_first; i0 < ndof; i0 += kU * stride) {
    if (i0 != i_first) load_chunk(i0);
#pragma unroll
    for (int k = 0; k < kU; ++k) {
      if (!ok[k]) continue;
      const int64_t i = i0 + k * stride;
#pragma unroll
      for (int R = 0; R < NR; ++R) {
        const int64_t o = R * ndof + i;
        const T xn = xv[k][R] + al[R] * pv[k][R];
        const T rn = rv[k][R] - al[R] * sv[k][R];
        x[o] = xn;
        if constexpr (LAST) {
          v[2 * R] += (double)rn * (double)rn;
          v[2 * R + 1] = fmax(v[2 * R + 1], fabs((double)rn));
          if (f) v[2 * NR] += (double)f[o] * (double)xn;
        } else {
          const T zn = dv[k] * rn;
          r[o] = rn;
          p[o] = zn + be[R] * pv[k][R];
          v[2 * R] += (double)rn * (double)zn;
          v[2 * R + 1] += (double)rn * (double)rn;
        }
      }
    }
  }
  if constexpr (LAST) {
    double* dst[2 * NR + 1];
#pragma unroll
    for (int R = 0; R < NR; ++R) {
      dst[2 * R] = pslot(P, P_RNF, R, maxp);
      dst[2 * R + 1] = pslot(P, P_RIF, R, maxp);
    }
    dst[2 * NR] = pslot(P, P_DOT, 0, maxp);
    write_parts<2 * NR + 1, 0xAAAu, kVecBlock>(v, dst, blockIdx.x);
  } else {
    double w[2 * NR];
    double* dst[2 * NR];
#pragma unroll
    for (int R = 0; R < NR; ++R) {
      w[2 * R] = v[2 * R];
      w[2 * R + 1] = v[2 * R + 1];
      dst[2 * R] = pslot(P, P_RZ0 + (par ^ 1), R, maxp);
      dst[2 * R + 1] = pslot(P, P_RN0 + (par ^ 1), R, maxp);
    }
    write_parts<2 * NR, 0u, kVecBlock>(w, dst, blockIdx.x);
  }
}

// Threads of the one-block finishing kernels: a block of 256 measured twice
// as fast as one of 1024 for the few thousand partials they reduce (fewer
// waves meet at each barrier).
constexpr int kFinishThreads = 256;

// Reduce the final residual norms into the scalars (slots RNF, RIF with n_r
// partials, f.f from FN); with `info`, also write the outer-iteration record
// (compliance from DOT, projection results, gradient mean).
template <int NR>
__global__ void __launch_bounds__(kFinishThreads)
    k_pcg_finish(const double* P, int maxp, int n_r, int n_fn, Scalars* sc, double* info, int n_dot, int n_e,
                 int n_gsum, int64_t E) {
  double v[3 * NR + 4];
  const double* src[3 * NR + 4];
  int cnt[3 * NR + 4];
#pragma unroll
  for (int R = 0; R < NR; ++R) {
    src[3 * R + 0] = pslot(P, P_RNF, R, maxp);
    src[3 * R + 1] = pslot(P, P_RIF, R, maxp);
    src[3 * R + 2] = pslot(P, P_FN, R, maxp);
    cnt[3 * R + 0] = n_r;
    cnt[3 * R + 1] = n_r;
    cnt[3 * R + 2] = n_fn;
  }
  src[3 * NR + 0] = pslot(P, P_DOT, 0, maxp);
  src[3 * NR + 1] = pslot(P, P_VOL, 0, maxp);
  src[3 * NR + 2] = pslot(P, P_DX, 0, maxp);
  src[3 * NR + 3] = pslot(P, P_GSUM, 0, maxp);
  cnt[3 * NR + 0] = info ? n_dot : 0;
  cnt[3 * NR + 1] = info ? n_e : 0;
  cnt[3 * NR + 2] = info ? n_e : 0;
  cnt[3 * NR + 3] = info ? n_gsum : 0;
  // the scalars read by the lead thread are loaded before the reduction,
  // so their latency overlaps it
  double st_in[NR], proj_status = 0.0, lam = 0.0;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int R = 0; R < NR; ++R) st_in[R] = sc->status[R];
    proj_status = sc->proj_status;
    lam = sc->lam;
  }
  // max-reduced entries: |r|_inf of each RHS (3 R + 1, R < NR) and
  // |dx|_inf (3 NR + 2); the rest are sums
  constexpr unsigned MM = rinf_mask(NR) | (1u << (3 * NR + 2));
  reduce_parts<3 * NR + 4, MM, kFinishThreads>(v, src, cnt);
  if (threadIdx.x == 0) {
    double rinf = 0.0, rrel = 0.0, status = 0.0;
#pragma unroll
    for (int R = 0; R < NR; ++R) {
      const double rn = sqrt(v[3 * R]), fnrm = sqrt(v[3 * R + 2]);
      sc->rnorm2[R] = rn;
      sc->rinf[R] = v[3 * R + 1];
      sc->fnorm2[R] = fnrm;
      double stR = st_in[R];
      if (!isfinite(v[3 * R]) && stR == 0.0) {
        stR = (double)FBTO_ERR_NONFINITE;
        sc->status[R] = stR;
      }
      rinf = fmax(rinf, v[3 * R + 1]);
      rrel = fmax(rrel, fnrm > 0.0 ? rn / fnrm : rn);
      if (stR != 0.0) status = stR;
    }
    if (info) {
      // the projection's status: non-finite values take precedence, an
      // inexact projection (FBTO_INEXACT) only reports when the solve had none
      if (proj_status > 0.0 && (status == 0.0 || proj_status == (double)FBTO_ERR_NONFINITE)) status = proj_status;
      sc->dot[0] = v[3 * NR];
      info[FBTO_OI_COMPLIANCE] = v[3 * NR];
      info[FBTO_OI_DX_INF] = v[3 * NR + 2];
      info[FBTO_OI_R_INF] = rinf;
      info[FBTO_OI_LAMBDA] = lam;
      info[FBTO_OI_VOLUME] = v[3 * NR + 1];
      info[FBTO_OI_RREL] = rrel;
      info[FBTO_OI_STATUS] = status;
      info[FBTO_OI_GRAD_MEAN] = v[3 * NR + 3] / (double)E;
    }
  }
}

// The parts of two outer-iteration records that a filter-step launch writes (see
// OuterRec), by one block of kFinishThreads threads beside the filter's: the same
// sums as k_pcg_finish, whose launch of one block (4.4 us at the end of an
// iteration, with nothing beside it) is then left to a call's last iteration.
// Per iteration of a call of 20, FP32: 183.1 -> 179.6 us at 128x64x64, 112.2 ->
// 107.9 at 64x32x32, 78.6 -> 71.5 at 16x8x8.
constexpr int kRecVals = 7;
__device__ __forceinline__ void outer_record(const OuterRec& O, const double* P, int maxp, int n_gsum, Scalars* sc,
                                             int64_t E, double* lds) {
  double v[kRecVals];
  const double* src[kRecVals] = {pslot(P, P_RNF, 0, maxp), pslot(P, P_RIF, 0, maxp), pslot(P, P_FN, 0, maxp),
                          pslot(P, P_DOT, 0, maxp), pslot(P, P_VOL, 0, maxp), pslot(P, P_DX, 0, maxp),
                          pslot(P, P_GSUM, 0, maxp)};
  const int ns = O.solve ? 1 : 0, np = O.prev ? O.n_e : 0;
  const int cnt[kRecVals] = {ns * O.n_r, ns * O.n_r, ns * O.n_fn, ns * O.n_dot, np, np, ns * n_gsum};
  double st = 0.0, proj_status = 0.0, lam = 0.0, status = 0.0;
  if (threadIdx.x == 0) {
    st = sc->status[0];
    proj_status = sc->proj_status;
    lam = sc->lam;
    if (O.prev) status = O.prev[FBTO_OI_STATUS];
  }
  reduce_parts<kRecVals, 0x22u, kFinishThreads>(v, src, cnt, lds);
  if (threadIdx.x != 0) return;
  if (O.prev) {
    if (proj_status > 0.0 && (status == 0.0 || proj_status == (double)FBTO_ERR_NONFINITE)) status = proj_status;
    O.prev[FBTO_OI_DX_INF] = v[5];
    O.prev[FBTO_OI_LAMBDA] = lam;
    O.prev[FBTO_OI_VOLUME] = v[4];
    O.prev[FBTO_OI_STATUS] = status;
  }
  if (O.solve) {
    const double rn = sqrt(v[0]), fnrm = sqrt(v[2]);
    sc->rnorm2[0] = rn;
    sc->rinf[0] = v[1];
    sc->fnorm2[0] = fnrm;
    if (!isfinite(v[0]) && st == 0.0) {
      st = (double)FBTO_ERR_NONFINITE;
      sc->status[0] = st;
    }
    if (O.info) {
      sc->dot[0] = v[3];
      O.info[FBTO_OI_COMPLIANCE] = v[3];
      O.info[FBTO_OI_R_INF] = fmax(0.0, v[1]);
      O.info[FBTO_OI_RREL] = fmax(0.0, fnrm > 0.0 ? rn / fnrm : rn);
      O.info[FBTO_OI_STATUS] = st;
      O.info[FBTO_OI_GRAD_MEAN] = v[6] / (double)E;
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(kVecBlock)
    k_relax_update(int64_t ndof, int nrhs, T* u, const T* r, const T* invD, T omega, int use_diag) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ndof;
       i += (int64_t)gridDim.x * blockDim.x) {
    const T w = use_diag ? omega * invD[i] : omega;
    for (int R = 0; R < nrhs; ++R) u[R * ndof + i] += w * r[R * ndof + i];
  }
}

#define FBTO_NR_DISPATCH(nrhs, CALL) \
  switch (nrhs) {                    \
    case 1: { constexpr int NR = 1; CALL; break; } \
    case 2: { constexpr int NR = 2; CALL; break; } \
    case 3: { constexpr int NR = 3; CALL; break; } \
    default: { constexpr int NR = 4; CALL; break; } \
  }

template <typename T>
hipError_t launch_cg_step(fbto_grid_s* g, const T* x_in, T* x, T* r, const T* s, T* p, const T* invD, const T* f,
                          int nrhs, int step, bool last, const CgCnt& cn, double rtol, hipStream_t st,
                          int* nb_out) {
  const int nb = vec_blocks(g->geo.ndof);
  if (nb_out) *nb_out = nb;
  if (last) {
    FBTO_NR_DISPATCH(nrhs, hipLaunchKernelGGL((k_cg_step<T, NR, true>), dim3(nb), dim3(kVecBlock), 0, st, g->geo.ndof,
                                              x_in, x, r, s, p, invD, f, g->partials, g->max_partials, cn, step,
                                              rtol, g->sc));
  } else {
    FBTO_NR_DISPATCH(nrhs, hipLaunchKernelGGL((k_cg_step<T, NR, false>), dim3(nb), dim3(kVecBlock), 0, st,
                                              g->geo.ndof, x_in, x, r, s, p, invD, f, g->partials, g->max_partials,
                                              cn, step, rtol, g->sc));
  }
  return hipGetLastError();
}
hipError_t launch_pcg_finish(fbto_grid_s* g, int nrhs, int n_r, int n_fn, double* info, int n_dot, int n_e,
                             int n_gsum, hipStream_t st) {
  FBTO_NR_DISPATCH(nrhs, hipLaunchKernelGGL((k_pcg_finish<NR>), dim3(1), dim3(kFinishThreads), 0, st,
                                            (const double*)g->partials, g->max_partials, n_r, n_fn, g->sc, info,
                                            n_dot, n_e, n_gsum, g->geo.E));
  return hipGetLastError();
}
template <typename T>
hipError_t launch_relax_update(fbto_grid_s* g, T* u, const T* r, const T* invD, int nrhs,
                               double omega, int use_diag, hipStream_t st) {
  const int nb = vec_blocks(g->geo.ndof);
  hipLaunchKernelGGL((k_relax_update<T>), dim3(nb), dim3(kVecBlock), 0, st, g->geo.ndof, nrhs, u, r,
                     invD, (T)omega, use_diag);
  return hipGetLastError();
}

// ===========================================================================
// Krylov step of Alg. 3 (Eq. LSP, beta = 1): the new iterate minimises the
// residual over u + span{r, K r, ..., K^D r}.  It is computed by the MINRES
// recurrence (Lanczos vectors and Givens rotations, as in Paige and
// Saunders), D + 1 iterations from u.  Iteration itn (1 .. D + 1) is a product
// Y = K R2 (partials <R1, R2>, <Y, R2>) and a vector pass, which
//   - reduces beta = ||R2|| (the previous pass's partials) and, from the
//     product's partials, alpha = <v, K v - (beta/oldb) R1> with v = R2/beta;
//   - finishes iteration itn - 1: its Givens rotation needs beta, then
//     w = (v' - oldeps w'' - delta w') / gamma, x += damp * phi * w, where
//     v' = R1 / oldb is that iteration's Lanczos vector;
//   - forms the next Lanczos vector y = K v - (beta/oldb) R1 - (alpha/beta) R2
//     into R1's buffer and leaves ||y||^2 as partials.
// The first product (LZ mode) leaves ||R2||^2 of R2 = f - K u.  The vector passes
// of iterations 1 .. D are fused with the next product (k_apply's MRF mode,
// k_plane_minres); this kernel is that of iteration D + 1 and pass D + 2, which
// only finishes that iteration.  Every block runs the scalar recurrence on the same
// reduced values in the same order; block 0 keeps its state for the next
// pass.  The caller rotates the buffers: R1 <- R2, R2 <- the buffer y went
// to, W <- the buffer w went to (W2), W2 <- W.  `damp` scales the step
// (Alg. 3's beta_k).
// ===========================================================================
template <typename T>
__global__ void __launch_bounds__(kVecBlock)
    k_minres(int64_t n, int itn, int last, const T* Y, T* R1, const T* R2, T* W2, const T* W, T* x,
             double* P, int maxp, int n_apply, int n_prev, Scalars* sc, double damp) {
  double nv[1];
  {
    const double* src[1] = {pslot(P, P_KRN0 + ((itn - 1) & 1), 0, maxp)};
    const int cnt[1] = {n_prev};
    reduce_parts<1, 0u>(nv, src, cnt);
  }
  const double nrm2 = nv[0];
  const bool lanczos = itn < last;
  const bool finish = itn >= 2;
  double yr2 = 0.0, r12 = 0.0;
  if (lanczos) {
    double v[2];
    const double* src[2] = {pslot(P, P_RZ0 + (itn & 1), 0, maxp), pslot(P, P_PQ0 + (itn & 1), 0, maxp)};
    const int cnt[2] = {n_apply, n_apply};
    reduce_parts<2, 0u>(v, src, cnt);
    r12 = v[0];
    yr2 = v[1];
  }
  double ks[7];  // written by pass itn - 1
#pragma unroll
  for (int i = 0; i < 7; ++i) ks[i] = sc->kr[(itn + 1) & 1][i];
  const MinresCoef q =
      minres_scalars(itn, lanczos, nrm2, r12, yr2, ks, sc->kr[itn & 1], blockIdx.x == 0 && threadIdx.x == 0);
  const int j = itn - 1;  // the iteration finished here
  const T inv_oldb = (T)q.inv_oldb;
  const T wc1 = (T)q.wc1, wc2 = (T)q.wc2, inv_gamma = (T)q.inv_gamma;
  const T step = (T)(damp * q.phi);
  const T ts = (T)q.s, tc1 = (T)q.c1, ta = (T)q.as;
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const T r1 = R1[i];
    if (finish) {
      const T w1v = W[i], w2v = W2[i];  // w of iterations j - 1 and j - 2 (zero before the first)
      const T wp = j >= 2 ? w1v : (T)0, wpp = j >= 3 ? w2v : (T)0;
      const T wn = (r1 * inv_oldb - wc1 * wpp - wc2 * wp) * inv_gamma;
      W2[i] = wn;
      x[i] += step * wn;
    }
    if (lanczos) {
      const T r1m = itn >= 2 ? r1 : (T)0;  // R1 holds no vector yet on the first iteration
      const T yn = ts * Y[i] - tc1 * r1m - ta * R2[i];
      R1[i] = yn;
      acc += (double)yn * (double)yn;
    }
  }
  if (lanczos) {
    double v[1] = {acc};
    double* dst[1] = {pslot(P, P_KRN0 + (itn & 1), 0, maxp)};
    write_parts<1, 0u>(v, dst, blockIdx.x);
  }
}

template <typename T>
hipError_t launch_minres(fbto_grid_s* g, int itn, int last, const T* Y, T* R1, const T* R2, T* W2, const T* W,
                         T* x, int n_apply, int n_prev, double damp, hipStream_t st, int* nb_out) {
  const int nb = vec_blocks(g->geo.ndof);
  if (nb > g->max_partials || n_apply > g->max_partials) return hipErrorInvalidValue;
  if (nb_out) *nb_out = nb;
  hipLaunchKernelGGL((k_minres<T>), dim3(nb), dim3(kVecBlock), 0, st, g->geo.ndof, itn, last, Y, R1, R2, W2, W,
                     x, g->partials, g->max_partials, n_apply, n_prev, g->sc, damp);
  return hipGetLastError();
}

// ===========================================================================
// Sensitivity: dobj_e = -ds_e sum_r lam_{r,e}^T KE u_{r,e} (times 1/Hs_e when
// Hsi is given, which turns the filter transpose into a plain weighted sum),
// element strains recomputed from the nodal vectors.  A block owns 32 x 4 x 2
// elements, one per thread, and stages their 33 x 5 x 3 nodes in LDS, masked,
// all loads issued up front (the next load case's during the products of this
// one): 1.9 nodes read per element instead of the eight that a thread gathering
// its own element reads.  (Two elements per thread took 256 registers in FP64
// and were no faster than the gather.)
// ===========================================================================
constexpr int kSensX = 32, kSensY = 4, kSensZ = 2;
constexpr int kSensLX = kSensX + 1, kSensLY = kSensY + 1, kSensN = kSensLX * kSensLY * (kSensZ + 1);
constexpr int kSensTurns = (kSensN + kVecBlock - 1) / kVecBlock;
static_assert(kSensX * kSensY * kSensZ == kVecBlock, "one element per thread");
template <typename T>
struct Vec3 {
  T v[3];
};

template <typename T, bool LAM>
__global__ void __launch_bounds__(kVecBlock)
    k_sens(Geo G, const T* rho, const T* u, const T* lam, int nrhs, T* dobj, const uint8_t* mask, Modal<T> km,
           Simp sp, const T* Hsi) {
  using V3 = Vec3<T>;
  __shared__ T un[kSensN][3];
  __shared__ T ln[LAM ? kSensN : 1][3];
  const int tid = threadIdx.x, tx = tid % kSensX, ty = tid / kSensX % kSensY, tz = tid / (kSensX * kSensY);
  const int x0 = blockIdx.x * kSensX, y0 = blockIdx.y * kSensY, z0 = blockIdx.z * kSensZ;
  int node[kSensTurns];   // staged nodes of this thread (0 outside the grid: no element of the grid reads those)
  unsigned m[kSensTurns];
#pragma unroll
  for (int t = 0; t < kSensTurns; ++t) {
    const int i = tid + t * kVecBlock;
    const int row = i / kSensLX, lz = row / kSensLY;
    const int jx = x0 + i - row * kSensLX, jy = y0 + row - lz * kSensLY, jz = z0 + lz;
    node[t] = (i < kSensN && jx <= G.nx && jy <= G.ny && jz <= G.nz) ? jx + G.nxn * (jy + G.nyn * jz) : 0;
    m[t] = mask[node[t]];
  }
  V3 uv[kSensTurns], lv[LAM ? kSensTurns : 1];
  auto load = [&](int R) {
#pragma unroll
    for (int t = 0; t < kSensTurns; ++t) {
      const int64_t o = R * G.ndof + 3 * (int64_t)node[t];
      uv[t] = *reinterpret_cast<const V3*>(u + o);
      if constexpr (LAM) lv[t] = *reinterpret_cast<const V3*>(lam + o);
    }
  };
  load(0);
  const int ex = x0 + tx, ey = y0 + ty, ez = z0 + tz;
  const bool el = ex < G.nx && ey < G.ny && ez < G.nz;
  const int e = el ? ex + G.nx * (ey + G.ny * ez) : 0;
  const T rv = rho[e];
  const T hv = Hsi ? Hsi[e] : (T)1;
  double acc = 0.0;
  for (int R = 0; R < nrhs; ++R) {
    if (R > 0) __syncthreads();  // the last case's products have read the LDS
#pragma unroll
    for (int t = 0; t < kSensTurns; ++t) {
      const int i = tid + t * kVecBlock;
      if (i < kSensN) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          un[i][c] = zmasked(m[t], c, uv[t].v[c]);
          if constexpr (LAM) ln[i][c] = zmasked(m[t], c, lv[t].v[c]);
        }
      }
    }
    __syncthreads();
    if (R + 1 < nrhs) load(R + 1);
    T ue[8][3], le[8][3];
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      const int i = tx + (a & 1) + kSensLX * (ty + ((a >> 1) & 1) + kSensLY * (tz + (a >> 2)));
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        ue[a][c] = un[i][c];
        if constexpr (LAM) le[a][c] = ln[i][c];
      }
    }
    if constexpr (LAM) acc += elem_bilinear<T>(le, ue, km);
    else acc += elem_bilinear<T>(ue, ue, km);
  }
  if (!el) return;
  double val = -(double)simp_ds<T>(rv, sp) * acc;
  if (Hsi) val *= (double)hv;
  dobj[e] = (T)val;
}

// The same for grids that fill few of the tiles' elements (see sens_staged): one
// element per thread in the order of their numbers, its eight nodes gathered
// through the caches.  No thread is idle on any grid, but a node is read eight
// times.  Same operations in the same order as k_sens.  In FP64 lam is tested
// once more, which it always passes: the branch keeps its loads behind u's share
// of the product (2x1024x1024 47 us, without the branch 55; FP32 33.0 and 32.3).
template <typename T>
__device__ __forceinline__ void gather_elem(const Geo& G, const T* v, const uint8_t* mask, int ex, int ey, int ez,
                                            T (&ue)[8][3]) {
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    const int n = ex + (a & 1) + G.nxn * (ey + ((a >> 1) & 1) + G.nyn * (ez + (a >> 2)));
    const unsigned m = mask[n];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const T x = v[3 * n + c];  // 3 N < 2^31
      ue[a][c] = ((m >> c) & 1u) ? (T)0 : x;
    }
  }
}
template <typename T, bool LAM>
__global__ void __launch_bounds__(kVecBlock)
    k_sens_gather(Geo G, const T* rho, const T* u, const T* lam, int nrhs, T* dobj, const uint8_t* mask, Modal<T> km,
                  Simp sp, const T* Hsi) {
  const int e = blockIdx.x * kVecBlock + threadIdx.x;
  if (e >= (int)G.E) return;
  const int row = fdiv(e, G.nx, G.rnx);
  const int ex = e - row * G.nx;
  const int ez = fdiv(row, G.ny, G.rny);
  const int ey = row - ez * G.ny;
  double acc = 0.0;
  for (int R = 0; R < nrhs; ++R) {
    T ue[8][3];
    gather_elem<T>(G, u + R * G.ndof, mask, ex, ey, ez, ue);
    if (LAM && (sizeof(T) == 4 || lam)) {
      T le[8][3];
      gather_elem<T>(G, lam + R * G.ndof, mask, ex, ey, ez, le);
      acc += elem_bilinear<T>(le, ue, km);
    } else {
      acc += elem_bilinear<T>(ue, ue, km);
    }
  }
  double val = -(double)simp_ds<T>(rho[e], sp) * acc;
  if (Hsi) val *= (double)Hsi[e];
  dobj[e] = (T)val;
}

// Share of the LDS tiles that a grid's elements have to fill for the staged
// kernel to be chosen: below it, its idle threads cost more than the repeated
// reads.  Staged against gathered on 2.2M elements, FP32, FP64, FP32 with lam, FP64
// with lam: all of the tiles filled (1024x1024x2) 0.83, 0.61, 0.65, 0.62 of the
// time; 0.87 to 0.93 of them (56, 60 x N^2, 30x270x270) 1.05-0.97, 0.86-0.74,
// 0.79-0.74, 0.89-0.75; 0.69 to 0.74 (22, 24, 48 x N^2) 1.22-1.16, 0.93-0.90,
// 0.94-0.88, 0.98-0.94; 0.62 (20x330x330) 1.32, 1.03, 1.01, 1.09; 0.56 (18, 36 x
// N^2) 1.46, 1.11, 1.12, 1.17; 1/32 (1x1483x1483) 19, 14, 16, 13.
template <typename T, bool LAM>
static bool sens_staged(const Geo& G, const dim3& grid) {
  constexpr double min_fill = sizeof(T) == 4 ? (LAM ? 0.72 : 0.9) : (LAM ? 0.68 : 0.72);
  return (double)G.E >= min_fill * kVecBlock * ((double)grid.x * grid.y * grid.z);
}

template <typename T, bool LAM>
static void run_sens(fbto_grid_s* g, const T* rho, const T* u, const T* lam, int nrhs, T* dobj, const T* Hsi,
                     hipStream_t st) {
  const Geo& G = g->geo;
  // axes of at most 65,534 elements: within the limits of a grid
  const dim3 grid((G.nx + kSensX - 1) / kSensX, (G.ny + kSensY - 1) / kSensY, (G.nz + kSensZ - 1) / kSensZ);
  if (sens_staged<T, LAM>(G, grid))
    hipLaunchKernelGGL((k_sens<T, LAM>), grid, dim3(kVecBlock), 0, st, G, rho, u, lam, nrhs, dobj, g->mask,
                       modal_of<T>(g), g->simp, Hsi);
  else
    hipLaunchKernelGGL((k_sens_gather<T, LAM>), dim3((G.E + kVecBlock - 1) / kVecBlock), dim3(kVecBlock), 0, st, G,
                       rho, u, lam, nrhs, dobj, g->mask, modal_of<T>(g), g->simp, Hsi);
}

template <typename T>
hipError_t launch_sens(fbto_grid_s* g, const T* rho, const T* u, const T* lam, int nrhs, T* dobj,
                       const T* Hsi, hipStream_t st) {
  if (g->dim == 2) return plane_sens<T>(g, rho, u, lam, nrhs, dobj, Hsi, st);
  if (lam) run_sens<T, true>(g, rho, u, lam, nrhs, dobj, Hsi, st);
  else run_sens<T, false>(g, rho, u, lam, nrhs, dobj, Hsi, st);
  return hipGetLastError();
}

// partials of sum_r a_r . b_r (vectors of length ndof) into slot DOT
template <typename T>
__global__ void __launch_bounds__(kVecBlock)
    k_dot(int64_t n, int nrhs, const T* a, const T* b, double* P, int maxp) {
  double v[1] = {0.0};
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    for (int R = 0; R < nrhs; ++R) v[0] += (double)a[R * n + i] * (double)b[R * n + i];
  }
  double* dst[1] = {pslot(P, P_DOT, 0, maxp)};
  write_parts<1, 0u>(v, dst, blockIdx.x);
}

__global__ void __launch_bounds__(kVecBlock) k_dot_store(const double* P, int maxp, int nb, double* out) {
  double v[1];
  const double* src[1] = {pslot(P, P_DOT, 0, maxp)};
  const int cnt[1] = {nb};
  reduce_parts<1, 0u>(v, src, cnt);
  if (threadIdx.x == 0) out[0] = v[0];
}

template <typename T>
hipError_t launch_dot(fbto_grid_s* g, const T* a, const T* b, int nrhs, hipStream_t st) {
  const int nb = vec_blocks(g->geo.ndof);
  hipLaunchKernelGGL((k_dot<T>), dim3(nb), dim3(kVecBlock), 0, st, g->geo.ndof, nrhs, a, b, g->partials,
                     g->max_partials);
  return hipGetLastError();
}
hipError_t launch_dot_store(fbto_grid_s* g, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_dot_store, dim3(1), dim3(kVecBlock), 0, st, (const double*)g->partials,
                     g->max_partials, vec_blocks(g->geo.ndof), out);
  return hipGetLastError();
}

// ===========================================================================
// Linear cone filter: gather over the stencil (offsets with r - |d| > 0).
//   FWD:    out_e = sum_o w_o in_{e+o} / Hs_e
//   TRANS:  out_j = sum_o w_o in_{j+o} / Hs_{j+o}
//   SUM:    out_j = sum_o w_o in_{j+o}      (input already divided by Hs)
// One element per thread; want_sum: partials of sum(out) into slot GSUM.
// ===========================================================================
enum { FILT_FWD = 0, FILT_TRANS = 1, FILT_SUM = 2 };

template <typename T, int R>
struct StencilW {
  T w[(2 * R + 1) * (2 * R + 1) * (2 * R + 1)];   // weight of offset (dx, dy, dz), x fastest
};

template <typename T, int R>
__global__ void __launch_bounds__(kVecBlock)
    k_filter(Geo G, int kind, const T* in, T* out, const T* Hsi, StencilW<T, R> W, int want_sum,
             double* P, int maxp) {
  constexpr int D = 2 * R + 1;
  double v[1] = {0.0};
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < (int)G.E; e += gridDim.x * blockDim.x) {
    const int row = fdiv(e, G.nx, G.rnx);
    const int ex = e - row * G.nx;
    const int ez = fdiv(row, G.ny, G.rny);
    const int ey = row - ez * G.ny;
    T acc = (T)0;
#pragma unroll
    for (int dz = -R; dz <= R; ++dz)
#pragma unroll
      for (int dy = -R; dy <= R; ++dy)
#pragma unroll
        for (int dx = -R; dx <= R; ++dx) {
          const int jx = ex + dx, jy = ey + dy, jz = ez + dz;
          const bool ok = jx >= 0 && jx < G.nx && jy >= 0 && jy < G.ny && jz >= 0 && jz < G.nz;
          const int j = ok ? e + dx + G.nx * (dy + G.ny * dz) : e;
          const T wv = ok ? W.w[(dx + R) + D * ((dy + R) + D * (dz + R))] : (T)0;
          const T x = kind == FILT_TRANS ? in[j] * Hsi[j] : in[j];
          acc += wv * x;
        }
    const T res = kind == FILT_FWD ? acc * Hsi[e] : acc;
    out[e] = res;
    v[0] += (double)res;
  }
  if (want_sum) {
    double* dst[1] = {pslot(P, P_GSUM, 0, maxp)};
    write_parts<1, 0u>(v, dst, blockIdx.x);
  }
}

// The evaluation of one search pass at lam for one entry: f(lam) and the linear
// piece of f just right (+) and just left (-) of lam, f(l) = C - l nA (an
// entry adds its bound to C where it is clamped, else its value to C and one
// to nA), plus the nearest breakpoints on either side:
//   v = {f, nA+, C+, nA-, C-, max breakpoint below lam, -(min above)}.
// (Written with selects only: branches here let the compiler pick the last two
// by a dynamic index, which puts the array in scratch memory.)
constexpr int kEval = kProjEval;
constexpr unsigned kEvalMax = 0x60u;  // the max-reduced entries
static_assert(kEval == 7, "entries of an evaluation");
__device__ __forceinline__ void proj_eval(double (&v)[kEval], double yd, double lam, double lo, double hi) {
  const double t = yd - lam;
  v[0] += fmin(fmax(t, lo), hi);
  const bool rU = t > hi, rL = !rU && t <= lo, rA = !rU && !rL;   // just right of lambda
  v[1] += rA ? 1.0 : 0.0;
  v[2] += rU ? hi : (rL ? lo : yd);
  const bool lU = t >= hi, lL = !lU && t < lo, lA = !lU && !lL;   // just left of lambda
  v[3] += lA ? 1.0 : 0.0;
  v[4] += lU ? hi : (lL ? lo : yd);
  const double b1 = yd - lo, b2 = yd - hi;
  v[5] = fmax(v[5], fmax(b1 < lam ? b1 : -INFINITY, b2 < lam ? b2 : -INFINITY));
  v[6] = fmax(v[6], fmax(b1 > lam ? -b1 : -INFINITY, b2 > lam ? -b2 : -INFINITY));
}
__device__ __forceinline__ void proj_eval_init(double (&v)[kEval]) {
#pragma unroll
  for (int i = 0; i < kEval; ++i) v[i] = (kEvalMax >> i) & 1u ? -INFINITY : 0.0;
}

// The step's partials of one block in one reduction: the projection's seed
// (sum clamp(y), max y, #interior: slots S0, YMAX, NACT) and the evaluation
// at the warm-start multiplier (evaluation set 0, the next slots).
static_assert(P_YMAX == P_S0 + 1 && P_NACT == P_S0 + 2 && P_E0 == P_S0 + 3, "seed and set 0 are consecutive slots");
constexpr unsigned kSeedEvalMax = 0x2u | (kEvalMax << 3);  // max y, and the evaluation's
template <int NTHR>
__device__ __forceinline__ void step_parts(double (&v3)[3], double (&ev)[kEval], double* P, int maxp, int block,
                                           double* lds) {
  double w[3 + kEval];
  double* dst[3 + kEval];
#pragma unroll
  for (int i = 0; i < 3 + kEval; ++i) {
    w[i] = i < 3 ? v3[i] : ev[i - 3];
    dst[i] = pslot(P, P_S0 + i, 0, maxp);
  }
  write_parts<3 + kEval, kSeedEvalMax, NTHR>(w, dst, block, lds);
}

// Density filter for R <= 1: a block owns 64 x 4 element columns and four
// layers and stages them with their halo in LDS, every load issued up front
// (one memory latency per block, 2.3 loads per output); a thread then sums the
// windows of its column's four outputs.  Read by each thread from memory, the
// window took 13.5 loads per output (27 transposed, with Hsi), and the final
// projection pass clamped each of them.  Out-of-grid neighbours are 0 (the
// stencil is truncated at the boundary).
constexpr int kFiltBX = 64, kFiltBY = 4, kFiltDZ = 4;

// The gradient step fused into the plain-sum filter (the transposed filter
// after the 1/Hs fold): each filtered value g_e gives y_e = x_e -
// half_alpha (g_e - mean), with the projection's seed and its evaluation at
// the warm-start multiplier, as k_step forms them.  The mean comes from the
// partials in slot GSUM (the sensitivity kernel's sum of the unfiltered
// gradient, equal to the filtered one's since the weights are symmetric).
template <typename T>
struct FiltStep {
  const T* x;
  T* y;
  double half_alpha;
  int mean_project, nb_sum;
  double lo, hi;
  Scalars* sc;
  int rec_on;  // the first layer of blocks writes `rec`
  OuterRec rec;
};

// Thread geometry of the filter: a tile of 64 x 4 element columns
// and kFiltDZ layers; the thread's column (ex, ey) and output layers
// [z0, z1).
struct FiltPos {
  int block;           // number of the block's partials
  int tx, ty, x0, y0;  // thread in the tile, the tile's first column
  int ex, ey, z0, z1;
  bool col;  // the column lies in the grid
};
__device__ __forceinline__ FiltPos filt_pos(const Geo& G, int bz) {
  FiltPos q;
  const int tx = threadIdx.x % kFiltBX, ty = threadIdx.x / kFiltBX;
  const int bx = blockIdx.x, by = blockIdx.y;
  q.block = bx + gridDim.x * (by + gridDim.y * bz);
  q.tx = tx;
  q.ty = ty;
  q.x0 = bx * kFiltBX;
  q.y0 = by * kFiltBY;
  q.ex = q.x0 + tx;
  q.ey = q.y0 + ty;
  q.z0 = bz * kFiltDZ;
  q.z1 = min(q.z0 + kFiltDZ, G.nz);
  q.col = q.ex < G.nx && q.ey < G.ny;
  return q;
}

// The values a block stages: its columns and layers with R more on each side,
// kN of them in threads' turns of one, x fastest.
template <int R>
struct FiltStage {
  static constexpr int LX = kFiltBX + 2 * R, LY = kFiltBY + 2 * R, LZ = kFiltDZ + 2 * R;
  static constexpr int kThreads = kFiltBX * kFiltBY, kN = LX * LY * LZ, kTurns = (kN + kThreads - 1) / kThreads;
  static constexpr int kLds = R > 0 ? kN : 1;  // values in LDS (none without neighbours)
};
static_assert(FiltStage<0>::kTurns == kFiltDZ, "without a halo, turn l is the thread's own output of layer l");
// Issues the thread's loads (trans: times Hsi); bit t of ok: turn t lies in
// the grid.  Out-of-grid values are 0.  Without neighbours (R = 0) turn t is the
// thread's own output of layer t.
template <typename T, int R>
__device__ __forceinline__ void filt_load(const Geo& G, const FiltPos& q, const T* in, const T* Hsi, bool trans,
                                          T (&v)[FiltStage<R>::kTurns], unsigned& ok) {
  using S = FiltStage<R>;
  ok = 0u;
  if constexpr (R == 0) {  // the thread's own column; the products after all loads
    const int plane = G.nx * G.ny, col = q.col ? q.ex + G.nx * q.ey : 0;
    T h[kFiltDZ];
#pragma unroll
    for (int t = 0; t < kFiltDZ; ++t) {
      const bool in_grid = q.col && q.z0 + t < G.nz;
      const int j = in_grid ? col + (q.z0 + t) * plane : 0;
      const T x = in[j];
      h[t] = trans ? Hsi[j] : (T)1;
      v[t] = in_grid ? x : (T)0;
      ok |= in_grid ? 1u << t : 0u;
    }
    if (trans)
#pragma unroll
      for (int t = 0; t < kFiltDZ; ++t) v[t] *= h[t];
  } else {
#pragma unroll
    for (int t = 0; t < S::kTurns; ++t) {
      const int i = (int)threadIdx.x + t * S::kThreads;
      const int row = i / S::LX, lz = row / S::LY;
      const int jx = q.x0 - R + i - row * S::LX, jy = q.y0 - R + row - lz * S::LY, jz = q.z0 - R + lz;
      const bool in_grid = i < S::kN && jx >= 0 && jx < G.nx && jy >= 0 && jy < G.ny && jz >= 0 && jz < G.nz;
      const int j = in_grid ? jx + G.nx * (jy + G.ny * jz) : 0;
      T x = in[j];
      if (trans) x *= Hsi[j];
      v[t] = in_grid ? x : (T)0;
      ok |= in_grid ? 1u << t : 0u;
    }
  }
}

// The window of the thread's outputs, kFiltDZ layers and R more on each side of
// its (2R + 1)^2 columns, from the values the block's threads loaded, exchanged
// through LDS.  Without neighbours (R = 0) a thread has loaded its own: numbered
// and exchanged all the same, the identity filter took 12.1 instead of 10.1 us at
// 1000x2000x1 FP64, transposed 16.3 instead of 11.3, and 17.3 instead of 15.8 at
// 256x128x128.
template <typename T, int R>
__device__ __forceinline__ void filt_window(const T (&v)[FiltStage<R>::kTurns], T* sh, const FiltPos& q,
                                            T (&win)[kFiltDZ + 2 * R][2 * R + 1][2 * R + 1]) {
  using S = FiltStage<R>;
  if constexpr (R == 0) {
#pragma unroll
    for (int l = 0; l < kFiltDZ; ++l) win[l][0][0] = v[l];
  } else {
#pragma unroll
    for (int t = 0; t < S::kTurns; ++t) {
      const int i = (int)threadIdx.x + t * S::kThreads;
      if (i < S::kN) sh[i] = v[t];
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < S::LZ; ++p)
#pragma unroll
      for (int dy = 0; dy < 2 * R + 1; ++dy)
#pragma unroll
        for (int dx = 0; dx < 2 * R + 1; ++dx) win[p][dy][dx] = sh[q.tx + dx + S::LX * (q.ty + dy + S::LY * p)];
  }
}

// The stencil sum of output layer l of the window.
template <typename T, int R>
__device__ __forceinline__ T filt_sum(const StencilW<T, R>& W, const T (&win)[kFiltDZ + 2 * R][2 * R + 1][2 * R + 1],
                                      int l) {
  constexpr int D = 2 * R + 1;
  T acc = (T)0;
#pragma unroll
  for (int dz = 0; dz < D; ++dz)
#pragma unroll
    for (int dy = 0; dy < D; ++dy)
#pragma unroll
      for (int dx = 0; dx < D; ++dx) acc += W.w[dx + D * (dy + D * dz)] * win[l + dz][dy][dx];
  return acc;
}

template <typename T, int R, bool STEP>
__global__ void __launch_bounds__(kFiltBX * kFiltBY)
    k_filter_z(Geo G, int kind, const T* in, T* out, const T* Hsi, StencilW<T, R> W, int want_sum,
               double* P, int maxp, FiltStep<T> S) {
  // The staged values and, in the step, every reduction share one LDS array:
  // the record's block uses nothing else, the mean's reduction lies behind the
  // staged values, the final one on top of both after a barrier.  With an array
  // each the step took 46.5 KB (FP32; FP64 56.0) where it now takes 20.6 (21.1),
  // and a SIMD held 3 (2) of its waves instead of 5 (3): at 256x128x128 41.0
  // (56.7) us instead of 34.7 (47.0), also in calls without records.
  constexpr int kThreads = kFiltBX * kFiltBY;
  constexpr int kStaged = (int)((FiltStage<R>::kLds * sizeof(T) + sizeof(double) - 1) / sizeof(double));
  constexpr int kMean = reduce_lds_words<1, kThreads>();
  constexpr int kWords = STEP ? std::max({kStaged + kMean, reduce_lds_words<3 + kEval, kThreads>(),
                                          reduce_lds_words<kRecVals, kThreads>()})
                              : kStaged;
  __shared__ double lds[kWords];
  int bz = blockIdx.z;
  if constexpr (STEP) {
    if (S.rec_on) {
      if (bz == 0) {
        if (blockIdx.x == 0 && blockIdx.y == 0) outer_record(S.rec, P, maxp, S.nb_sum, S.sc, G.E, lds);
        return;
      }
      --bz;
    }
  }
  const FiltPos q = filt_pos(G, bz);
  T* const sh = reinterpret_cast<T*>(lds);
  T sv[FiltStage<R>::kTurns];
  unsigned ok;
  filt_load<T, R>(G, q, in, Hsi, kind == FILT_TRANS, sv, ok);
  // step: the design values of the slab's outputs, and the mean of g
  T xv[kFiltDZ];
  double mean = 0.0, lam_w = 0.0;
  if constexpr (STEP) {
#pragma unroll
    for (int l = 0; l < kFiltDZ; ++l) {
      const int ez = q.z0 + l;
      xv[l] = S.x[(q.col && ez < q.z1) ? q.ex + G.nx * (q.ey + G.ny * ez) : 0];
    }
    lam_w = S.sc->lam_prev;
    if (S.mean_project) {
      double v[1];
      const double* src[1] = {pslot(P, P_GSUM, 0, maxp)};
      const int cnt[1] = {S.nb_sum};
      reduce_parts<1, 0u, kThreads>(v, src, cnt, lds + kStaged);
      mean = v[0] / (double)G.E;
    }
  }
  T hs[kFiltDZ];  // forward: 1/Hs of the outputs (without neighbours read where it is used)
  if (R > 0 && !STEP && kind == FILT_FWD) {
#pragma unroll
    for (int l = 0; l < kFiltDZ; ++l) {
      const int ez = q.z0 + l;
      hs[l] = Hsi[(q.col && ez < q.z1) ? q.ex + G.nx * (q.ey + G.ny * ez) : 0];
    }
  }
  T win[kFiltDZ + 2 * R][2 * R + 1][2 * R + 1];  // [plane][dy][dx]
  filt_window<T, R>(sv, sh, q, win);
  double vs[1] = {0.0};
  double v3[3] = {0.0, -INFINITY, 0.0};  // step: sum clamp(y), max y, #interior
  double ev[kEval];                      // step: evaluation at lam_w
  proj_eval_init(ev);
#pragma unroll
  for (int l = 0; l < kFiltDZ; ++l) {
    const int ez = q.z0 + l;
    const T acc = filt_sum<T, R>(W, win, l);
    if (q.col && ez < q.z1) {
      const int e = q.ex + G.nx * (q.ey + G.ny * ez);
      const T res = !STEP && kind == FILT_FWD ? acc * (R > 0 ? hs[l] : Hsi[e]) : acc;
      if constexpr (STEP) {
        const T ye = (T)((double)xv[l] - S.half_alpha * ((double)res - mean));
        S.y[e] = ye;
        const double yd = (double)ye;
        v3[0] += fmin(fmax(yd, S.lo), S.hi);
        v3[1] = fmax(v3[1], yd);
        v3[2] += (yd > S.lo && yd < S.hi) ? 1.0 : 0.0;
        proj_eval(ev, yd, lam_w, S.lo, S.hi);
      } else {
        out[e] = res;
        vs[0] += (double)res;
      }
    }
  }
  if constexpr (STEP) {
    __syncthreads();  // every window is read
    step_parts<kThreads>(v3, ev, P, maxp, q.block, lds);
  } else if (want_sum) {
    double* dst[1] = {pslot(P, P_GSUM, 0, maxp)};
    write_parts<1, 0u>(vs, dst, q.block);
  }
}

// Density filter for R = 2 (radius 2 to 3) by z-march: a block owns a BX x
// (256 / BX) tile of element columns and a slab of layers.  Each plane the slab
// reads is staged in LDS once, with the tile's halo of two columns on every
// side (its loads issued one plane ahead), and a thread adds the plane's
// 21 or 25 neighbours of its column to the five outputs they reach, so a value
// is read from memory (BX + 4) (BY + 4) / 256 (dz + 4) / dz times instead of
// 125 times through the L1, which bound the gather.  The taps with
// |offset|^2 >= 9 have no weight at any radius up to 3 and are left out; the
// others are taken in the gather's order (dz, dy, dx).  Bound by its 93 FMAs
// per element on large grids (68 us at 384x192x192 FP32, 170 MB at 2.5 TB/s)
// and by the latency of its planes on small ones.  Gather -> this, FP32
// forward / transpose: 384x192x192 1158 / 2641 -> 68 / 90 us, 256x128x128
// 354 / 769 -> 29 / 43 us, 97x53x41 26 / 41 -> 9.0 / 9.4 us; FP64 at
// 384x192x192 2344 / 4674 -> 123 / 170 us.
constexpr int kFilt2Halo = 2;
template <typename T>
struct Stencil2 {
  T w[9];  // weight by squared offset
};

template <typename T, int BX>
__global__ void __launch_bounds__(kVecBlock)
    k_filter_r2(Geo G, int kind, const T* in, T* out, const T* Hsi, Stencil2<T> W, int want_sum, double* P, int maxp,
                int tiles_x, int tiles_y, int dz, int nwork) {
  constexpr int H = kFilt2Halo, BY = kVecBlock / BX;
  constexpr int LX = BX + 2 * H, LY = BY + 2 * H, LN = LX * LY;
  constexpr int NL = (LN + kVecBlock - 1) / kVecBlock;  // values a thread stages per plane
  __shared__ T sh[2][LN];
  const int tid = threadIdx.x, tx = tid % BX, ty = tid / BX;
  const int plane = G.nx * G.ny;
  double v[1] = {0.0};
  for (int wk = blockIdx.x; wk < nwork; wk += gridDim.x) {
    const int bx = wk % tiles_x, t2 = wk / tiles_x, by = t2 % tiles_y, bz = t2 / tiles_y;
    const int x0 = bx * BX, y0 = by * BY, z0 = bz * dz, z1 = min(z0 + dz, G.nz);
    int col[NL];  // offset of each staged column in its plane, -1 outside the grid
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int i = tid + k * kVecBlock;
      const int gx = x0 + i % LX - H, gy = y0 + i / LX - H;
      col[k] = (i < LN && gx >= 0 && gx < G.nx && gy >= 0 && gy < G.ny) ? gx + G.nx * gy : -1;
    }
    auto load = [&](int z, T (&q)[NL]) {
      const bool zok = z >= 0 && z < G.nz && z < z1 + H;
#pragma unroll
      for (int k = 0; k < NL; ++k) {
        const bool ok = zok && col[k] >= 0;
        const int64_t j = ok ? col[k] + (int64_t)z * plane : 0;
        T x = in[j];
        if (kind == FILT_TRANS) x *= Hsi[j];
        q[k] = ok ? x : (T)0;
      }
    };
    const bool own = x0 + tx < G.nx && y0 + ty < G.ny;
    const int ecol = x0 + tx + G.nx * (y0 + ty);
    T acc[2 * H + 1];  // outputs z - 2 .. z + 2 of the current plane z
#pragma unroll
    for (int i = 0; i < 2 * H + 1; ++i) acc[i] = (T)0;
    T q[NL];
    load(z0 - H, q);
    for (int z = z0 - H; z < z1 + H; ++z) {
      T* const b = sh[z & 1];
#pragma unroll
      for (int k = 0; k < NL; ++k)
        if (tid + k * kVecBlock < LN) b[tid + k * kVecBlock] = q[k];
      load(z + 1, q);
      T hs = (T)1;
      const int zo = z - H;  // the output this plane completes
      const bool emit = own && zo >= z0;
      const int64_t e = emit ? ecol + (int64_t)zo * plane : 0;
      if (kind == FILT_FWD) hs = Hsi[e];
      __syncthreads();
#pragma unroll
      for (int dy = -H; dy <= H; ++dy)
#pragma unroll
        for (int dx = -H; dx <= H; ++dx) {
          const T x = b[(ty + H + dy) * LX + tx + H + dx];
#pragma unroll
          for (int d = -H; d <= H; ++d) {
            constexpr int kMax = 8;
            const int d2 = dx * dx + dy * dy + d * d;
            if (d2 <= kMax) acc[H - d] += W.w[d2] * x;
          }
        }
      if (emit) {
        const T res = kind == FILT_FWD ? acc[0] * hs : acc[0];
        out[e] = res;
        v[0] += (double)res;
      }
#pragma unroll
      for (int i = 0; i < 2 * H; ++i) acc[i] = acc[i + 1];
      acc[2 * H] = (T)0;
    }
    __syncthreads();  // the next tile restages the buffers
  }
  if (want_sum) {
    double* dst[1] = {pslot(P, P_GSUM, 0, maxp)};
    write_parts<1, 0u, kVecBlock>(v, dst, blockIdx.x);
  }
}

// Generic gather for wide stencils (R > 2): offsets and weights from memory.
template <typename T>
__global__ void __launch_bounds__(kVecBlock)
    k_filter_wide(Geo G, int kind, const T* in, T* out, const T* Hsi, int nst, const int* off,
                  const T* w, int want_sum, double* P, int maxp) {
  double v[1] = {0.0};
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < (int)G.E; e += gridDim.x * blockDim.x) {
    const int row = fdiv(e, G.nx, G.rnx);
    const int ex = e - row * G.nx;
    const int ez = fdiv(row, G.ny, G.rny);
    const int ey = row - ez * G.ny;
    T acc = (T)0;
    for (int o = 0; o < nst; ++o) {
      const int jx = ex + off[3 * o], jy = ey + off[3 * o + 1], jz = ez + off[3 * o + 2];
      if (jx < 0 || jx >= G.nx || jy < 0 || jy >= G.ny || jz < 0 || jz >= G.nz) continue;
      const int j = jx + G.nx * (jy + G.ny * jz);
      acc += w[o] * (kind == FILT_TRANS ? in[j] * Hsi[j] : in[j]);
    }
    const T res = kind == FILT_FWD ? acc * Hsi[e] : acc;
    out[e] = res;
    v[0] += (double)res;
  }
  if (want_sum) {
    double* dst[1] = {pslot(P, P_GSUM, 0, maxp)};
    write_parts<1, 0u>(v, dst, blockIdx.x);
  }
}

template <typename T>
__global__ void k_hs(Geo G, T* Hsi, int nst, const int* off, const T* w) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < (int)G.E; e += gridDim.x * blockDim.x) {
    const int row = fdiv(e, G.nx, G.rnx);
    const int ex = e - row * G.nx;
    const int ez = fdiv(row, G.ny, G.rny);
    const int ey = row - ez * G.ny;
    double acc = 0.0;
    for (int o = 0; o < nst; ++o) {
      const int jx = ex + off[3 * o], jy = ey + off[3 * o + 1], jz = ez + off[3 * o + 2];
      if (jx < 0 || jx >= G.nx || jy < 0 || jy >= G.ny || jz < 0 || jz >= G.nz) continue;
      acc += (double)w[o];
    }
    Hsi[e] = (T)(1.0 / acc);
  }
}

template <typename T, int R>
static StencilW<T, R> stencil_weights(double r) {
  StencilW<T, R> W{};
  constexpr int D = 2 * R + 1;
  for (int dz = -R; dz <= R; ++dz)
    for (int dy = -R; dy <= R; ++dy)
      for (int dx = -R; dx <= R; ++dx) {
        double w = r - std::sqrt((double)(dx * dx + dy * dy + dz * dz));
        if (r <= 1.0) w = (dx == 0 && dy == 0 && dz == 0) ? 1.0 : 0.0;
        W.w[(dx + R) + D * ((dy + R) + D * (dz + R))] = (T)(w > 0.0 ? w : 0.0);
      }
  return W;
}

static dim3 filt_grid(const Geo& G) {
  return dim3((G.nx + kFiltBX - 1) / kFiltBX, (G.ny + kFiltBY - 1) / kFiltBY, (G.nz + kFiltDZ - 1) / kFiltDZ);
}
static int64_t filt_blocks(const Geo& G) {
  const dim3 d = filt_grid(G);
  return (int64_t)d.x * d.y * d.z;
}

template <typename T>
hipError_t launch_filter(fbto_grid_s* g, int kind, const T* in, T* out, int want_sum, hipStream_t st) {
  Vecs& V = vecs_of<T>(g);
  if (g->dim == 2) return plane_filter<T>(g, kind, in, out, (const T*)V.Hs, want_sum, st);
  // with a sum, the grid is capped so that its partials stay few
  const int nb = want_sum ? vec_blocks(g->geo.E) : flat_grid(g->geo.E);
  const double r = g->desc.filter_radius;
  const int R = r > 1.0 ? (int)std::ceil(r) - 1 : 0;
  const T* Hsi = (const T*)V.Hs;
  const Geo& G = g->geo;
  const int64_t nbz = filt_blocks(G);
  if (R <= 1 && nbz <= g->max_partials) {
    if (want_sum) g->n_gsum = (int)nbz;
    if (R == 0)
      hipLaunchKernelGGL((k_filter_z<T, 0, false>), filt_grid(G), dim3(kFiltBX * kFiltBY), 0, st, G, kind, in,
                         out, Hsi, stencil_weights<T, 0>(r), want_sum, g->partials, g->max_partials, FiltStep<T>{});
    else
      hipLaunchKernelGGL((k_filter_z<T, 1, false>), filt_grid(G), dim3(kFiltBX * kFiltBY), 0, st, G, kind, in,
                         out, Hsi, stencil_weights<T, 1>(r), want_sum, g->partials, g->max_partials, FiltStep<T>{});
    return hipGetLastError();
  }
  if (R == 2) {
    // tiles of 32 x 8 columns (16 x 16 where the rows are that short); slabs
    // of 4 to 32 layers, so that a small grid still gives 2 blocks per CU
    // (halo planes cost 4 / dz more) and a large one reads its halo seldom
    Stencil2<T> W{};
    for (int d2 = 0; d2 <= 8; ++d2) W.w[d2] = (T)std::max(0.0, r - std::sqrt((double)d2));
    const int bx = G.nx <= 16 ? 16 : 32, by = kVecBlock / bx;
    const int tx = (G.nx + bx - 1) / bx, ty = (G.ny + by - 1) / by;
    const int64_t tiles = (int64_t)tx * ty;
    const int64_t want = std::max<int64_t>(1, 2 * (int64_t)g->n_cu / tiles);  // slabs
    const int dz = (int)std::min<int64_t>(32, std::max<int64_t>(4, (G.nz + want - 1) / want));
    const int64_t nwork = tiles * ((G.nz + dz - 1) / dz);
    if (nwork > INT32_MAX) return hipErrorInvalidValue;
    const int grid = (int)std::min<int64_t>(nwork, g->max_partials);
    if (want_sum) g->n_gsum = grid;
    if (bx == 16)
      hipLaunchKernelGGL((k_filter_r2<T, 16>), dim3(grid), dim3(kVecBlock), 0, st, G, kind, in, out, Hsi, W, want_sum,
                         g->partials, g->max_partials, tx, ty, dz, (int)nwork);
    else
      hipLaunchKernelGGL((k_filter_r2<T, 32>), dim3(grid), dim3(kVecBlock), 0, st, G, kind, in, out, Hsi, W, want_sum,
                         g->partials, g->max_partials, tx, ty, dz, (int)nwork);
    return hipGetLastError();
  }
  if (want_sum) g->n_gsum = nb;
  if (R <= 1)
    hipLaunchKernelGGL((k_filter<T, 1>), dim3(nb), dim3(kVecBlock), 0, st, g->geo, kind, in, out, Hsi,
                       stencil_weights<T, 1>(r), want_sum, g->partials, g->max_partials);
  else
    hipLaunchKernelGGL((k_filter_wide<T>), dim3(nb), dim3(kVecBlock), 0, st, g->geo, kind, in, out, Hsi,
                       g->n_stencil, (const int*)g->stencil_off, stencil_w_of<T>(g), want_sum, g->partials,
                       g->max_partials);
  return hipGetLastError();
}

// Whether the grid's filter is k_filter_z (voxel grid, stencil of radius R <= 1,
// its tiles within the partial slots): the variants fused with the step and with
// the final projection pass need it.
bool zmarch_filter(const fbto_grid_s* g) {
  if (g->dim == 2) return false;
  const double r = g->desc.filter_radius;
  const int R = r > 1.0 ? (int)std::ceil(r) - 1 : 0;
  const Geo& G = g->geo;
  const int64_t nbz = filt_blocks(G);
  return R <= 1 && nbz <= g->max_partials;
}

template <typename T>
hipError_t launch_filter_step(fbto_grid_s* g, const T* ge, const T* x, T* y, double half_alpha,
                              int mean_project, int nb_sum, double lo, double hi, const OuterRec* rec,
                              hipStream_t st, int* nb_seed) {
  if (!zmarch_filter(g)) return hipErrorNotSupported;
  const double r = g->desc.filter_radius;
  const int R = r > 1.0 ? (int)std::ceil(r) - 1 : 0;
  const Geo& G = g->geo;
  const int64_t nbz = filt_blocks(G);
  if (mean_project && (nb_sum < 1 || nb_sum > g->max_partials)) return hipErrorInvalidValue;
  static_assert(kFinishThreads == kFiltBX * kFiltBY, "the record's block is one of the filter's");
  const FiltStep<T> S{x, y, half_alpha, mean_project, nb_sum, lo, hi, g->sc, rec ? 1 : 0, rec ? *rec : OuterRec{}};
  dim3 grid = filt_grid(G);
  if (rec) ++grid.z;
  const T* Hsi = (const T*)vecs_of<T>(g).Hs;  // not read by the plain sum
  if (R == 0)
    hipLaunchKernelGGL((k_filter_z<T, 0, true>), grid, dim3(kFiltBX * kFiltBY), 0, st, G, (int)FILT_SUM,
                       ge, (T*)nullptr, Hsi, stencil_weights<T, 0>(r), 0, g->partials, g->max_partials, S);
  else
    hipLaunchKernelGGL((k_filter_z<T, 1, true>), grid, dim3(kFiltBX * kFiltBY), 0, st, G, (int)FILT_SUM,
                       ge, (T*)nullptr, Hsi, stencil_weights<T, 1>(r), 0, g->partials, g->max_partials, S);
  *nb_seed = (int)nbz;
  return hipGetLastError();
}

template <typename T>
hipError_t launch_hs(fbto_grid_s* g, T* Hs, hipStream_t st) {
  if (g->dim == 2) return plane_hs<T>(g, Hs, st);
  hipLaunchKernelGGL((k_hs<T>), dim3(flat_grid(g->geo.E)), dim3(kVecBlock), 0, st, g->geo, Hs, g->n_stencil,
                     (const int*)g->stencil_off, stencil_w_of<T>(g));
  return hipGetLastError();
}
template hipError_t launch_hs<double>(fbto_grid_s*, double*, hipStream_t);
template hipError_t launch_hs<float>(fbto_grid_s*, float*, hipStream_t);
// ===========================================================================
// Design step and projection onto {lo <= x <= hi, sum x <= vmax}.
//
// f(l) = sum_e clamp(y_e - l, lo, hi) is continuous, non-increasing and
// linear between the breakpoints y_e - lo, y_e - hi (Eq. piecewiseLinearEQ).
// Each search pass evaluates, at the current l, f and the classification of
// every entry just right (+) and just left (-) of l, which fixes the linear
// piece on either side:  f(l') = hi nU + lo nL + sum_A y - l' nA.  The next
// pass solves that piece exactly; if the solution leaves the piece (beyond
// the nearest breakpoint) it becomes a Newton step safeguarded by the
// bracket [a, b] with f(a) > vmax >= f(b), else bisection.
// The kernels that reduce partials first take a thread's entries four at a time,
// a grid apart, the first four loaded before that reduction.
constexpr int kProjChunk = 4;
template <typename T>
__device__ __forceinline__ void load_chunk(const T* a, int64_t n, int64_t first, int64_t stride, T (&v)[kProjChunk]) {
#pragma unroll
  for (int k = 0; k < kProjChunk; ++k) {
    const int64_t e = first + k * stride;
    v[k] = a[e < n ? e : 0];
  }
}

// The gradient step y = x - alpha/2 (g - mean g), with the seed of the
// projection (sum clamp(y), max y, #interior) and its first evaluation, at
// the multiplier of the previous projection (the warm start), into
// evaluation set 0: the first search pass decides from it directly.
template <typename T>
__global__ void __launch_bounds__(kVecBlock)
    k_step(int64_t E, const T* x, const T* gx, T* y, double half_alpha, int mean_project, double lo,
           double hi, double* P, int maxp, int nb_sum, const Scalars* sc) {
  // the first entries are loaded before the reduction of the mean
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  T xv[kProjChunk], gv[kProjChunk];
  load_chunk(x, E, first, stride, xv);
  load_chunk(gx, E, first, stride, gv);
  const double lam_w = sc->lam_prev;
  double mean = 0.0;
  if (mean_project) {
    double v[1];
    const double* src[1] = {pslot(P, P_GSUM, 0, maxp)};
    const int cnt[1] = {nb_sum};
    reduce_parts<1, 0u>(v, src, cnt);
    mean = v[0] / (double)E;
  }
  double v[3] = {0.0, -INFINITY, 0.0};
  double ev[kEval];
  proj_eval_init(ev);
  for (int64_t e0 = first; e0 < E; e0 += kProjChunk * stride) {
    if (e0 != first) {
      load_chunk(x, E, e0, stride, xv);
      load_chunk(gx, E, e0, stride, gv);
    }
#pragma unroll
    for (int k = 0; k < kProjChunk; ++k) {
      const int64_t e = e0 + k * stride;
      if (e >= E) break;
      const T ye = (T)((double)xv[k] - half_alpha * ((double)gv[k] - mean));
      y[e] = ye;
      const double yd = (double)ye;
      v[0] += fmin(fmax(yd, lo), hi);
      v[1] = fmax(v[1], yd);
      v[2] += (yd > lo && yd < hi) ? 1.0 : 0.0;
      proj_eval(ev, yd, lam_w, lo, hi);
    }
  }
  __shared__ double lds[reduce_lds_words<3 + kEval, kVecBlock>()];
  step_parts<kVecBlock>(v, ev, P, maxp, blockIdx.x, lds);
}

__device__ __forceinline__ double* lslot(const ProjWs& W, int i) { return W.base + i * W.stride; }

// Seed of a cold projection: sum clamp(y), max y and the interior count;
// the warm start of the search is cleared.
template <typename T>
__global__ void __launch_bounds__(kVecBlock)
    k_proj_init(int64_t E, const T* y, double lo, double hi, ProjWs W) {
  if (blockIdx.x == 0 && threadIdx.x == 0) W.sc->lam_prev = 0.0;
  double v[3] = {0.0, -INFINITY, 0.0};
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < E;
       e += (int64_t)gridDim.x * blockDim.x) {
    const double yd = (double)y[e];
    v[0] += fmin(fmax(yd, lo), hi);
    v[1] = fmax(v[1], yd);
    v[2] += (yd > lo && yd < hi) ? 1.0 : 0.0;
  }
  double* dst[3] = {lslot(W, L_S0), lslot(W, L_YMAX), lslot(W, L_NACT)};
  write_parts<3, 0x2u, kVecBlock>(v, dst, blockIdx.x);
}

struct ProjDecision {
  double lam, a, b;
  bool done;
  bool bad;
};

// First slot of the evaluation set q of the projection passes.
__host__ __device__ constexpr int proj_set(int q) { return L_E0 + kEval * (q & 1); }
// pass t reads set t and writes set t + 1: two disjoint runs of slots
static_assert(proj_set(0) + kEval <= proj_set(1) && proj_set(1) + kEval <= L_VOL, "projection slot sets overlap");

// Decision from an evaluation v (proj_eval) at lam, with the bracket [a, b] of
// the root.
__device__ __forceinline__ ProjDecision proj_decide_eval(const double (&v)[kEval], double vmax, double lam, double a,
                                                         double b) {
  ProjDecision d{};
  const double F = v[0];
  const double lb = v[5], ub = -v[6];
  double next;
  bool done = false;
  d.bad = !isfinite(F);
  if (d.bad) {
    d.done = true;
    d.lam = b;
    d.a = a;
    d.b = b;
    return d;
  }
  if (F > vmax) {
    a = lam;
    const double nA = v[1];
    if (nA > 0.0) {
      const double ls = (v[2] - vmax) / nA;
      if (ls <= ub) { next = fmax(ls, lam); done = true; }
      else next = (ls > a && ls < b) ? ls : 0.5 * (a + b);
    } else {
      next = 0.5 * (a + b);
    }
  } else if (F < vmax) {
    b = lam;
    const double nA = v[3];
    if (nA > 0.0) {
      const double ls = (v[4] - vmax) / nA;
      if (ls >= lb) { next = fmin(ls, lam); done = true; }
      else next = (ls > a && ls < b) ? ls : 0.5 * (a + b);
    } else {
      next = 0.5 * (a + b);
    }
  } else {
    next = lam;
    done = true;
  }
  if (!done && (!(b > a) || next <= a || next >= b)) {  // bracket exhausted: b is feasible
    done = true;
    next = b;
  }
  d.lam = next;
  d.a = a;
  d.b = b;
  d.done = done;
  return d;
}

// The search state after a pass (identical in every block).  `first`: from
// the seed (sum clamp(y), max y, #interior), and -- warm_eval -- from the
// evaluation at the warm start lam_prev in set 0 when lam_prev lies in the
// bracket; otherwise from the evaluation at `lam` left in set `set`.
__device__ __forceinline__ ProjDecision proj_decide(const ProjWs& W, int nb, bool first, int set, double lo, double hi,
                                                    double vmax, double lam_prev, double lam, double a, double b,
                                                    bool warm_eval = false) {
  double ev[kEval];
  if (!first) {
    const double* src[kEval];
    int cnt[kEval];
#pragma unroll
    for (int i = 0; i < kEval; ++i) {
      src[i] = lslot(W, proj_set(set) + i);
      cnt[i] = nb;
    }
    reduce_parts<kEval, kEvalMax, kVecBlock>(ev, src, cnt);
    return proj_decide_eval(ev, vmax, lam, a, b);
  }
  // the seed and, behind it, the evaluation at the warm start: one reduction
  static_assert(L_S0 == 0 && L_E0 == 3, "the seed's slots come before set 0");
  ProjDecision d{};
  double v[3 + kEval];
  {
    const double* src[3 + kEval];
    int cnt[3 + kEval];
#pragma unroll
    for (int i = 0; i < 3 + kEval; ++i) {
      src[i] = lslot(W, L_S0 + i);
      cnt[i] = i < 3 || warm_eval ? nb : 0;
    }
    reduce_parts<3 + kEval, kSeedEvalMax, kVecBlock>(v, src, cnt);
  }
  const double S0 = v[0], ymax = v[1], nact0 = v[2];
  d.bad = !isfinite(S0);
  if (S0 <= vmax || d.bad) {
    d.done = true;
    d.lam = 0.0;
    d.a = d.b = 0.0;
    return d;
  }
  d.a = 0.0;
  d.b = ymax - lo;
  if (warm_eval && lam_prev > d.a && lam_prev < d.b) {
#pragma unroll
    for (int i = 0; i < kEval; ++i) ev[i] = v[3 + i];
    return proj_decide_eval(ev, vmax, lam_prev, d.a, d.b);
  }
  double l0;
  if (lam_prev > d.a && lam_prev < d.b) l0 = lam_prev;
  else if (nact0 > 0.0) {
    l0 = (S0 - vmax) / nact0;
    if (!(l0 > d.a && l0 < d.b)) l0 = 0.5 * (d.a + d.b);
  } else {
    l0 = 0.5 * (d.a + d.b);
  }
  d.lam = l0;
  d.done = false;
  return d;
}

// Pass t of the search: decides from the seed (t = 0) or from pass t - 1's
// evaluation (set t & 1), then evaluates at the new multiplier into set
// (t + 1) & 1.  The two sets keep a block that starts late from reading
// partials that blocks of the same pass have already overwritten.
template <typename T>
__global__ void __launch_bounds__(kVecBlock)
    k_proj_pass(int64_t E, const T* y, double lo, double hi, double vmax, int pass, ProjWs W, int nb,
                int warm_eval) {
  // nb: the partials the decision reduces (on pass 0 the seed's, which the
  // step may have written with another grid)
  Scalars* sc = W.sc;
  const double* in = sc->ps[pass & 1];
  double* out = sc->ps[(pass + 1) & 1];
  if (pass > 0 && in[3] != 0.0) {            // already solved: carry the state forward
    if (blockIdx.x == 0 && threadIdx.x == 0)
      for (int i = 0; i < 4; ++i) out[i] = in[i];
    return;
  }
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  T yv[kProjChunk];
  load_chunk(y, E, first, stride, yv);
  const ProjDecision d =
      proj_decide(W, nb, pass == 0, pass, lo, hi, vmax, sc->lam_prev, in[0], in[1], in[2], warm_eval != 0);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    out[0] = d.lam;
    out[1] = d.a;
    out[2] = d.b;
    out[3] = d.done ? 1.0 : 0.0;
    if (d.bad) sc->proj_status = (double)FBTO_ERR_NONFINITE;
    else if (pass == 0) sc->proj_status = 0.0;
  }
  if (d.done) return;
  const double lam = d.lam;
  double v[kEval];
  proj_eval_init(v);
  for (int64_t e0 = first; e0 < E; e0 += kProjChunk * stride) {
    if (e0 != first) load_chunk(y, E, e0, stride, yv);
#pragma unroll
    for (int k = 0; k < kProjChunk; ++k) {
      if (e0 + k * stride >= E) break;
      proj_eval(v, (double)yv[k], lam, lo, hi);
    }
  }
  double* dst[kEval];
#pragma unroll
  for (int i = 0; i < kEval; ++i) dst[i] = lslot(W, proj_set(pass + 1) + i);
  write_parts<kEval, kEvalMax, kVecBlock>(v, dst, blockIdx.x);
}

// x = clamp(y - lambda, lo, hi) after `passes` passes.  A search still open
// then decides once more from the last evaluation (set passes & 1); if that
// does not land on the root's piece either, x takes the feasible end of the
// bracket and the status says FBTO_INEXACT.  The lead thread records the
// status (also into *status_out) and lambda.
template <typename T>
__global__ void __launch_bounds__(kVecBlock)
    k_proj_final(int64_t E, const T* y, T* x, double lo, double hi, double vmax, const T* x_old, ProjWs W, int nb,
                 int passes, double* lam_out, double* status_out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  T yv[kProjChunk], xv[kProjChunk];
  load_chunk(y, E, first, stride, yv);
  if (x_old) load_chunk(x_old, E, first, stride, xv);
  Scalars* sc = W.sc;
  const double* in = sc->ps[passes & 1];
  double lam = in[0];
  bool bad = false, unfinished = false;
  if (in[3] == 0.0) {  // pass budget spent: decide from the last evaluation
    const ProjDecision d =
        proj_decide(W, nb, false, passes, lo, hi, vmax, sc->lam_prev, in[0], in[1], in[2]);
    lam = d.done ? d.lam : d.b;
    bad = d.bad;
    unfinished = !d.done;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    double status = sc->proj_status;  // 0, or FBTO_ERR_NONFINITE from a pass
    if (bad) status = (double)FBTO_ERR_NONFINITE;
    else if (unfinished && status == 0.0) status = (double)FBTO_INEXACT;
    sc->proj_status = status;
    sc->lam = lam;
    sc->lam_prev = lam;   // warm start of the next projection (no block here reads it)
    if (lam_out) *lam_out = lam;
    if (status_out) *status_out = status;
  }
  double v[2] = {0.0, 0.0};
  for (int64_t e0 = first; e0 < E; e0 += kProjChunk * stride) {
    if (e0 != first) {
      load_chunk(y, E, e0, stride, yv);
      if (x_old) load_chunk(x_old, E, e0, stride, xv);
    }
#pragma unroll
    for (int k = 0; k < kProjChunk; ++k) {
      const int64_t e = e0 + k * stride;
      if (e >= E) break;
      const T xe = (T)fmin(fmax((double)yv[k] - lam, lo), hi);
      if (x_old) v[1] = fmax(v[1], fabs((double)xe - (double)xv[k]));
      x[e] = xe;
      v[0] += (double)xe;
    }
  }
  double* dst[2] = {lslot(W, L_VOL), lslot(W, L_DX)};
  write_parts<2, 0x2u, kVecBlock>(v, dst, blockIdx.x);
}

// The final pass fused with the forward filter of the next outer iteration:
// both need only y and the multiplier.  Each thread writes x = clamp(y -
// lam, lo, hi) at its own elements, as k_proj_final does, and rho = (H x) /
// Hs there from the same values in the window around them, recomputed from
// y, so that no block waits for another's x.  The multiplier, the status
// and the partials (sum x, max |x - x_old|, x updated in place) are those of
// k_proj_final; rho equals the forward filter of the new x bitwise.
template <typename T, int R>
__global__ void __launch_bounds__(kFiltBX * kFiltBY)
    k_proj_final_filter(Geo G, const T* y, T* x, T* rho, const T* Hsi, StencilW<T, R> Wf, double lo, double hi,
                        double vmax, ProjWs W, int nb, int passes) {
  constexpr int D = 2 * R + 1;
  const FiltPos q = filt_pos(G, blockIdx.z);
  __shared__ T sh[FiltStage<R>::kLds];
  T sv[FiltStage<R>::kTurns];
  unsigned ok;
  filt_load<T, R>(G, q, y, nullptr, false, sv, ok);
  T xo[kFiltDZ], hs[kFiltDZ];  // the design before the step (only its owner reads it) and 1/Hs at the own elements
#pragma unroll
  for (int l = 0; l < kFiltDZ; ++l) {
    const int ez = q.z0 + l;
    const int e = (q.col && ez < q.z1) ? q.ex + G.nx * (q.ey + G.ny * ez) : 0;
    xo[l] = x[e];
    hs[l] = Hsi[e];
  }
  Scalars* sc = W.sc;
  const double* in = sc->ps[passes & 1];
  double lam = in[0];
  bool bad = false, unfinished = false;
  if (in[3] == 0.0) {  // pass budget spent: decide from the last evaluation
    const ProjDecision d =
        proj_decide(W, nb, false, passes, lo, hi, vmax, sc->lam_prev, in[0], in[1], in[2]);
    lam = d.done ? d.lam : d.b;
    bad = d.bad;
    unfinished = !d.done;
  }
  if (q.block == 0 && threadIdx.x == 0) {
    double status = sc->proj_status;  // 0, or FBTO_ERR_NONFINITE from a pass
    if (bad) status = (double)FBTO_ERR_NONFINITE;
    else if (unfinished && status == 0.0) status = (double)FBTO_INEXACT;
    sc->proj_status = status;
    sc->lam = lam;
    sc->lam_prev = lam;
  }
  // the staged values become the new design's (in FP64, rounded to T)
#pragma unroll
  for (int t = 0; t < FiltStage<R>::kTurns; ++t)
    sv[t] = (ok >> t) & 1u ? (T)fmin(fmax((double)sv[t] - lam, lo), hi) : (T)0;
  T win[kFiltDZ + 2 * R][D][D];
  filt_window<T, R>(sv, sh, q, win);
  double v[2] = {0.0, 0.0};
#pragma unroll
  for (int l = 0; l < kFiltDZ; ++l) {
    const int ez = q.z0 + l;
    const T acc = filt_sum<T, R>(Wf, win, l);
    if (q.col && ez < q.z1) {
      const int e = q.ex + G.nx * (q.ey + G.ny * ez);
      const T xe = win[l + R][R][R];
      v[1] = fmax(v[1], fabs((double)xe - (double)xo[l]));
      x[e] = xe;
      v[0] += (double)xe;
      rho[e] = acc * hs[l];
    }
  }
  double* dst[2] = {lslot(W, L_VOL), lslot(W, L_DX)};
  write_parts<2, 0x2u, kFiltBX * kFiltBY>(v, dst, q.block);
}

template <typename T>
hipError_t launch_proj_final_filter(fbto_grid_s* g, const ProjWs& W, const T* y, T* x, T* rho, double lo,
                                    double hi, double vmax, int passes, hipStream_t st, int* nb_final) {
  if (!zmarch_filter(g)) return hipErrorNotSupported;
  const double r = g->desc.filter_radius;
  const int R = r > 1.0 ? (int)std::ceil(r) - 1 : 0;
  const Geo& G = g->geo;
  const int64_t nbz = filt_blocks(G);
  if (nbz > W.maxp) return hipErrorInvalidValue;
  const int nb = vec_blocks(G.E);  // the passes' partials
  const T* Hsi = (const T*)vecs_of<T>(g).Hs;
  if (R == 0)
    hipLaunchKernelGGL((k_proj_final_filter<T, 0>), filt_grid(G), dim3(kFiltBX * kFiltBY), 0, st, G, y, x, rho,
                       Hsi, stencil_weights<T, 0>(r), lo, hi, vmax, W, nb, passes);
  else
    hipLaunchKernelGGL((k_proj_final_filter<T, 1>), filt_grid(G), dim3(kFiltBX * kFiltBY), 0, st, G, y, x, rho,
                       Hsi, stencil_weights<T, 1>(r), lo, hi, vmax, W, nb, passes);
  *nb_final = (int)nbz;
  return hipGetLastError();
}

template <typename T>
hipError_t launch_step(fbto_grid_s* g, const T* x, const T* gx, T* y, double half_alpha,
                       int mean_project, double lo, double hi, hipStream_t st) {
  const int nb = vec_blocks(g->geo.E);
  hipLaunchKernelGGL((k_step<T>), dim3(nb), dim3(kVecBlock), 0, st, g->geo.E, x, gx, y, half_alpha,
                     mean_project, lo, hi, g->partials, g->max_partials, g->n_gsum, (const Scalars*)g->sc);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_project(const ProjWs& W, int64_t E, const T* y, T* x, double lo, double hi, double vmax,
                          int seeded, int passes, const T* x_old, double* lam_out, double* status_out,
                          hipStream_t st, int nb_seed, int skip_final) {
  const int nb = vec_blocks(E);
  if (nb > W.maxp || nb_seed > W.maxp) return hipErrorInvalidValue;
  if (!seeded || nb_seed < 1) nb_seed = nb;
  if (!seeded) {
    hipLaunchKernelGGL((k_proj_init<T>), dim3(nb), dim3(kVecBlock), 0, st, E, y, lo, hi, W);
  }
  for (int p = 0; p < passes; ++p) {
    hipLaunchKernelGGL((k_proj_pass<T>), dim3(nb), dim3(kVecBlock), 0, st, E, y, lo, hi, vmax, p, W,
                       p == 0 ? nb_seed : nb, seeded);
  }
  if (skip_final) return hipGetLastError();
  hipLaunchKernelGGL((k_proj_final<T>), dim3(nb), dim3(kVecBlock), 0, st, E, y, x, lo, hi, vmax, x_old, W, nb,
                     passes, lam_out, status_out);
  return hipGetLastError();
}

// ===========================================================================
// Conversions and iterative-refinement helpers.
// ===========================================================================
__global__ void k_f64_to_f32(const double* in, float* out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = (float)in[i];
}
__global__ void k_f32_to_f64(const float* in, double* out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = (double)in[i];
}
__global__ void k_axpy64(double* u, const double* d, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    u[i] += d[i];
}
__global__ void k_accum_f32(double* u, const float* d, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    u[i] += (double)d[i];
}

static int flat_blocks(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096)); }

template <typename T>
hipError_t launch_convert(const void* in, void* out, int64_t n, int to_double, hipStream_t st) {
  if (to_double)
    hipLaunchKernelGGL(k_f32_to_f64, dim3(flat_blocks(n)), dim3(256), 0, st, (const float*)in, (double*)out, n);
  else
    hipLaunchKernelGGL(k_f64_to_f32, dim3(flat_blocks(n)), dim3(256), 0, st, (const double*)in, (float*)out, n);
  return hipGetLastError();
}
template hipError_t launch_convert<float>(const void*, void*, int64_t, int, hipStream_t);

hipError_t launch_axpy64(double* u, const double* d, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_axpy64, dim3(flat_blocks(n)), dim3(256), 0, st, u, d, n);
  return hipGetLastError();
}
hipError_t launch_ir_scale(fbto_grid_s* g, const double* r64, float* r32, int nrhs, hipStream_t st) {
  return launch_convert<float>(r64, r32, g->geo.ndof * nrhs, 0, st);
}
hipError_t launch_ir_accum(fbto_grid_s* g, double* u64, const float* d32, int nrhs, hipStream_t st) {
  const int64_t n = g->geo.ndof * nrhs;
  hipLaunchKernelGGL(k_accum_f32, dim3(flat_blocks(n)), dim3(256), 0, st, u64, d32, n);
  return hipGetLastError();
}

__global__ void k_solve_info(Scalars* sc, double* info, int nrhs, double steps_override) {
  for (int R = 0; R < nrhs; ++R) {
    double* o = info + R * FBTO_SOLVE_INFO;
    o[FBTO_SI_RNORM2] = sc->rnorm2[R];
    o[FBTO_SI_RNORMI] = sc->rinf[R];
    o[FBTO_SI_FNORM2] = sc->fnorm2[R];
    o[FBTO_SI_STEPS] = steps_override >= 0.0 ? steps_override : sc->steps[R];
    o[FBTO_SI_STATUS] = sc->status[R];
    for (int k = 5; k < FBTO_SOLVE_INFO; ++k) o[k] = 0.0;
  }
}
hipError_t launch_solve_info(fbto_grid_s* g, double* info, int nrhs, double steps_override, hipStream_t st) {
  hipLaunchKernelGGL(k_solve_info, dim3(1), dim3(1), 0, st, g->sc, info, nrhs, steps_override);
  return hipGetLastError();
}

// ===========================================================================
// Optimality metrics of a design (Sec. 4, the error metrics of Thm. 1).
// ===========================================================================
template <typename T>
__global__ void __launch_bounds__(kVecBlock)
    k_sqdist(int64_t n, const T* a, const T* b, double* P, int maxp, int slot) {
  double v[1] = {0.0};
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const double d = (double)a[i] - (double)b[i];
    v[0] += d * d;
  }
  double* dst[1] = {pslot(P, slot, 0, maxp)};
  write_parts<1, 0u>(v, dst, blockIdx.x);
}

template <typename T>
hipError_t launch_sqdist(fbto_grid_s* g, const T* a, const T* b, int64_t n, int slot, hipStream_t st, int* nb_out) {
  const int nb = vec_blocks(n);
  hipLaunchKernelGGL((k_sqdist<T>), dim3(nb), dim3(kVecBlock), 0, st, n, a, b, g->partials, g->max_partials, slot);
  if (nb_out) *nb_out = nb;
  return hipGetLastError();
}

__global__ void __launch_bounds__(kVecBlock)
    k_opt_finish(const double* P, int maxp, int nrhs, int nb_dot, int nb_lo, int nb_hi, double alpha,
                 const Scalars* sc, const Scalars* sc_proj, double* out) {
  double v[3];
  const double* src[3] = {pslot(P, P_DOT, 0, maxp), pslot(P, P_MET0, 0, maxp), pslot(P, P_MET1, 0, maxp)};
  const int cnt[3] = {nb_dot, nb_lo, nb_hi};
  reduce_parts<3, 0u, kVecBlock>(v, src, cnt);
  if (threadIdx.x == 0) {
    double rrel = 0.0, status = 0.0;
    for (int R = 0; R < nrhs; ++R) {
      const double fn = sc->fnorm2[R];
      rrel = fmax(rrel, fn > 0.0 ? sc->rnorm2[R] / fn : sc->rnorm2[R]);
      if (sc->status[R] != 0.0) status = sc->status[R];
    }
    const double ps = sc_proj->proj_status;
    if (ps > 0.0 && (status == 0.0 || ps == (double)FBTO_ERR_NONFINITE)) status = ps;
    out[0] = 0.5 * v[0];
    out[1] = v[2] / (alpha * alpha);
    out[2] = v[1];
    out[3] = rrel;
    out[4] = status;
  }
}

hipError_t launch_opt_finish(fbto_grid_s* g, int nrhs, int nb_dot, int nb_lo, int nb_hi, double alpha,
                             const Scalars* sc_proj, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_opt_finish, dim3(1), dim3(kVecBlock), 0, st, (const double*)g->partials, g->max_partials,
                     nrhs, nb_dot, nb_lo, nb_hi, alpha, (const Scalars*)g->sc, sc_proj, out);
  return hipGetLastError();
}

// ---- explicit instantiations ----------------------------------------------
#define FBTO_INST(T)                                                                                   \
  template hipError_t launch_apply<T>(fbto_grid_s*, const T*, const T*, T*, int, hipStream_t);         \
  template hipError_t launch_resid<T>(fbto_grid_s*, const T*, const T*, const T*, T*, int, int, hipStream_t, \
                                      int*);                                                           \
  template hipError_t launch_resid_diag<T>(fbto_grid_s*, const T*, const T*, const T*, T*, T*, int,    \
                                           hipStream_t, int*);                                         \
  template hipError_t launch_apply_cg<T>(fbto_grid_s*, const T*, const T*, T*, int, int, hipStream_t, int*); \
  template hipError_t launch_apply_lanczos<T>(fbto_grid_s*, const T*, const T*, T*, int, hipStream_t, int*); \
  template hipError_t launch_cg_step<T>(fbto_grid_s*, const T*, T*, T*, const T*, T*, const T*, const T*, int, int, \
                                        bool, const CgCnt&, double, hipStream_t, int*);                \
  template hipError_t launch_cg_sens<T>(fbto_grid_s*, const T*, const CgSet<T>&, T*, const T*, T*, const T*, int, \
                                        const CgCnt&, double, hipStream_t, int*);                      \
  template hipError_t launch_cg_fused<T>(fbto_grid_s*, const T*, const CgSet<T>&, const CgSet<T>&,      \
                                         int, int, int, const CgCnt&, double, hipStream_t, int*);      \
  template hipError_t launch_diag<T>(fbto_grid_s*, const T*, T*, hipStream_t);                         \
  template hipError_t launch_relax_update<T>(fbto_grid_s*, T*, const T*, const T*, int, double, int,    \
                                             hipStream_t);                                             \
  template hipError_t launch_minres<T>(fbto_grid_s*, int, int, const T*, T*, const T*, T*, const T*, T*, \
                                       int, int, double, hipStream_t, int*);                          \
  template hipError_t launch_minres_fused<T>(fbto_grid_s*, const T*, int, const T*, const T*, const T*, T*, T*, T*, \
                                             T*, T*, int, int, double, int, hipStream_t, int*);        \
  template hipError_t launch_sens<T>(fbto_grid_s*, const T*, const T*, const T*, int, T*, const T*,    \
                                     hipStream_t);                                                     \
  template hipError_t launch_dot<T>(fbto_grid_s*, const T*, const T*, int, hipStream_t);               \
  template hipError_t launch_filter<T>(fbto_grid_s*, int, const T*, T*, int, hipStream_t);             \
  template hipError_t launch_sqdist<T>(fbto_grid_s*, const T*, const T*, int64_t, int, hipStream_t, int*); \
  template hipError_t launch_step<T>(fbto_grid_s*, const T*, const T*, T*, double, int, double,       \
                                     double, hipStream_t);                                             \
  template hipError_t launch_project<T>(const ProjWs&, int64_t, const T*, T*, double, double, double, int, \
                                        int, const T*, double*, double*, hipStream_t, int, int);          \
  template hipError_t launch_proj_final_filter<T>(fbto_grid_s*, const ProjWs&, const T*, T*, T*, double, \
                                                  double, double, int, hipStream_t, int*);               \
  template hipError_t launch_filter_step<T>(fbto_grid_s*, const T*, const T*, T*, double, int, int, double, \
                                            double, const OuterRec*, hipStream_t, int*);

FBTO_INST(double)
FBTO_INST(float)

}  // namespace fbto
