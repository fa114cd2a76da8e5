// HIP kernels of the semcheb path for gfx950 (CDNA4, wave64).
//
// Data layout in HBM
//   global vectors      interior lattice unknowns, (I-1) + nx*((J-1) + ny*(K-1))
//   element-local (E-)  [e][k][j][i], (N+1)^3 per element, element e = ex + nex*(ey + ney*ez)
//   geometric factors   [e][c][k][j][i], c = rr, rs, rt, ss, st, tt
// Element-local results of the operator are summed onto the lattice (direct
// stiffness summation) by the kernel that consumes them, reading the 1, 2, 4
// or 8 element copies of each unknown in a fixed order: no atomics, results
// are bitwise reproducible run to run.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>

#include "device_ops.h"

namespace semcheb {
namespace {
using namespace dev;

// Variants of the operator kernel chosen per level by the setup-time autotuner:
// PF (factor prefetch), OCC (waves per SIMD requested from the register allocator)
// and TILE (0: u column in registers with one LDS plane, 1: whole u tile in LDS,
// 2: u tile and the element's BF16 factors in LDS, single precision only; 3: one thread per
// pencil, FP64; 6: one thread per pencil, BF16 factors in LDS; 7: as 3 with ordinary instead
// of non-temporal factor loads; 4: as 2 with every contraction on the
// matrix cores, BF16 factors at N = 7 only; 5: as 0 with the blocks taking elements in
// launch order instead of keeping runs of consecutive elements on one XCD: the FP64
// operator at 32^3, N = 7 then streams its factors as one front through memory and runs
// 5 % faster, although neighbouring elements share fewer u lines in L2).
// pdot (FP64 variants, optional): per-block partials of u . A_L u (see ax_body).
template <int N, typename T, typename GT, int PF, int OCC, int TILE = 0>
__global__ void __launch_bounds__(AxShape<N>::block, OCC)
ax_local_kernel(Box b, int64_t E, const T *__restrict__ u, const GT *__restrict__ G,
                const T *__restrict__ Dm, T *__restrict__ wL, double *__restrict__ pdot) {
  if constexpr (TILE == 5) ax_body<N, T, GT, PF>(blockIdx.x, b, E, u, G, Dm, wL, pdot);
  else if constexpr (TILE == 4) ax_body_mfma<N>(xcd_block(blockIdx.x, gridDim.x), b, E, u, G, Dm, wL);
  else if constexpr (TILE == 3) ax_body_pencil<N, T, GT, GEO_REG, PF>(blockIdx.x, b, E, u, G, Dm, wL, nullptr, pdot);
  else if constexpr (TILE == 7)
    ax_body_pencil<N, T, GT, GEO_REG, PF, false, false>(blockIdx.x, b, E, u, G, Dm, wL, nullptr, pdot);
  else if constexpr (TILE == 6) ax_body_pencil<N, T, GT, GEO_DMA, 0>(xcd_block(blockIdx.x, gridDim.x), b, E, u, G, Dm, wL);
  else if constexpr (TILE == 2) ax_body_dma<N>(xcd_block(blockIdx.x, gridDim.x), b, E, u, G, Dm, wL);
  else if constexpr (TILE == 1)
    ax_body_tile<N, T, GT, PF>(xcd_block(blockIdx.x, gridDim.x), b, E, u, G, Dm, wL, pdot);
  else ax_body<N, T, GT, PF>(xcd_block(blockIdx.x, gridDim.x), b, E, u, G, Dm, wL, pdot);
}

// Operator of trilinear elements with factors computed in the kernel; OCC as above and
// TILE 0 (ax_body_tri, u column in registers) or 1 (one thread per pencil).
// Variants: 0 = (kLoopOcc, 0), 1 = (1, 0), 2 = (min_waves, 1; FP64: 2 waves per SIMD).
// DOT: with the p . Ap sums, whose registers a plain application does without. Order 12, 8.8 M
// nodes, plain: 184 registers and 197 us with the sums' code in the kernel, 168, one wave per SIMD
// more and 139 us without it; pencils at order 10: 40 registers spilled and 102 us, none and 85 us.
template <int N, typename T, int OCC, int TILE, bool DOT>
__global__ void __launch_bounds__(AxShape<N>::block, OCC)
ax_tri_kernel(Box b, int64_t E, const T *__restrict__ u, const T *__restrict__ tri, const T *__restrict__ gxw,
              const T *__restrict__ Dm, T *__restrict__ wL, double *__restrict__ pdot_arg) {
  double *pdot = DOT ? pdot_arg : nullptr;
  if constexpr (TILE == 1)
    ax_body_pencil<N, T, T, GEO_TRI, 0>(xcd_block(blockIdx.x, gridDim.x), b, E, u, tri, Dm, wL, nullptr, pdot, gxw);
  else ax_body_tri<N, T>(xcd_block(blockIdx.x, gridDim.x), b, E, u, tri, gxw, Dm, wL, pdot);
}

// ------------------------------------------------------------------ summation / vector kernels
// out = the summed element copies, VEC unknowns per thread spaced a wavefront apart (see
// strided_first): a block then covers 256 VEC consecutive unknowns, so the element rows that
// share a cache line are mostly read by the same block (FP64, 32^3 at N = 7: 251 MB fetched
// for 134 MB of copies with one unknown per thread)
template <typename T, typename TO = T, int VEC = 1>
__global__ void __launch_bounds__(256) dss_kernel(Box b, int64_t n, const T *__restrict__ wL, TO *__restrict__ out) {
  const int64_t g0 = strided_first<VEC>(blockIdx.x);
  if (g0 >= n) return;
  Ijk cc = ijk_of(b, g0);
#pragma unroll
  for (int q = 0; q < VEC; ++q) {
    if (g0 + 64 * q < n) out[g0 + 64 * q] = (TO)dss_ijk(wL, b, cc);
    if (q + 1 < VEC) ijk_advance(b, cc, 64);
  }
}

// Block reduction of one double to thread 0 (fixed order).
__device__ __forceinline__ double block_sum(double v, double *sm) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) sm[wid] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += sm[w];
  __syncthreads();
  return s;
}

// One thread per VEC unknowns spaced a wavefront apart (see strided_first), one
// partial per block; no grid-stride loop, so every load of a thread is independent.
template <typename T, int VEC>
__device__ __forceinline__ void dss_dot_body(unsigned blk, const Box &b, int64_t n, const T *__restrict__ wL,
                                             T *__restrict__ out, const T *__restrict__ p,
                                             double *__restrict__ partial) {
  __shared__ double sm[4];
  double acc = 0.0;
  const int64_t g0 = strided_first<VEC>(blk);
  if (g0 < n) {
    T pv[VEC], ov[VEC];
#pragma unroll
    for (int q = 0; q < VEC; ++q) pv[q] = (g0 + 64 * q < n) ? p[g0 + 64 * q] : T(0);
    Ijk cc = ijk_of(b, g0);
#pragma unroll
    for (int q = 0; q < VEC; ++q) {
      ov[q] = (g0 + 64 * q < n) ? dss_ijk(wL, b, cc) : T(0);
      if (q + 1 < VEC) ijk_advance(b, cc, 64);
    }
#pragma unroll
    for (int q = 0; q < VEC; ++q) {
      acc += (double)pv[q] * (double)ov[q];
      if (g0 + 64 * q < n) out[g0 + 64 * q] = ov[q];
    }
  }
  const double s = block_sum(acc, sm);
  if (threadIdx.x == 0) *partial = s;
}

template <typename T, int VEC>
__global__ void __launch_bounds__(256)
dss_dot_kernel(Box b, int64_t n, const T *__restrict__ wL, T *__restrict__ out,
               const T *__restrict__ p, double *__restrict__ partials) {
  dss_dot_body<T, VEC>(blockIdx.x, b, n, wL, out, p, partials + blockIdx.x);
}

// Chebyshev step (Algorithms 1 and 2) fused with the summation of A d:
//   rr = R_FROM_B ? b : r_in;  if S_ON_R: rr *= invdiag
//   if SUB_AD:  rr -= (mode 1 ? invdiag * Ad : Ad)
//   dd = (D_INIT ? 0 : d) * a + bc * (mode 4 ? invdiag * rr : rr)
//   x  = (X_INIT ? 0 : X_FROM_D ? cprev * d : x) + c * dd   (not stored with NO_X)
// A smoother started from a zero guess stores no x in its first step (x = c d there) and
// forms it in the second from the direction it reads anyway: the same products, so the
// same results, with one vector write and one read less. The last step of a smoothing
// stores only x (LAST): the residual that follows is formed from x.
// One thread updates VEC unknowns spaced a wavefront apart (see strided_first).
template <typename T, bool SEM, int VEC>
__device__ __forceinline__ void cheb_body(unsigned blk, const Box &b, int64_t n, const T *__restrict__ wsrc,
                                          const T *__restrict__ bvec, const T *__restrict__ r_in,
                                          T *__restrict__ r_out, T *__restrict__ d, T *__restrict__ x,
                                          const T *__restrict__ invdiag, T a, T bc, T c, int flags, int mode,
                                          T cprev = T(0)) {
  const int64_t g0 = strided_first<VEC>(blk);
  if (g0 >= n) return;
  const T *rsrc = (flags & CHEB_R_FROM_B) ? bvec : r_in;
  T sv[VEC], rr[VEC], dd[VEC], xx[VEC], ad[VEC];
#pragma unroll
  for (int q = 0; q < VEC; ++q) {
    const int64_t g = g0 + 64 * q;
    const bool ok = g < n;
    sv[q] = (ok && !(flags & CHEB_R_ONLY)) ? invdiag[g] : T(0);
    rr[q] = ok ? rsrc[g] : T(0);
    dd[q] = (ok && !(flags & CHEB_D_INIT)) ? d[g] : T(0);
    xx[q] = (ok && !(flags & (CHEB_X_INIT | CHEB_X_FROM_D))) ? x[g] : T(0);
    ad[q] = (!SEM && ok && (flags & CHEB_SUB_AD)) ? wsrc[g] : T(0);
  }
  if (SEM && (flags & CHEB_SUB_AD)) {
    Ijk cc = ijk_of(b, g0);
#pragma unroll
    for (int q = 0; q < VEC; ++q) {
      if (g0 + 64 * q < n) ad[q] = dss_ijk(wsrc, b, cc);
      if (q + 1 < VEC) ijk_advance(b, cc, 64);
    }
  }
  if (flags & CHEB_R_ONLY) {  // residual only: r_out = rr - Ad
#pragma unroll
    for (int q = 0; q < VEC; ++q) {
      const int64_t g = g0 + 64 * q;
      if (g < n) r_out[g] = (flags & CHEB_SUB_AD) ? rr[q] - ad[q] : rr[q];
    }
    return;
  }
#pragma unroll
  for (int q = 0; q < VEC; ++q) {
    T r = rr[q], dn, xn;
    cheb_update<T>(r, ad[q], sv[q], dd[q], xx[q], a, bc, c, cprev, flags, mode, dn, xn);
    const int64_t g = g0 + 64 * q;
    if (g < n) {
      if ((flags & CHEB_WRITE_R) && !(flags & CHEB_LAST)) r_out[g] = r;
      if (!(flags & CHEB_LAST)) d[g] = dn;
      if (!(flags & CHEB_NO_X)) x[g] = xn;
    }
  }
}

template <typename T, bool SEM, int VEC>
__global__ void __launch_bounds__(256)
cheb_kernel(Box b, int64_t n, const T *__restrict__ wsrc, const T *__restrict__ bvec,
            const T *__restrict__ r_in, T *__restrict__ r_out, T *__restrict__ d,
            T *__restrict__ x, const T *__restrict__ invdiag, T a, T bc, T c, int flags,
            int mode, T cprev) {
  cheb_body<T, SEM, VEC>(blockIdx.x, b, n, wsrc, bvec, r_in, r_out, d, x, invdiag, a, bc, c, flags, mode, cprev);
}

// rw = (b - DSS(wL)) / multiplicity  (or b / multiplicity when wL is null): the
// weighted residual W_f r_f that the restriction P^T consumes.
template <typename T, int VEC>
__device__ __forceinline__ void resid_weight_body(unsigned blk, const Box &b, int64_t n, const T *__restrict__ wL,
                                                  const T *__restrict__ bvec, T *__restrict__ rw) {
  const int64_t g0 = strided_first<VEC>(blk);
  if (g0 >= n) return;
  T r[VEC];
#pragma unroll
  for (int q = 0; q < VEC; ++q) r[q] = (g0 + 64 * q < n) ? bvec[g0 + 64 * q] : T(0);
  Ijk cc = ijk_of(b, g0);
#pragma unroll
  for (int q = 0; q < VEC; ++q) {
    const int64_t g = g0 + 64 * q;
    if (g < n) {
      T v = r[q];
      int faces;
      if (wL) v -= dss_ijk(wL, b, cc, &faces);
      else faces = face_count(b, cc);
      rw[g] = v * (T)inv_mult_faces(faces);
    }
    if (q + 1 < VEC) ijk_advance(b, cc, 64);
  }
}

template <typename T, int VEC>
__global__ void __launch_bounds__(256)
resid_weight_kernel(Box b, int64_t n, const T *__restrict__ wL, const T *__restrict__ bvec,
                    T *__restrict__ rw) {
  resid_weight_body<T, VEC>(blockIdx.x, b, n, wL, bvec, rw);
}

// ------------------------------------------------------------------ order transfers
// Restriction P^T: for every coarse element, gather the weighted fine residual,
// contract with J^T along i, j, k and write coarse element-local values.
// NF, NC > 0 fix the fine and coarse orders at compile time and BS the block size
// (index arithmetic and loop trip counts then resolve at compile time); 0 reads them at run time.
template <typename T, int NF = 0, int NC = 0, int BS = 0>
__device__ __forceinline__ void restrict_body(int64_t e, const Box &fb, const Box &cb, int64_t E,
                                              const T *__restrict__ rw, const T *__restrict__ Jm,
                                              T *__restrict__ rcL, T *smem) {
  const int nf = NF > 0 ? NF + 1 : fb.N + 1, nc = NC > 0 ? NC + 1 : cb.N + 1;
  const int Nf = nf - 1;
  const int bs = BS > 0 ? BS : (int)blockDim.x;
  T *sJ = smem;                                 // nf*nc
  T *sf = sJ + nf * nc;                         // nf^3 (later nf*nc*nc)
  T *t1 = sf + nf * nf * nf;                    // nf*nf*nc
  if (e >= E) return;
  const Exyz ec = elem_xyz(fb, e);
  const int ex = ec.x, ey = ec.y, ez = ec.z;
  for (int q = threadIdx.x; q < nf * nc; q += bs) sJ[q] = Jm[q];
  for (int q = threadIdx.x; q < nf * nf * nf; q += bs) {
    const int i = q % nf, j = (q / nf) % nf, k = q / (nf * nf);
    const int64_t g = lattice_index(fb, ex * Nf + i, ey * Nf + j, ez * Nf + k);
    const T v = rw[g >= 0 ? g : 0];  // unconditional load, then select
    sf[q] = g >= 0 ? v : T(0);
  }
  __syncthreads();
  // t1[k][j][a] = sum_i J[i][a] sf[k][j][i]
  for (int q = threadIdx.x; q < nf * nf * nc; q += bs) {
    const int a = q % nc, j = (q / nc) % nf, k = q / (nc * nf);
    T s = 0;
    for (int i = 0; i < nf; ++i) s += sJ[i * nc + a] * sf[(k * nf + j) * nf + i];
    t1[(k * nf + j) * nc + a] = s;
  }
  __syncthreads();
  // sf[k][b][a] = sum_j J[j][b] t1[k][j][a]
  for (int q = threadIdx.x; q < nf * nc * nc; q += bs) {
    const int a = q % nc, bq = (q / nc) % nc, k = q / (nc * nc);
    T s = 0;
    for (int j = 0; j < nf; ++j) s += sJ[j * nc + bq] * t1[(k * nf + j) * nc + a];
    sf[(k * nc + bq) * nc + a] = s;
  }
  __syncthreads();
  // out[c][b][a] = sum_k J[k][c] sf[k][b][a]
  T *out = rcL + e * nc * nc * nc;
  for (int q = threadIdx.x; q < nc * nc * nc; q += bs) {
    const int a = q % nc, bq = (q / nc) % nc, c = q / (nc * nc);
    T s = 0;
    for (int k = 0; k < nf; ++k) s += sJ[k * nc + c] * sf[(k * nc + bq) * nc + a];
    out[q] = s;
  }
}

template <typename T, int NF, int NC>
__global__ void __launch_bounds__(128)
restrict_kernel(Box fb, Box cb, int64_t E, const T *__restrict__ rw, const T *__restrict__ Jm,
                T *__restrict__ rcL) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  restrict_body<T, NF, NC, 128>(blockIdx.x, fb, cb, E, rw, Jm, rcL, reinterpret_cast<T *>(smem_raw));
}

// Prolongation x_f += P x_c: every fine element interpolates the coarse element
// values and updates the fine unknowns it owns (local i, j, k < N_f).
template <typename T, int NF = 0, int NC = 0, int BS = 0>
__device__ __forceinline__ void prolong_body(int64_t e, const Box &fb, const Box &cb, int64_t E,
                                             const T *__restrict__ xc, const T *__restrict__ Jm,
                                             T *__restrict__ xf, double *__restrict__ zout, T *smem) {
  const int nf = NF > 0 ? NF + 1 : fb.N + 1, nc = NC > 0 ? NC + 1 : cb.N + 1;
  const int Nf = nf - 1, Nc = nc - 1;
  const int bs = BS > 0 ? BS : (int)blockDim.x;
  T *sJ = smem;                                 // nf*nc
  T *sc = sJ + nf * nc;                         // nc^3
  T *t1 = sc + nc * nc * nc;                    // nc*nc*nf
  T *t2 = t1 + nc * nc * nf;                    // nc*nf*nf
  if (e >= E) return;
  const Exyz ec = elem_xyz(fb, e);
  const int ex = ec.x, ey = ec.y, ez = ec.z;
  for (int q = threadIdx.x; q < nf * nc; q += bs) sJ[q] = Jm[q];
  for (int q = threadIdx.x; q < nc * nc * nc; q += bs) {
    const int a = q % nc, bq = (q / nc) % nc, c = q / (nc * nc);
    const int64_t g = lattice_index(cb, ex * Nc + a, ey * Nc + bq, ez * Nc + c);
    const T v = xc[g >= 0 ? g : 0];
    sc[q] = g >= 0 ? v : T(0);
  }
  __syncthreads();
  // t1[c][b][i] = sum_a J[i][a] sc[c][b][a]
  for (int q = threadIdx.x; q < nc * nc * nf; q += bs) {
    const int i = q % nf, bq = (q / nf) % nc, c = q / (nf * nc);
    T s = 0;
    for (int a = 0; a < nc; ++a) s += sJ[i * nc + a] * sc[(c * nc + bq) * nc + a];
    t1[(c * nc + bq) * nf + i] = s;
  }
  __syncthreads();
  // t2[c][j][i] = sum_b J[j][b] t1[c][b][i]
  for (int q = threadIdx.x; q < nc * nf * nf; q += bs) {
    const int i = q % nf, j = (q / nf) % nf, c = q / (nf * nf);
    T s = 0;
    for (int bq = 0; bq < nc; ++bq) s += sJ[j * nc + bq] * t1[(c * nc + bq) * nf + i];
    t2[(c * nf + j) * nf + i] = s;
  }
  __syncthreads();
#pragma unroll 1
  for (int q = threadIdx.x; q < Nf * Nf * Nf; q += bs) {
    const int i = q % Nf, j = (q / Nf) % Nf, k = q / (Nf * Nf);
    const int64_t g = lattice_index(fb, ex * Nf + i, ey * Nf + j, ez * Nf + k);
    if (g < 0) continue;
    T s = 0;
    for (int c = 0; c < nc; ++c) s += sJ[k * nc + c] * t2[(c * nf + j) * nf + i];
    if (zout) zout[g] = (double)(xf[g] + s);  // last step of a cycle: widened result only
    else xf[g] += s;
  }
}

template <typename T, int NF, int NC>
__global__ void __launch_bounds__(128)
prolong_kernel(Box fb, Box cb, int64_t E, const T *__restrict__ xc, const T *__restrict__ Jm,
               T *__restrict__ xf, double *__restrict__ zout) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  prolong_body<T, NF, NC, 128>(blockIdx.x, fb, cb, E, xc, Jm, xf, zout, reinterpret_cast<T *>(smem_raw));
}

// Transfers for compiled (fine, coarse) order pairs: a block covers EX consecutive
// elements along x (same ey, ez), so its fine-lattice rows are EX*Nf contiguous unknowns
// (coalesced loads and stores instead of Nf-long runs per element). The per-element
// contractions and their summation order are those of restrict_body / prolong_body.
template <int NF, int NC, typename T>
constexpr int rows_ex() {
  return (sizeof(T) == 4 ? 64 : 32) / NF < 1 ? 1 : ((sizeof(T) == 4 ? 64 : 32) / NF > 8 ? 8 : (sizeof(T) == 4 ? 64 : 32) / NF);
}

// Elements per block of the prolongation: row runs of about 450-500 bytes (the partial
// cache lines at the run ends cost less the longer the run), within 36 KB of LDS per block.
// FP64 runs stop at 56 unknowns: the contractions of a longer run take more than one pass of the block.
template <int NF, int NC, typename T>
constexpr int prolong_ex() {
  constexpr int nf = NF + 1, nc = NC + 1;
  constexpr int per = (int)sizeof(T) * (nc * nc * nc + nc * nf * (nc + 1) + nc * nf * (nf + 1) + nf);
  int ex = (sizeof(T) == 4 ? 128 : 56) / NF;
  if (ex > 16) ex = 16;
  while (ex > 1 && ex * per > 36864) --ex;
  return ex < 1 ? 1 : ex;
}

// Elements per block where the standard runs give less than one block per compute unit: a
// quarter (512 elements at order 7, FP64: prolongation 10.6 -> 6.6 us, restriction
// 9.3 -> 5.0 us; with 512 standard blocks, 4096 elements, it is the slower form: 15.8 against 17.2 us).
template <int EX>
constexpr int short_ex() {
  return EX >= 4 ? EX / 4 : 1;
}
inline bool short_runs(const Level &F, int ex) {
  return ex > 1 && (int64_t)((F.nex + ex - 1) / ex) * F.ney * F.nez < 256;
}

// A thread of the contractions reads one line of the element and forms all of its products, the
// interpolation matrix in scalar registers: an LDS read per value and direction instead of two per
// multiply-add, which bounded the kernels. LDS values of a block: down, the staged rows and the
// results of the first two contractions; up, the coarse values and the results; the pitches put the
// lines that a wave reads together into distinct banks. 24 x 16 x 20 elements, FP64, 7 -> 5:
// restriction 34.9 -> 25.5 us, prolongation 25.0 -> 20.9 us; 32^3, single precision, 7 -> 3: 26.9 ->
// 24.4 and 65.9 -> 59.5 us (the latter with the Krylov reductions, near its HBM bytes).
template <int NF, int NC, int EX>
struct RowsLds {
  static constexpr int nf = NF + 1, nc = NC + 1, RW = EX * NF + 1;
  static constexpr int p1 = nc * (nf + 1);                          // down: per k of t1
  static constexpr int down = nf * nf * RW + EX * nf * p1 + EX * nf * nc * nc;
  static constexpr int u1 = nf * (nc + 1), u2 = nf * (nf + 1);      // up: per c of t1 and of t2
  static constexpr int up = EX * (nc * nc * nc + nc * u1 + nc * u2 + nf);
};

template <typename T, int NF, int NC, int EX>
__device__ __forceinline__ void
restrict_rows_body(unsigned blk, const Box &fb, const Box &cb, const T *__restrict__ rw, const T *__restrict__ Jm,
                   T *__restrict__ rcL, const T *__restrict__ wL, const T *__restrict__ bvec, T *lds) {
  constexpr int nf = NF + 1, nc = NC + 1, RW = EX * NF + 1;
  using X = RowsLds<NF, NC, EX>;
  ConstTable<T> *J = (ConstTable<T> *)Jm;
  T *srow = lds;                           // fine rows [k][j][i_global]
  T *t1 = srow + nf * nf * RW;             // [el][k](p1) [j][a]
  T *t2 = t1 + EX * nf * X::p1;            // [el][k][b][a]
  const int ngx = (fb.nex + EX - 1) / EX;
  const int gx = blk % ngx;
  const int ey = (blk / ngx) % fb.ney, ez = blk / (ngx * fb.ney);
  const int ex0 = gx * EX;
  const int nel = fb.nex - ex0 < EX ? fb.nex - ex0 : EX;
  const int t = threadIdx.x;
  // stage the fine rows: when a thread's share is small (kL values) all of its loads are
  // issued before the first LDS store, so they are in flight together. With rw == nullptr
  // the weighted residual is formed here, as resid_weight_body forms it (same operations,
  // same order): (b - sum of the element copies of wL) / multiplicity, or b / multiplicity
  // without wL
  constexpr int kL = (nf * nf * RW + 255) / 256;
  auto fine = [&](int64_t g, int I, int J, int K) -> T {
    if (rw) return rw[g];
    const Ijk cc{I, J, K};
    T v = bvec[g];
    int faces;
    if (wL) v -= dss_ijk(wL, fb, cc, &faces);
    else faces = face_count(fb, cc);
    return v * (T)inv_mult_faces(faces);
  };
  if constexpr (kL <= 24) {
    T v[kL];
#pragma unroll
    for (int it = 0; it < kL; ++it) {
      const int q = t + 256 * it;
      v[it] = T(0);
      if (q < nf * nf * RW) {
        const int ig = q % RW, j = (q / RW) % nf, k = q / (RW * nf);
        const int I = ex0 * NF + ig, J = ey * NF + j, K = ez * NF + k;
        const int64_t g = lattice_index(fb, I, J, K);
        if (g >= 0) v[it] = fine(g, I, J, K);
      }
    }
#pragma unroll
    for (int it = 0; it < kL; ++it)
      if (t + 256 * it < nf * nf * RW) srow[t + 256 * it] = v[it];
  } else {
    for (int q = t; q < nf * nf * RW; q += 256) {
      const int ig = q % RW, j = (q / RW) % nf, k = q / (RW * nf);
      const int I = ex0 * NF + ig, J = ey * NF + j, K = ez * NF + k;
      const int64_t g = lattice_index(fb, I, J, K);
      srow[q] = g >= 0 ? fine(g, I, J, K) : T(0);
    }
  }
  __syncthreads();
  for (int q = t; q < EX * nf * nf; q += 256) {  // t1[el][k][j][a] = sum_i J[i][a] f[k][j][i]
    const int jk = q % (nf * nf), el = q / (nf * nf), j = jk % nf, k = jk / nf;
    const T *row = srow + jk * RW + el * NF;
    T v[nf];
#pragma unroll
    for (int i = 0; i < nf; ++i) v[i] = row[i];
    T *o = t1 + (el * nf + k) * X::p1 + j * nc;
#pragma unroll
    for (int a = 0; a < nc; ++a) {
      T acc = 0;
#pragma unroll
      for (int i = 0; i < nf; ++i) acc += J[i * nc + a] * v[i];
      o[a] = acc;
    }
  }
  __syncthreads();
  for (int q = t; q < EX * nf * nc; q += 256) {  // t2[el][k][b][a] = sum_j J[j][b] t1[el][k][j][a]
    const int a = q % nc, ek = q / nc;
    T v[nf];
#pragma unroll
    for (int j = 0; j < nf; ++j) v[j] = t1[ek * X::p1 + j * nc + a];
    T *o = t2 + ek * nc * nc + a;
#pragma unroll
    for (int bq = 0; bq < nc; ++bq) {
      T acc = 0;
#pragma unroll
      for (int j = 0; j < nf; ++j) acc += J[j * nc + bq] * v[j];
      o[bq * nc] = acc;
    }
  }
  __syncthreads();
  const int64_t e0 = ex0 + (int64_t)fb.nex * (ey + (int64_t)fb.ney * ez);
  for (int q = t; q < nel * nc * nc; q += 256) {  // out[el][c][b][a] = sum_k J[k][c] t2[el][k][b][a]
    const int ab = q % (nc * nc), el = q / (nc * nc);
    T v[nf];
#pragma unroll
    for (int k = 0; k < nf; ++k) v[k] = t2[(el * nf + k) * nc * nc + ab];
    T *o = rcL + (e0 + el) * (nc * nc * nc) + ab;
#pragma unroll
    for (int c = 0; c < nc; ++c) {
      T acc = 0;
#pragma unroll
      for (int k = 0; k < nf; ++k) acc += J[k * nc + c] * v[k];
      o[c * nc * nc] = acc;
    }
  }
}

template <typename T, int NF, int NC, int EX>
__global__ void __launch_bounds__(256)
restrict_rows_kernel(Box fb, Box cb, const T *__restrict__ rw, const T *__restrict__ Jm, T *__restrict__ rcL,
                     const T *__restrict__ wL, const T *__restrict__ bvec) {
  __shared__ T lds[RowsLds<NF, NC, EX>::down];
  restrict_rows_body<T, NF, NC, EX>(blockIdx.x, fb, cb, rw, Jm, rcL, wL, bvec, lds);
}

template <typename T, int NF, int NC, int EX, typename TC>
__device__ __forceinline__ void
prolong_rows_body(unsigned blk, const Box &fb, const Box &cb, const TC *__restrict__ xc, const T *__restrict__ Jm,
                  T *__restrict__ xf, double *__restrict__ zout, const double *__restrict__ dr1,
                  const double *__restrict__ dr2, double *__restrict__ partials, T *lds) {
  constexpr int nf = NF + 1, nc = NC + 1;
  using X = RowsLds<NF, NC, EX>;
  ConstTable<T> *J = (ConstTable<T> *)Jm;
  T *sc = lds;                             // [el][c][b][a]
  T *t1 = sc + EX * nc * nc * nc;          // [el][c](u1) [b][i]
  T *t2 = t1 + EX * nc * X::u1;            // [el](nc * u2 + nf) [c](u2) [j][i]
  const int ngx = (fb.nex + EX - 1) / EX;
  const int gx = blk % ngx;
  const int ey = (blk / ngx) % fb.ney, ez = blk / (ngx * fb.ney);
  const int ex0 = gx * EX;
  const int nel = fb.nex - ex0 < EX ? fb.nex - ex0 : EX;
  const int t = threadIdx.x;
  // owned fine nodes (local i, j, k < NF) of the run in columns along k: rows of EX*NF contiguous
  // unknowns, those past a ragged end lie outside the lattice (the divisions of the index then are
  // by constants). A thread's operands are loaded before the contractions where it has one column
  constexpr int RL = EX * NF, ncol = NF * RL;
  constexpr int kIt = (ncol + 255) / 256;
  const int64_t plane = (int64_t)fb.nx * fb.ny;
  T xq[NF];
  double r1q[NF], r2q[NF];
  auto column = [&](int q, int64_t &g0) {  // unknown at k = 0 of the column (may lie below the lattice)
    const int ig = q % RL, j = q / RL;
    const int I = ex0 * NF + ig, Jy = ey * NF + j;
    g0 = (I - 1) + (int64_t)fb.nx * ((Jy - 1) + (int64_t)fb.ny * (ez * NF - 1));
    return q < ncol && I >= 1 && I <= fb.nx && Jy >= 1 && Jy <= fb.ny;
  };
  auto inside = [&](int k) { return ez * NF + k >= 1 && ez * NF + k <= fb.nz; };
  auto load = [&](bool ok, int64_t g0) {
#pragma unroll
    for (int k = 0; k < NF; ++k) {
      const int64_t gs = ok && inside(k) ? g0 + plane * k : 0;  // in bounds; the value is not used
      xq[k] = xf[gs];
      r1q[k] = dr1 ? dr1[gs] : 0.0;
      r2q[k] = dr2 ? dr2[gs] : 0.0;
    }
  };
  int64_t g0 = 0;
  bool ok = column(t, g0);
  if constexpr (kIt == 1) load(ok, g0);
  for (int q = t; q < EX * nc * nc * nc; q += 256) {
    const int a = q % nc, bq = (q / nc) % nc, c = (q / (nc * nc)) % nc, el = q / (nc * nc * nc);
    const int64_t g = el < nel ? lattice_index(cb, (ex0 + el) * NC + a, ey * NC + bq, ez * NC + c) : -1;
    const T v = (T)xc[g >= 0 ? g : 0];
    sc[q] = g >= 0 ? v : T(0);
  }
  __syncthreads();
  for (int q = t; q < EX * nc * nc; q += 256) {  // t1[el][c][b][i] = sum_a J[i][a] sc[el][c][b][a]
    const int bq = q % nc, ecl = q / nc;
    T v[nc];
#pragma unroll
    for (int a = 0; a < nc; ++a) v[a] = sc[q * nc + a];
    T *o = t1 + ecl * X::u1 + bq * nf;
#pragma unroll
    for (int i = 0; i < nf; ++i) {
      T acc = 0;
#pragma unroll
      for (int a = 0; a < nc; ++a) acc += J[i * nc + a] * v[a];
      o[i] = acc;
    }
  }
  __syncthreads();
  for (int q = t; q < EX * nc * nf; q += 256) {  // t2[el][c][j][i] = sum_b J[j][b] t1[el][c][b][i]
    const int i = q % nf, ecl = q / nf, c = ecl % nc, el = ecl / nc;
    T v[nc];
#pragma unroll
    for (int bq = 0; bq < nc; ++bq) v[bq] = t1[ecl * X::u1 + bq * nf + i];
    T *o = t2 + el * (nc * X::u2 + nf) + c * X::u2 + i;
#pragma unroll
    for (int j = 0; j < nf; ++j) {
      T acc = 0;
#pragma unroll
      for (int bq = 0; bq < nc; ++bq) acc += J[j * nc + bq] * v[bq];
      o[j * nf] = acc;
    }
  }
  __syncthreads();
  double d1 = 0.0, d2 = 0.0;
  for (int q = t; q < ncol; q += 256) {
    if constexpr (kIt > 1) {
      ok = column(q, g0);
      load(ok, g0);
    }
    const int ig = q % RL, j = q / RL, el = ig / NF, i = ig - el * NF;
    T v[nc];
#pragma unroll
    for (int c = 0; c < nc; ++c) v[c] = t2[el * (nc * X::u2 + nf) + c * X::u2 + j * nf + i];
#pragma unroll
    for (int k = 0; k < NF; ++k) {
      T acc = 0;
#pragma unroll
      for (int c = 0; c < nc; ++c) acc += J[k * nc + c] * v[c];
      if (ok && inside(k)) {
        const int64_t g = g0 + plane * k;
        const T xv = xq[k] + acc;
        if (zout) zout[g] = (double)xv;
        else xf[g] = xv;
        d1 += (double)xv * r1q[k];
        d2 += (double)xv * r2q[k];
      }
    }
  }
  // optional Krylov reductions over the written result z (z . r1, z . r2): one partial per block
  if (dr1) {
    __shared__ double sm[4];
    const int nd = dr2 ? 2 : 1;
    double s = block_sum(d1, sm);
    if (threadIdx.x == 0) partials[(int64_t)blk * nd] = s;
    if (dr2) {
      s = block_sum(d2, sm);
      if (threadIdx.x == 0) partials[(int64_t)blk * nd + 1] = s;
    }
  }
}

template <typename T, int NF, int NC, int EX, typename TC = T>
__global__ void __launch_bounds__(256)
prolong_rows_kernel(Box fb, Box cb, const TC *__restrict__ xc, const T *__restrict__ Jm, T *__restrict__ xf,
                    double *__restrict__ zout, const double *__restrict__ dr1, const double *__restrict__ dr2,
                    double *__restrict__ partials) {
  __shared__ T lds[RowsLds<NF, NC, EX>::up];
  prolong_rows_body<T, NF, NC, EX, TC>(blockIdx.x, fb, cb, xc, Jm, xf, zout, dr1, dr2, partials, lds);
}

// ------------------------------------------------------------------ Schwarz smoother
// Fast-diagonalisation solve of one extended element (nb = N + 3 unknowns per axis) per block,
// one thread per line of nb values: a line is read once, multiplied with the axis' eigenvector
// matrix in registers and put back, so a value crosses LDS once per direction instead of being
// read nb times. The block's three matrices are wave-uniform and come through scalar registers.
// Lines along z are the threads' own columns (registers only); x forward, the division by the
// eigenvalue sums and x backward happen in one visit of a line. RAS keeps an element's own nodes
// only: the last contractions skip the outer layer and the result is stored as an element-local
// vector ([e][(N+1)^3]); ASM stores all nb^3 values. VALU bound (6 nb^4 multiply-adds per element).
// 24^3 elements at N = 7, single precision, RAS: 178.8 -> 53.1 us per launch with one thread per
// output and plane; order 3: 25.9 -> 13.0 us.
template <int N>
struct SwShape {
  static constexpr int nb = N + 3, nb2 = nb * nb, nb3 = nb2 * nb;
  static constexpr int block = (nb2 + 63) / 64 * 64;
};

// o[c] = sum_k M[k * nb + c] v[k] (forward) and o[k] = sum_c M[k * nb + c] v[c] (backward), M
// wave-uniform, one row of M at a time; the backward product only for rows lo <= k < hi
template <int nb, typename T>
__device__ __forceinline__ void sw_forward(const T *__restrict__ M, const T (&v)[nb], T (&o)[nb]) {
#pragma unroll
  for (int c = 0; c < nb; ++c) o[c] = 0;
#pragma unroll
  for (int k = 0; k < nb; ++k)
#pragma unroll
    for (int c = 0; c < nb; ++c) o[c] += M[k * nb + c] * v[k];
}
template <int nb, int lo, int hi, typename T>
__device__ __forceinline__ void sw_backward(const T *__restrict__ M, const T (&v)[nb], T (&o)[nb]) {
#pragma unroll
  for (int k = lo; k < hi; ++k) {
    T acc = 0;
#pragma unroll
    for (int c = 0; c < nb; ++c) acc += M[k * nb + c] * v[c];
    o[k] = acc;
  }
}

template <int N, typename T, bool RAS>
__global__ void __launch_bounds__(SwShape<N>::block)
schwarz_local_kernel(Box b, int64_t E, const T *__restrict__ v, const T *__restrict__ Sm,
                     const T *__restrict__ Dinv, T *__restrict__ ye) {
  using S = SwShape<N>;
  constexpr int nb = S::nb, nb2 = S::nb2, nb3 = S::nb3, n1 = N + 1;
  constexpr int rp = nb | 1;                          // odd row pitch: lines along x in distinct banks
  constexpr int lo = RAS ? 1 : 0, hi = RAS ? nb - 1 : nb;  // rows kept by the last contractions
  __shared__ T A[nb2 * rp];
  const int64_t e = xcd_block(blockIdx.x, gridDim.x);  // grid: one block per element
  const int t = threadIdx.x;
  const bool act = t < nb2;
  const int tc = act ? t : 0;
  const int i = tc % nb, j = tc / nb;
  const Exyz ec = elem_xyz(b, e);
  const int I = ec.x * N - 1 + i, J = ec.y * N - 1 + j;
  const bool inIJ = act && I >= 1 && I <= b.nx && J >= 1 && J <= b.ny;
  const int64_t gIJ = (int64_t)(I - 1) + (int64_t)b.nx * (J - 1), plane = (int64_t)b.nx * b.ny;
  T p[nb], q[nb], dv[nb];
#pragma unroll
  for (int k = 0; k < nb; ++k) {
    const int K = ec.z * N - 1 + k;
    const bool ok = inIJ && K >= 1 && K <= b.nz;
    const T val = v[ok ? gIJ + plane * (K - 1) : 0];
    p[k] = ok ? val : T(0);
  }
#pragma unroll
  for (int a = 0; a < nb; ++a) dv[a] = Dinv[e * nb3 + (int64_t)tc * nb + a];  // line t along x
  const T *Sx = Sm + e * 3 * nb2, *Sy = Sx + nb2, *Sz = Sy + nb2;
  const int cz = j * rp + i, cy = j * nb * rp + i, cx = tc * rp;  // the thread's three lines
  sw_forward<nb, T>(Sz, p, q);
  if (act) {
#pragma unroll
    for (int k = 0; k < nb; ++k) A[k * nb * rp + cz] = q[k];
  }
  __syncthreads();
#pragma unroll
  for (int l = 0; l < nb; ++l) p[l] = A[cy + l * rp];
  sw_forward<nb, T>(Sy, p, q);
  if (act) {  // in place: a line is read and written by the same thread
#pragma unroll
    for (int l = 0; l < nb; ++l) A[cy + l * rp] = q[l];
  }
  __syncthreads();
#pragma unroll
  for (int l = 0; l < nb; ++l) p[l] = A[cx + l];
  sw_forward<nb, T>(Sx, p, q);
#pragma unroll
  for (int l = 0; l < nb; ++l) q[l] *= dv[l];
  sw_backward<nb, lo, hi, T>(Sx, q, p);
  if (act) {
#pragma unroll
    for (int l = lo; l < hi; ++l) A[cx + l] = p[l];
  }
  __syncthreads();
#pragma unroll
  for (int l = 0; l < nb; ++l) p[l] = A[cy + l * rp];
  sw_backward<nb, lo, hi, T>(Sy, p, q);
  if (act) {
#pragma unroll
    for (int l = lo; l < hi; ++l) A[cy + l * rp] = q[l];
  }
  __syncthreads();
  if (!act || i < lo || i >= hi || j < lo || j >= hi) return;
#pragma unroll
  for (int k = 0; k < nb; ++k) p[k] = A[k * nb * rp + cz];
  sw_backward<nb, lo, hi, T>(Sz, p, q);
  constexpr int no = RAS ? n1 : nb;  // stored values per axis
  T *out = ye + e * (int64_t)(no * no * no) + (j - lo) * no + (i - lo);
#pragma unroll
  for (int k = lo; k < hi; ++k) out[(k - lo) * no * no] = q[k];
}

// Subdomains containing lattice coordinate I along one axis (N >= 3): at most two, as
// (element, subdomain-local index) pairs.
__device__ __forceinline__ int sw_axis(int I, int N, const FastDiv &fN, int nelem, int *el, int *loc) {
  const int q = fdiv(fN, I), r = I - q * N;
  int cnt = 0;
  auto add = [&](int e, int l) {
    if (e >= 0 && e < nelem) {
      el[cnt] = e;
      loc[cnt] = l;
      ++cnt;
    }
  };
  add(q, r + 1);  // the element whose own nodes hold I (for r == 0: its local node 0)
  if (r == 0) add(q - 1, N + 1);
  if (r == 1) add(q - 1, N + 2);
  if (r == N - 1) add(q + 1, 0);
  return cnt;
}

// The weighted node sum of the subdomain results fused with the Chebyshev update. RAS: the
// element copies of the own nodes, averaged (the direct-stiffness gather of dss_ijk, all copies
// requested at once); ASM: every subdomain that holds the node. The Chebyshev vectors are
// requested before the copies. 24^3, N = 7, single precision, RAS: 35.5 -> 18.8 us (order 3: 15.8 -> 6.3).
template <typename T, int VEC, bool RAS>
__global__ void __launch_bounds__(256)
schwarz_gather_kernel(Box b, int64_t n, const T *__restrict__ ye, int gmode, T *__restrict__ z,
                      T *__restrict__ rv, T *__restrict__ d, T *__restrict__ x, T a, T bc, T c, int flags) {
  const int nb = b.N + 3;
  const int64_t nb3 = (int64_t)nb * nb * nb;
  const int64_t g0 = strided_first<VEC>(blockIdx.x);
  if (g0 >= n) return;
  T rr[VEC], dd[VEC], xx[VEC], zv[VEC];
#pragma unroll
  for (int q = 0; q < VEC; ++q) {
    const int64_t g = g0 + 64 * q;
    const bool ok = g < n && gmode != SWG_PLAIN;
    rr[q] = (ok && gmode == SWG_CHEB1 && !(flags & CHEB_D_INIT)) ? rv[g] : T(0);
    dd[q] = (ok && !(flags & CHEB_D_INIT)) ? d[g] : T(0);
    xx[q] = (ok && !(flags & CHEB_X_INIT)) ? x[g] : T(0);
  }
  Ijk cc = ijk_of(b, g0);
#pragma unroll
  for (int q = 0; q < VEC; ++q) {
    if (g0 + 64 * q < n) {
      if constexpr (RAS) {
        int faces;
        const T acc = dss_ijk(ye, b, cc, &faces);
        zv[q] = acc * (T)inv_mult_faces(faces);
      } else {
        int ex[2], lx[2], ey[2], ly[2], ez[2], lz[2];
        const int cx = sw_axis(cc.I, b.N, b.fN, b.nex, ex, lx);
        const int cy = sw_axis(cc.J, b.N, b.fN, b.ney, ey, ly);
        const int cz = sw_axis(cc.K, b.N, b.fN, b.nez, ez, lz);
        T acc = 0;
        for (int w = 0; w < cz; ++w)
          for (int v2 = 0; v2 < cy; ++v2)
            for (int u2 = 0; u2 < cx; ++u2) {
              const int64_t e = ex[u2] + (int64_t)b.nex * (ey[v2] + (int64_t)b.ney * ez[w]);
              acc += ye[e * nb3 + ((int64_t)lz[w] * nb + ly[v2]) * nb + lx[u2]];
            }
        zv[q] = acc / (T)(cx * cy * cz);
      }
    }
    if (q + 1 < VEC) ijk_advance(b, cc, 64);
  }
#pragma unroll
  for (int q = 0; q < VEC; ++q) {
    const int64_t g = g0 + 64 * q;
    if (g >= n) continue;
    if (gmode == SWG_PLAIN) {
      z[g] = zv[q];
    } else if (gmode == SWG_CHEB4) {
      const T dn = a * dd[q] + bc * zv[q];
      d[g] = dn;
      x[g] = xx[q] + c * dn;
    } else {
      const T rn = (flags & CHEB_D_INIT) ? zv[q] : rr[q] - zv[q];
      rv[g] = rn;
      const T dn = a * dd[q] + bc * rn;
      d[g] = dn;
      x[g] = xx[q] + c * dn;
    }
  }
}

// ------------------------------------------------------------------ sparse / dense
// Dense row-major products of the coarse solve, one 256-thread block per row:
//   y = M1 x1 - M2 x2 (M2 optional), then y = b - y when sub = 1.
// Each thread issues its (up to kGemvUnroll) loads per matrix before summing, so a
// whole row is in flight at once; rows are short (about 1e3 entries) and the
// solve chains dozens of these products, so latency rather than bandwidth decides.
constexpr int kGemvUnroll = 8;
__device__ __forceinline__ void gemv_row(int64_t row, int64_t nrows, int64_t n1c, const double *__restrict__ M1,
                                         const double *__restrict__ x1, int64_t n2c,
                                         const double *__restrict__ M2, const double *__restrict__ x2,
                                         const double *__restrict__ bvec, double *__restrict__ y, int sub) {
  __shared__ double sm[4];
  if (row >= nrows) return;
  double acc = 0.0;
  for (int64_t c0 = 0; c0 < n1c; c0 += 256 * kGemvUnroll) {
    double mv[kGemvUnroll], xv[kGemvUnroll];
#pragma unroll
    for (int q = 0; q < kGemvUnroll; ++q) {
      const int64_t c = c0 + threadIdx.x + 256 * q;
      mv[q] = c < n1c ? M1[row * n1c + c] : 0.0;
      xv[q] = c < n1c ? x1[c] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < kGemvUnroll; ++q) acc += mv[q] * xv[q];
  }
  if (M2) {
    for (int64_t c0 = 0; c0 < n2c; c0 += 256 * kGemvUnroll) {
      double mv[kGemvUnroll], xv[kGemvUnroll];
#pragma unroll
      for (int q = 0; q < kGemvUnroll; ++q) {
        const int64_t c = c0 + threadIdx.x + 256 * q;
        mv[q] = c < n2c ? M2[row * n2c + c] : 0.0;
        xv[q] = c < n2c ? x2[c] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < kGemvUnroll; ++q) acc -= mv[q] * xv[q];
    }
  }
  const double s = block_sum(acc, sm);
  if (threadIdx.x == 0) y[row] = sub ? bvec[row] - s : s;
}


struct GemvJobs {
  int njobs;
  GemvJob job[2];
};

// One wavefront per output row, four rows per block: a lane keeps up to kRowUnroll
// loads of the row in flight and the row sum is a fixed-order wave reduction
// (no LDS, no barrier).
constexpr int kRowUnroll = 16;
// Each wave takes RPW consecutive rows of one job (the job's last wave may have fewer): the
// x values a lane loads for one chunk of columns serve all of its rows, so x is read from
// L2 once per RPW rows, and a lane keeps RPW * kRowUnroll matrix loads in flight.
template <int RPW>
__global__ void __launch_bounds__(256) gemv_jobs_kernel(const GemvJobs J) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t w0 = (J.job[0].nrows + RPW - 1) / RPW;
  const int64_t w1 = J.njobs > 1 ? (J.job[1].nrows + RPW - 1) / RPW : 0;
  if (wave >= w0 + w1) return;
  const bool second = wave >= w0;  // wave-uniform
  const GemvJob jb = second ? J.job[1] : J.job[0];
  const int64_t row0 = (second ? wave - w0 : wave) * RPW;
  const int nr = (int)(jb.nrows - row0 < RPW ? jb.nrows - row0 : RPW);  // rows of this wave, wave-uniform
  double acc[RPW];
#pragma unroll
  for (int r = 0; r < RPW; ++r) acc[r] = 0.0;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if (q >= jb.nseg) break;
    const GemvSeg g = jb.seg[q];
    const int64_t last = g.ncols - 1;
    double part[RPW];
#pragma unroll
    for (int r = 0; r < RPW; ++r) part[r] = 0.0;
    // loads are unconditional (past the end: the row's last entry, weighted by 0 when
    // summed; a missing row of the last wave re-reads the wave's first row, unused) so a
    // whole chunk is in flight without a branch or wait per load; the factor blocks are
    // streamed once per solve (non-temporal), x is shared by all rows
    auto rows = [&](auto *M) {  // M: the segment's matrix in its storage precision
      for (int64_t c0 = 0; c0 < g.ncols; c0 += 64 * kRowUnroll) {
        double xv[kRowUnroll];
#pragma unroll
        for (int u = 0; u < kRowUnroll; ++u) {
          const int64_t c = c0 + lane + 64 * u;
          xv[u] = g.x[c < last ? c : last];
        }
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
          const int64_t row = row0 + (r < nr ? r : 0);
          double mv[kRowUnroll];
#pragma unroll
          for (int u = 0; u < kRowUnroll; ++u) {
            const int64_t c = c0 + lane + 64 * u;
            mv[u] = (double)__builtin_nontemporal_load(M + row * g.ncols + (c < last ? c : last));
          }
#pragma unroll
          for (int u = 0; u < kRowUnroll; ++u)
            part[r] += (c0 + lane + 64 * u <= last ? 1.0 : 0.0) * (mv[u] * xv[u]);
        }
      }
    };
    if (g.M32) rows(g.M32);  // wave-uniform: single-precision storage, double products and sums
    else rows(g.M);
#pragma unroll
    for (int r = 0; r < RPW; ++r) acc[r] += g.sign * part[r];
  }
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    double a = acc[r];
    for (int off = 32; off > 0; off >>= 1) a += __shfl_down(a, off, 64);
    if (lane == 0 && r < nr) jb.y[row0 + r] = (jb.b ? jb.b[row0 + r] : 0.0) + a;
  }
}

// ------------------------------------------------------------------ reductions
// partials[blk*nd + q] = sum over the block's grid-stride range of x_q . y_q
template <typename T>
__global__ void __launch_bounds__(256)
dots_kernel(int64_t n, int nd, const T *__restrict__ x0, const T *__restrict__ y0,
            const T *__restrict__ x1, const T *__restrict__ y1, const T *__restrict__ x2,
            const T *__restrict__ y2, double *__restrict__ partials) {
  __shared__ double sm[4];
  double a0 = 0, a1 = 0, a2 = 0;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n;
       g += (int64_t)gridDim.x * blockDim.x) {
    a0 += (double)x0[g] * (double)y0[g];
    if (nd > 1) a1 += (double)x1[g] * (double)y1[g];
    if (nd > 2) a2 += (double)x2[g] * (double)y2[g];
  }
  double s = block_sum(a0, sm);
  if (threadIdx.x == 0) partials[blockIdx.x * nd + 0] = s;
  if (nd > 1) {
    s = block_sum(a1, sm);
    if (threadIdx.x == 0) partials[blockIdx.x * nd + 1] = s;
  }
  if (nd > 2) {
    s = block_sum(a2, sm);
    if (threadIdx.x == 0) partials[blockIdx.x * nd + 2] = s;
  }
}

// Sum over b = threadIdx.x, +blockDim.x, ... < nblocks of partials[b*nd + q], in that order,
// with eight loads in flight per round instead of one (reductions with tens of thousands of
// partials are otherwise a chain of dependent memory latencies).
template <int kRound = 8>
__device__ __forceinline__ double strided_partial_sum(const double *__restrict__ partials, int nblocks, int nd,
                                                      int q) {
  double a = 0.0;
  for (int b0 = threadIdx.x; b0 < nblocks; b0 += kRound * blockDim.x) {
    double v[kRound];
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const int bq = b0 + u * blockDim.x;
      v[u] = bq < nblocks ? partials[(int64_t)bq * nd + q] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kRound; ++u) a += v[u];
  }
  return a;
}

// out[slot + q] = sum_b partials[b*nd + q], fixed order; then an optional scalar
// step for the Krylov recurrences (see finalize_op). One block of 1024 threads, each loading
// 16 partials per round: the 32,768 partials of the FP64 operator's p.Ap take two dependent
// rounds (256 threads with 8 per round took 16, about 8 us).
constexpr int kFinThreads = 1024;
__global__ void __launch_bounds__(kFinThreads)
finalize_kernel(int nblocks, int nd, const double *__restrict__ partials, double *__restrict__ scal,
                int slot, int op) {
  __shared__ double sm[kFinThreads / 64];
  __shared__ double res[3];
  for (int q = 0; q < nd; ++q) {
    double v = strided_partial_sum<16>(partials, nblocks, nd, q);
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int w = 0; w < kFinThreads / 64; ++w) t += sm[w];
      res[q] = t;
    }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  for (int q = 0; q < nd; ++q) scal[slot + q] = res[q];
  if (op == FIN_INIT_RZ) {
    // res[0] = r.z of the first iteration: p = z, beta = 0
    scal[S_RZ] = res[0];
    scal[S_BETA] = 0.0;
  } else if (op == FIN_BETA_PCG || op == FIN_BETA_FCG) {
    // res[0] = z.r (new), res[1] = z.r_old (flexible only)
    const double rz_old = scal[S_RZ];
    const double num = (op == FIN_BETA_FCG) ? res[0] - res[1] : res[0];
    scal[S_BETA] = num / rz_old;
    scal[S_RZ] = res[0];
  }
}

// ------------------------------------------------------------------ GMRES vector kernels
// Classical Gram-Schmidt projections V_q . w for all q < k in one pass over w. A thread takes two
// consecutive entries per round (16-byte loads) and the basis in chunks of four vectors, whose
// loads are all requested before the first product (a chunk past k repeats vector k - 1; its sums
// are not stored). KM (8, 16 or 32) bounds k: the sums of 32 vectors would leave two waves per
// SIMD. The former loop tested every vector on its own, so each load waited for the last: 4.66 M
// unknowns, 4.5 vectors on average, 63.0 -> 39.4 us per launch (the update 63.8 -> 44.0).
constexpr int kChunk = 4;
typedef double dbl2 __attribute__((ext_vector_type(2)));
template <int KM>
__global__ void __launch_bounds__(256)
multi_dot_kernel(int64_t n, int k, const double *__restrict__ V, int64_t ldv, const double *__restrict__ w,
                 double *__restrict__ partials) {
  __shared__ double sm[4][KM];
  double acc[KM];
#pragma unroll
  for (int q = 0; q < KM; ++q) acc[q] = 0.0;
  const int64_t pairs = n / 2;
  const dbl2 *w2 = reinterpret_cast<const dbl2 *>(w);
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < pairs; g += (int64_t)gridDim.x * blockDim.x) {
    const dbl2 wg = w2[g];
#pragma unroll
    for (int c = 0; c < KM; c += kChunk) {
      if (c >= k) break;
      dbl2 v[kChunk];
#pragma unroll
      for (int q = 0; q < kChunk; ++q)
        v[q] = reinterpret_cast<const dbl2 *>(V + (int64_t)(c + q < k ? c + q : k - 1) * ldv)[g];
#pragma unroll
      for (int q = 0; q < kChunk; ++q) acc[c + q] += v[q].x * wg.x + v[q].y * wg.y;
    }
  }
  if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < KM; ++q)
      if (q < k) acc[q] += V[q * ldv + n - 1] * w[n - 1];
  }
  // all sums through the waves first, then one barrier for the block
#pragma unroll
  for (int q = 0; q < KM; ++q)
    if (q < k) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) acc[q] += __shfl_down(acc[q], off, 64);
      if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6][q] = acc[q];
    }
  __syncthreads();
  const int q = threadIdx.x;
  if (q < k) partials[(int64_t)blockIdx.x * k + q] = ((sm[0][q] + sm[1][q]) + sm[2][q]) + sm[3][q];
}

__global__ void __launch_bounds__(256)
finalize_many_kernel(int nblocks, int nd, const double *__restrict__ partials, double *__restrict__ out) {
  __shared__ double sm[4];
  const int q = blockIdx.x;
  const double a = strided_partial_sum(partials, nblocks, nd, q);
  const double t = block_sum(a, sm);
  if (threadIdx.x == 0) out[q] = t;
}

// y += sign * sum c_q V_q with the partials of y . y, in the same chunks; VEC = 1 where y is only
// 8-byte aligned (the caller's iterate)
template <int VEC>
__device__ __forceinline__ dbl2 load_pack(const double *p, int64_t g) {
  if constexpr (VEC == 2) return reinterpret_cast<const dbl2 *>(p)[g];
  else return dbl2{p[g], 0.0};
}
template <int VEC>
__global__ void __launch_bounds__(256)
multi_axpy_kernel(int64_t n, int k, const double *__restrict__ V, int64_t ldv, const double *__restrict__ c,
                  double sign, double *__restrict__ y, double *__restrict__ partials) {
  __shared__ double sm[4];
  __shared__ double sc[kMaxRestart];
  if (threadIdx.x < kMaxRestart) sc[threadIdx.x] = threadIdx.x < k ? c[threadIdx.x] : 0.0;
  __syncthreads();
  double acc = 0.0;
  const int64_t packs = n / VEC;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < packs; g += (int64_t)gridDim.x * blockDim.x) {
    const dbl2 yg = load_pack<VEC>(y, g);
    dbl2 t = {0.0, 0.0};
#pragma unroll
    for (int c0 = 0; c0 < kMaxRestart; c0 += kChunk) {
      if (c0 >= k) break;
      dbl2 v[kChunk];
#pragma unroll
      for (int q = 0; q < kChunk; ++q)
        v[q] = load_pack<VEC>(V + (int64_t)(c0 + q < k ? c0 + q : k - 1) * ldv, g);
#pragma unroll
      for (int q = 0; q < kChunk; ++q) {
        if (c0 + q < k) {
          t.x += sc[c0 + q] * v[q].x;
          t.y += sc[c0 + q] * v[q].y;
        }
      }
    }
    dbl2 o;
    o.x = yg.x + sign * t.x;
    o.y = yg.y + sign * t.y;
    if constexpr (VEC == 2) reinterpret_cast<dbl2 *>(y)[g] = o;
    else y[g] = o.x;
    acc += o.x * o.x + o.y * o.y;
  }
  if (VEC == 2 && (n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
    double t = 0.0;
    for (int q = 0; q < k; ++q) t += sc[q] * V[q * ldv + n - 1];
    const double v = y[n - 1] + sign * t;
    y[n - 1] = v;
    acc += v * v;
  }
  if (partials) {
    const double t = block_sum(acc, sm);
    if (threadIdx.x == 0) partials[blockIdx.x] = t;
  }
}

// y = x / sqrt(*nrm2), with the single-precision copy that a mixed cycle starts from (optional)
__global__ void scale_inv_sqrt_kernel(int64_t n, const double *__restrict__ x, const double *__restrict__ nrm2,
                                      double *__restrict__ y, float *__restrict__ y32) {
  const double d = sqrt(*nrm2);
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < n) {
    const double v = x[g] / d;
    y[g] = v;
    if (y32) y32[g] = (float)v;
  }
}

// r = b - w with the partial ||r||^2 and (optional) the single-precision copy of r:
// the residual of multigrid used as the solver, where w = A u.
__global__ void __launch_bounds__(256)
resid_norm_kernel(int64_t n, const double *__restrict__ b, const double *__restrict__ w, double *__restrict__ r,
                  double *__restrict__ partials, float *__restrict__ r32) {
  __shared__ double sm[4];
  double acc = 0.0;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n; g += (int64_t)gridDim.x * blockDim.x) {
    const double rv = b[g] - w[g];
    r[g] = rv;
    if (r32) r32[g] = (float)rv;
    acc += rv * rv;
  }
  const double t = block_sum(acc, sm);
  if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

// The CG iterate update x += alpha p is deferred to the pass that updates p, which reads
// p anyway: r_new = r - alpha w with its norm (alpha = r.z / p.w, kept in scal[S_ALPHA]),
// then x += alpha p and p = z + beta p in one pass, and x += alpha p alone when the
// iteration stops.
__global__ void __launch_bounds__(256)
update_r_kernel(int64_t n, double *__restrict__ scal, const double *__restrict__ r, const double *__restrict__ w,
                double *__restrict__ rnew, double *__restrict__ partials, float *__restrict__ r32) {
  __shared__ double sm[4];
  const double alpha = scal[S_RZ] / scal[S_PW];
  double acc = 0.0;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n; g += (int64_t)gridDim.x * blockDim.x) {
    const double rv = r[g] - alpha * w[g];
    rnew[g] = rv;
    if (r32) r32[g] = (float)rv;
    acc += rv * rv;
  }
  const double s = block_sum(acc, sm);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
  if (blockIdx.x == 0 && threadIdx.x == 0) scal[S_ALPHA] = alpha;
}

// The same residual update with A p given as element-local copies (the operator reduced p . Ap
// itself): r_new = r - alpha * sum of the copies, with the partial ||r_new||^2 per block and the
// optional single-precision copy. Lanes take VEC unknowns 64 apart (see strided_first).
template <int VEC>
__device__ __forceinline__ void
update_r_dss_body(unsigned blk, const Box &b, int64_t n, double *__restrict__ scal, const double *__restrict__ r,
                  const double *__restrict__ wL, double *__restrict__ rnew, double *__restrict__ partial,
                  float *__restrict__ r32) {
  __shared__ double sm[4];
  const double alpha = scal[S_RZ] / scal[S_PW];
  double acc = 0.0;
  const int64_t g0 = strided_first<VEC>(blk);
  if (g0 < n) {
    double rv[VEC], wv[VEC];
#pragma unroll
    for (int q = 0; q < VEC; ++q) rv[q] = (g0 + 64 * q < n) ? r[g0 + 64 * q] : 0.0;
    Ijk cc = ijk_of(b, g0);
#pragma unroll
    for (int q = 0; q < VEC; ++q) {
      wv[q] = (g0 + 64 * q < n) ? dss_ijk(wL, b, cc) : 0.0;
      if (q + 1 < VEC) ijk_advance(b, cc, 64);
    }
#pragma unroll
    for (int q = 0; q < VEC; ++q) {
      if (g0 + 64 * q < n) {
        const double v = rv[q] - alpha * wv[q];
        rnew[g0 + 64 * q] = v;
        if (r32) r32[g0 + 64 * q] = (float)v;
        acc += v * v;
      }
    }
  }
  const double t = block_sum(acc, sm);
  if (threadIdx.x == 0) *partial = t;
  if (blk == 0 && threadIdx.x == 0) scal[S_ALPHA] = alpha;
}

template <int VEC>
__global__ void __launch_bounds__(256)
update_r_dss_kernel(Box b, int64_t n, double *__restrict__ scal, const double *__restrict__ r,
                    const double *__restrict__ wL, double *__restrict__ rnew, double *__restrict__ partials,
                    float *__restrict__ r32) {
  update_r_dss_body<VEC>(blockIdx.x, b, n, scal, r, wL, rnew, partials + blockIdx.x, r32);
}

__global__ void update_xp_kernel(int64_t n, const double *__restrict__ scal, double *__restrict__ x,
                                 const double *__restrict__ z, double *__restrict__ p) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  const double pg = p[g];
  x[g] = x[g] + scal[S_ALPHA] * pg;
  p[g] = z[g] + scal[S_BETA] * pg;
}

// The same with the single-precision cycle's result z (its exact FP64 value is the widened one)
__global__ void update_xp32_kernel(int64_t n, const double *__restrict__ scal, double *__restrict__ x,
                                   const float *__restrict__ z, double *__restrict__ p) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  const double pg = p[g];
  x[g] = x[g] + scal[S_ALPHA] * pg;
  p[g] = (double)z[g] + scal[S_BETA] * pg;
}

__global__ void update_x_kernel(int64_t n, const double *__restrict__ scal, double *__restrict__ x,
                                const double *__restrict__ p) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  x[g] = x[g] + scal[S_ALPHA] * p[g];
}

template <typename TO, typename TI>
__global__ void convert_kernel(int64_t n, const TI *__restrict__ in, TO *__restrict__ out) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < n) out[g] = (TO)in[g];
}

__global__ void axpby_kernel(int64_t n, double a, const double *__restrict__ x, double b,
                             const double *__restrict__ y, double *__restrict__ out) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < n) out[g] = a * x[g] + b * (y ? y[g] : 0.0);
}

template <typename T>
__global__ void zero_kernel(int64_t n, T *__restrict__ out) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < n) out[g] = T(0);
}

__global__ void mul_kernel(int64_t n, const double *__restrict__ a, const double *__restrict__ b,
                           double *__restrict__ out) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < n) out[g] = a[g] * b[g];
}

// ------------------------------------------------------------------ adjoint contraction
// dG[e][c][q] from the element-local gradients of lambda and u (see sem_adjoint_contract).
template <int N>
__global__ void __launch_bounds__(AxShape<N>::block)
adjoint_kernel(Box b, int64_t E, const double *__restrict__ lam, const double *__restrict__ u,
               const double *__restrict__ Dm, double *__restrict__ dG) {
  using S = AxShape<N>;
  constexpr int n1 = S::n1, n3 = n1 * n1 * n1;
  __shared__ double sD[n1 * n1];
  __shared__ double sl[S::epb][n1][n1];
  __shared__ double su[S::epb][n1][n1];
  const int t = threadIdx.x;
  const int le = t / S::tpe;
  const int ij = t - le * S::tpe;
  const int i = ij % n1, j = ij / n1;
  const int64_t e = (int64_t)blockIdx.x * S::epb + le;
  const bool active = (le < S::epb) && (e < E);
  for (int q = t; q < n1 * n1; q += S::block) sD[q] = Dm[q];
  double lreg[n1], ureg[n1];
  int ex = 0, ey = 0, ez = 0;
  if (active) {
    const Exyz ec = elem_xyz(b, e);
    ex = ec.x;
    ey = ec.y;
    ez = ec.z;
  }
  const int I = ex * N + i, J = ey * N + j;
  const bool inIJ = active && I >= 1 && I <= b.nx && J >= 1 && J <= b.ny;
  const int64_t gIJ = (int64_t)(I - 1) + (int64_t)b.nx * (J - 1);
  const int64_t plane = (int64_t)b.nx * b.ny;
#pragma unroll
  for (int k = 0; k < n1; ++k) {
    const int K = ez * N + k;
    const bool in = inIJ && K >= 1 && K <= b.nz;
    lreg[k] = in ? lam[gIJ + plane * (K - 1)] : 0.0;
    ureg[k] = in ? u[gIJ + plane * (K - 1)] : 0.0;
  }
  __syncthreads();
  const int lec = active ? le : 0;
#pragma unroll
  for (int k = 0; k < n1; ++k) {
    if (active) {
      sl[lec][j][i] = lreg[k];
      su[lec][j][i] = ureg[k];
    }
    __syncthreads();
    double lr = 0, ls = 0, lt = 0, ur = 0, us = 0, ut = 0;
#pragma unroll
    for (int l = 0; l < n1; ++l) {
      lr += sD[i * n1 + l] * sl[lec][j][l];
      ls += sD[j * n1 + l] * sl[lec][l][i];
      lt += sD[k * n1 + l] * lreg[l];
      ur += sD[i * n1 + l] * su[lec][j][l];
      us += sD[j * n1 + l] * su[lec][l][i];
      ut += sD[k * n1 + l] * ureg[l];
    }
    if (active) {
      double *o = dG + e * 6 * n3 + (k * n1 + j) * n1 + i;
      o[0 * n3] = -(lr * ur);
      o[1 * n3] = -(lr * us + ls * ur);
      o[2 * n3] = -(lr * ut + lt * ur);
      o[3 * n3] = -(ls * us);
      o[4 * n3] = -(ls * ut + lt * us);
      o[5 * n3] = -(lt * ut);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ batched kernels
// A batched launch covers the active systems of a batch: blocks [begin[k],
// begin[k+1]) of the grid belong to system sys[k] of the launch table, and run the
// same bodies as the single-system kernels on that system's level data.
__device__ __forceinline__ int table_slot(const LaunchTable &t, unsigned b) {
  int lo = 0, hi = t.count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((unsigned)t.begin[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}
__device__ __forceinline__ Box lbox(const BatchLevelDev &L) {
  return Box{L.N, L.nex, L.ney, L.nez, L.nx, L.ny, L.nz, make_fastdiv(L.N)};
}
// order pairs of a batch: the finest level with the one below it, that level with order 1
#define SEMCHEB_BATCH_FINE(X) X(4, 2) X(5, 2) X(6, 3) X(7, 3) X(8, 4) X(9, 4) X(10, 5) X(11, 5) X(12, 6)
#define SEMCHEB_BATCH_MID(X) X(2, 1) X(3, 1) X(4, 1) X(5, 1) X(6, 1)
#define SEMCHEB_BATCH_SYS                                  \
  const int slot_ = table_slot(tab, blockIdx.x);           \
  const BatchSysDev &S = sys[tab.sys[slot_]];              \
  const unsigned blk = blockIdx.x - (unsigned)tab.begin[slot_];

// Operator variants of the batched kernels, numbered as the single-system autotuner's:
// 0 (prefetch, compiler's registers), 1 (no prefetch, min_waves), 2 (prefetch, min_waves),
// 3 (single precision: u tile in LDS, prefetch; FP64: pencils, ordinary factor loads), 4
// (single precision: pencils; FP64: u tile in LDS), 5 (single precision: factors staged in
// LDS by DMA; FP64: pencils, non-temporal factor loads).
// The batched setup times them on the batched launch of every order and level.
template <int N, int V>
struct BVar {
  static constexpr int pf = (V == 0 || V == 2 || V == 3) ? 1 : 0;
  static constexpr int occ = (V == 0 || V == 3) ? 1 : AxShape<N>::min_waves;
  static constexpr int tile = (V == 3 || V == 4) ? 1 : (V == 5 ? 2 : 0);
};

// single-precision operator of a cycle level: src 0 applies to d, 1 to x
template <int N, int V>
__global__ void __launch_bounds__(AxShape<N>::block, (BVar<N, V>::occ))
b_ax32_kernel(LaunchTable tab, const BatchSysDev *__restrict__ sys, int level, int src) {
  SEMCHEB_BATCH_SYS
  const BatchLevelDev &L = S.lev[level];
  const float *u = src == 0 ? L.d : L.x;
  constexpr int TILE = BVar<N, V>::tile, PF = BVar<N, V>::pf;
  // runs of consecutive elements of the system on one XCD, as in the single-system
  // single-precision operator (the block range of a system starts anywhere: its XCDs are
  // shifted, not mixed); order 7: 83.2 -> 78.9 us per batched launch of 64 systems
  // (the FP64 operator keeps launch order, which the single-system FP64 one prefers)
  const unsigned xb = xcd_block(blk, (unsigned)(tab.begin[slot_ + 1] - tab.begin[slot_]));
  if constexpr (TILE == 2) ax_body_dma<N>(xb, lbox(L), L.E, u, L.G, L.D, L.w);
  else if constexpr (V == 4) ax_body_pencil<N, float, uint16_t, GEO_DMA, 0>(xb, lbox(L), L.E, u, L.G, L.D, L.w);
  else if constexpr (TILE == 1) ax_body_tile<N, float, uint16_t, PF>(xb, lbox(L), L.E, u, L.G, L.D, L.w);
  else ax_body<N, float, uint16_t, PF>(xb, lbox(L), L.E, u, L.G, L.D, L.w);
}

// FP64 operator on the finest level applied to the Krylov direction p, with the partial p . Ap of
// every block (pdot: the partials of the launch's first block)
template <int N, int V>
__global__ void __launch_bounds__(AxShape<N>::block, ((V == 3 || V == 5) ? PencilShape<N>::occ : BVar<N, V>::occ))
b_ax64_kernel(LaunchTable tab, const BatchSysDev *__restrict__ sys, double *__restrict__ pdot) {
  SEMCHEB_BATCH_SYS
  const BatchLevelDev &L = S.lev[0];
  constexpr int TILE = BVar<N, V>::tile, PF = BVar<N, V>::pf;
  if constexpr (V == 3 || V == 5)
    ax_body_pencil<N, double, double, GEO_REG, PencilShape<N>::pfk, false, V == 5>(
        blk, lbox(L), L.E, S.p, L.G64, L.D64, L.w64, nullptr, pdot);
  else if constexpr (TILE == 1) ax_body_tile<N, double, double, PF>(blk, lbox(L), L.E, S.p, L.G64, L.D64, L.w64, pdot);
  else ax_body<N, double, double, PF>(blk, lbox(L), L.E, S.p, L.G64, L.D64, L.w64, pdot);
}

// The pencil operator of every order of a level in one launch, the order selected per block. Systems
// of one order are few waves: three launches of orders 5, 7, 9 each end in a thin last wave (and at
// orders 2, 3, 4 do not fill the chip at all), where one launch fills those gaps with the other
// orders' blocks. Registers are those of the largest order (115, still 4 waves per SIMD); LDS is
// sized by the launch to the orders present. Chosen at setup where it is faster than the launches
// per order: 16 systems of orders 5, 7, 9, finest level 33.1 -> 25.6 us, the level below 17.1 -> 6.8 us.
// (The FP64 operator in the same form, orders up to 7 and from 8 on apart, was not: 217 registers.)
template <bool FINE>
__global__ void __launch_bounds__(256, 4)
b_ax32_all_kernel(LaunchTable tab, const BatchSysDev *__restrict__ sys, int src) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  SEMCHEB_BATCH_SYS
  const BatchLevelDev &L = S.lev[FINE ? 0 : 1];
  const float *u = src == 0 ? L.d : L.x;
  const unsigned xb = xcd_block(blk, (unsigned)(tab.begin[slot_ + 1] - tab.begin[slot_]));
#define SEMCHEB_CASE(A, B)                                                                           \
  case A:                                                                                            \
    ax_body_pencil<A, float, uint16_t, GEO_DMA, 0, false, true, BlockShape<A>>(                      \
        xb, lbox(L), L.E, u, L.G, L.D, L.w, nullptr, nullptr, nullptr, smem_raw);                    \
    break;
  if constexpr (FINE) {
    switch (L.N) { SEMCHEB_BATCH_FINE(SEMCHEB_CASE) }
  } else {
    switch (L.N) { SEMCHEB_BATCH_MID(SEMCHEB_CASE) }
  }
#undef SEMCHEB_CASE
}

__global__ void __launch_bounds__(256)
b_cheb_kernel(LaunchTable tab, const BatchSysDev *__restrict__ sys, int level, int pp, int step, int flags,
              int mode) {
  SEMCHEB_BATCH_SYS
  const BatchLevelDev &L = S.lev[level];
  const double *cf = L.coef[pp][step];
  const float cprev = step > 0 ? (float)L.coef[pp][step - 1][2] : 0.0f;  // used with CHEB_X_FROM_D
  cheb_body<float, true, 4>(blk, lbox(L), L.n, L.w, L.b, L.r, L.r, L.d, L.x, L.inv, (float)cf[0], (float)cf[1],
                            (float)cf[2], flags, mode, cprev);
}

// Order transfers: the row bodies of the single-system transfers, compiled for every batched order
// (pairs N -> N/2 on the finest level, N/2 -> 1 below it) and selected per block, so one launch
// serves systems of all orders; run lengths of about 1000 fine values per block, at most 4 elements
// (systems are small: longer runs end ragged; 2800 values and 8 elements were no faster). The
// blocks of a system go to the XCDs in runs: the short rows of neighbouring blocks end inside the
// same cache lines. The residual is formed while the restriction reads. With the orders read at run
// time (one element per block, index divisions by variables) 16 systems of orders 5, 7, 9 with 6.3 K
// elements took 31 us down and 32 us up on the finest level (15 and 6.5 us more for the residuals),
// 10 and 11 us below it; now 25.5 and 15.9 us, 8.2 and 7.3 us.
template <int N>
constexpr int batch_ex() {
  constexpr int e = 1000 / ((N + 1) * (N + 1) * N);
  return e < 1 ? 1 : (e > 4 ? 4 : e);
}

template <bool FINE>
__global__ void __launch_bounds__(256)
b_restrict_kernel(LaunchTable tab, const BatchSysDev *__restrict__ sys) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  float *lds = reinterpret_cast<float *>(smem_raw);
  SEMCHEB_BATCH_SYS
  const unsigned xb = xcd_block(blk, (unsigned)(tab.begin[slot_ + 1] - tab.begin[slot_]));
  const BatchLevelDev &F = S.lev[FINE ? 0 : 1], &C = S.lev[FINE ? 1 : 2];
#define SEMCHEB_CASE(A, B)                                                                                      \
  case A:                                                                                                       \
    restrict_rows_body<float, A, B, batch_ex<A>()>(xb, lbox(F), lbox(C), nullptr, F.J, C.w, F.w, \
                                                   F.b, lds);                                                   \
    break;
  if constexpr (FINE) {
    switch (F.N) { SEMCHEB_BATCH_FINE(SEMCHEB_CASE) }
  } else {
    switch (F.N) { SEMCHEB_BATCH_MID(SEMCHEB_CASE) }
  }
#undef SEMCHEB_CASE
}

// correction added to x; the order-1 level's solution is read in FP64 (its values are rounded to
// single precision as they are read)
template <bool FINE>
__global__ void __launch_bounds__(256)
b_prolong_kernel(LaunchTable tab, const BatchSysDev *__restrict__ sys) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  float *lds = reinterpret_cast<float *>(smem_raw);
  SEMCHEB_BATCH_SYS
  const unsigned xb = xcd_block(blk, (unsigned)(tab.begin[slot_ + 1] - tab.begin[slot_]));
  const BatchLevelDev &F = S.lev[FINE ? 0 : 1], &C = S.lev[FINE ? 1 : 2];
  if constexpr (FINE) {
#define SEMCHEB_CASE(A, B)                                                                                    \
  case A:                                                                                                     \
    prolong_rows_body<float, A, B, batch_ex<A>(), float>(xb, lbox(F), lbox(C), C.x, F.J, F.x, nullptr,      \
                                                         nullptr, nullptr, nullptr, lds);                     \
    break;
    switch (F.N) { SEMCHEB_BATCH_FINE(SEMCHEB_CASE) }
#undef SEMCHEB_CASE
  } else {
#define SEMCHEB_CASE(A, B)                                                                                    \
  case A:                                                                                                     \
    prolong_rows_body<float, A, B, batch_ex<A>(), double>(xb, lbox(F), lbox(C), S.cx, F.J, F.x, nullptr,    \
                                                          nullptr, nullptr, nullptr, lds);                    \
    break;
    switch (F.N) { SEMCHEB_BATCH_MID(SEMCHEB_CASE) }
#undef SEMCHEB_CASE
  }
}

// coarse right-hand side: DSS of the restricted element-local values, kept in FP64 on the order-1
// level, where the dense solve reads it
__global__ void __launch_bounds__(256)
b_dss_kernel(LaunchTable tab, const BatchSysDev *__restrict__ sys, int level) {
  SEMCHEB_BATCH_SYS
  const BatchLevelDev &L = S.lev[level];
  const int64_t g = (int64_t)blk * blockDim.x + threadIdx.x;
  if (g >= L.n) return;
  const float v = dss_at(L.w, lbox(L), g);
  if (level == kBatchLevels - 1) S.cb[g] = (double)v;
  else L.b[g] = v;
}

// exact coarse solve, one block per row of the dense inverse
__global__ void __launch_bounds__(256)
b_coarse_kernel(LaunchTable tab, const BatchSysDev *__restrict__ sys) {
  SEMCHEB_BATCH_SYS
  gemv_row(blk, S.nc, S.nc, S.Minv, S.cb, 0, nullptr, nullptr, nullptr, S.cx, 0);
}

// per-system reduction of nd values per block written by a launch with the same table
__global__ void __launch_bounds__(1024)
b_finalize_kernel(LaunchTable tab, const BatchSysDev *__restrict__ sys, const double *__restrict__ partials,
                  int nd, int slot, int op) {
  __shared__ double sm[16];
  __shared__ double res[3];
  const int k = blockIdx.x;
  double *scal = sys[tab.sys[k]].scal;
  const int b0 = tab.begin[k], b1 = tab.begin[k + 1];
  for (int q = 0; q < nd; ++q) {
    double a = 0.0;
    for (int bq = b0 + (int)threadIdx.x; bq < b1; bq += blockDim.x) a += partials[(int64_t)bq * nd + q];
    const double s = block_sum(a, sm);
    if (threadIdx.x == 0) res[q] = s;
  }
  if (threadIdx.x != 0) return;
  for (int q = 0; q < nd; ++q) scal[slot + q] = res[q];
  if (op == FIN_INIT_RZ) {
    scal[S_RZ] = res[0];
    scal[S_BETA] = 0.0;
  } else if (op == FIN_BETA_PCG || op == FIN_BETA_FCG) {
    const double rz_old = scal[S_RZ];
    const double num = (op == FIN_BETA_FCG) ? res[0] - res[1] : res[0];
    scal[S_BETA] = num / rz_old;
    scal[S_RZ] = res[0];
  }
}

// The Krylov vectors are updated as in the single-system solver (update_r_dss, update_xp32): A p stays
// element-local and is summed where r is updated, the cycle result z stays in single precision (its
// widened value is exact), and u += alpha p waits for the pass that updates p, or for update_x when
// the system stops. Separate w, z and u passes before: 16 systems, 2.9 M unknowns, 28 + 19 + 21 + 16
// us and a widening pass per iteration, now 21 + 20 + 13 us.

// r[0] = b, u = 0, cycle input = b in single precision; partial b . b
__global__ void __launch_bounds__(256)
b_start_kernel(LaunchTable tab, const BatchSysDev *__restrict__ sys, double *__restrict__ partials) {
  __shared__ double sm[4];
  SEMCHEB_BATCH_SYS
  const int64_t n = S.lev[0].n, g0 = strided_first<2>(blk);
  double acc = 0.0;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int64_t g = g0 + 64 * q;
    if (g < n) {
      const double v = S.b[g];
      S.r[0][g] = v;
      S.u[g] = 0.0;
      S.lev[0].b[g] = (float)v;
      acc += v * v;
    }
  }
  const double s = block_sum(acc, sm);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// r[par^1] = r[par] - alpha A p (also in single precision into the cycle input); partial ||r||^2
__global__ void __launch_bounds__(256)
b_update_r_kernel(LaunchTable tab, const BatchSysDev *__restrict__ sys, int par, double *__restrict__ partials) {
  SEMCHEB_BATCH_SYS
  const BatchLevelDev &L = S.lev[0];
  update_r_dss_body<2>(blk, lbox(L), L.n, S.scal, S.r[par], L.w64, S.r[par ^ 1], partials + blockIdx.x, L.b);
}

// partial z . r[par] and, with two, z . r[par^1]
__global__ void __launch_bounds__(256)
b_dots_kernel(LaunchTable tab, const BatchSysDev *__restrict__ sys, int par, int two,
              double *__restrict__ partials) {
  __shared__ double sm[4];
  SEMCHEB_BATCH_SYS
  const int64_t n = S.lev[0].n, g0 = strided_first<4>(blk);
  const float *z = S.lev[0].x;
  const double *r1 = S.r[par], *r2 = S.r[par ^ 1];
  double zv[4], v1[4], v2[4], a0 = 0.0, a1 = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t g = g0 + 64 * q;
    zv[q] = g < n ? (double)z[g] : 0.0;
    v1[q] = g < n ? r1[g] : 0.0;
    v2[q] = two && g < n ? r2[g] : 0.0;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    a0 += zv[q] * v1[q];
    a1 += zv[q] * v2[q];
  }
  const int nd = two ? 2 : 1;
  double s = block_sum(a0, sm);
  if (threadIdx.x == 0) partials[(int64_t)blockIdx.x * nd] = s;
  if (two) {
    s = block_sum(a1, sm);
    if (threadIdx.x == 0) partials[(int64_t)blockIdx.x * nd + 1] = s;
  }
}

// op 0: u += alpha p, p = z + beta p; op 1: p = z; op 2: u += alpha p
__global__ void __launch_bounds__(256)
b_update_xp_kernel(LaunchTable tab, const BatchSysDev *__restrict__ sys, int op) {
  SEMCHEB_BATCH_SYS
  const int64_t n = S.lev[0].n, g0 = strided_first<2>(blk);
  const float *z = S.lev[0].x;
  const double alpha = S.scal[S_ALPHA], beta = S.scal[S_BETA];
  double pv[2], uv[2], zv[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int64_t g = g0 + 64 * q;
    pv[q] = op != 1 && g < n ? S.p[g] : 0.0;
    uv[q] = op != 1 && g < n ? S.u[g] : 0.0;
    zv[q] = op != 2 && g < n ? (double)z[g] : 0.0;
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int64_t g = g0 + 64 * q;
    if (g >= n) continue;
    if (op != 1) S.u[g] = uv[q] + alpha * pv[q];
    if (op == 0) S.p[g] = zv[q] + beta * pv[q];
    else if (op == 1) S.p[g] = zv[q];
  }
}

inline unsigned nblk(int64_t n, int bs = 256) { return (unsigned)((n + bs - 1) / bs); }

inline Box mkbox(const Level &L) { return Box{L.N, L.nex, L.ney, L.nez, L.nx, L.ny, L.nz, make_fastdiv(L.N)}; }

// Events that the next operator launch of this host thread takes as the kernel's own start and
// end timestamps (hipExtLaunchKernelGGL: no markers of their own on the stream), then clears.
thread_local hipEvent_t t_ax_start = nullptr, t_ax_stop = nullptr;
template <typename K, typename... Args>
void ax_launch(K kernel, dim3 grid, dim3 block, hipStream_t s, Args... args) {
  if (t_ax_start) {
    hipExtLaunchKernelGGL(kernel, grid, block, 0, s, t_ax_start, t_ax_stop, 0, args...);
    t_ax_start = t_ax_stop = nullptr;
  } else {
    hipLaunchKernelGGL(kernel, grid, block, 0, s, args...);
  }
}
inline bool al16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

// variant 0: prefetch, compiler's register choice; 1: no prefetch, AxShape::min_waves;
// 2: prefetch, AxShape::min_waves; 3 (FP64) and 5 (FP64), 4 (BF16): one thread per pencil
template <int N, typename T, typename GT>
void launch_ax_n(const Level &L, const T *u, const GT *G, const T *D, T *wL, int variant, hipStream_t s,
                 double *pdot = nullptr) {
  using S = AxShape<N>;
  const unsigned grid = (unsigned)((L.E + S::epb - 1) / S::epb);
  if constexpr (sizeof(GT) == 8) {
    if (variant == 6) {
      ax_launch((ax_local_kernel<N, T, GT, 1, S::min_waves, 5>), dim3(grid), dim3(S::block), s,
                mkbox(L), L.E, u, G, D, wL, pdot);
      return;
    }
  }
  if constexpr (sizeof(GT) == 8) {
    if (variant == 3) {
      ax_launch((ax_local_kernel<N, T, GT, PencilShape<N>::pfk, PencilShape<N>::occ, 7>), dim3(grid), dim3(S::block), s,
                mkbox(L), L.E, u, G, D, wL, pdot);
      return;
    }
    if (variant == 5) {
      ax_launch((ax_local_kernel<N, T, GT, PencilShape<N>::pfk, PencilShape<N>::occ, 3>), dim3(grid), dim3(S::block), s,
                mkbox(L), L.E, u, G, D, wL, pdot);
      return;
    }
  }
  if constexpr (sizeof(GT) == 2 && N == 7) {
    if (variant == 6) {
      ax_launch((ax_local_kernel<N, T, GT, 0, S::min_waves, 4>), dim3(grid), dim3(S::block), s,
                mkbox(L), L.E, u, G, D, wL, pdot);
      return;
    }
  }
  if constexpr (sizeof(GT) == 2) {
    if (variant >= 5) {
      ax_launch((ax_local_kernel<N, T, GT, 0, S::min_waves, 2>), dim3(grid), dim3(S::block), s,
                mkbox(L), L.E, u, G, D, wL, pdot);
      return;
    }
  }
  if (sizeof(GT) == 2 && variant == 3) {
    if constexpr (sizeof(GT) == 2)
      ax_launch((ax_local_kernel<N, T, GT, 1, 1, 1>), dim3(grid), dim3(S::block), s, mkbox(L), L.E, u, G, D, wL, pdot);
  } else if (sizeof(GT) == 2 && variant == 4) {
    if constexpr (sizeof(GT) == 2)
      ax_launch((ax_local_kernel<N, T, GT, 0, S::min_waves, 6>), dim3(grid), dim3(S::block), s,
                mkbox(L), L.E, u, G, D, wL, pdot);
  } else if (variant == 4)
    ax_launch((ax_local_kernel<N, T, GT, 0, S::min_waves, 1>), dim3(grid), dim3(S::block), s,
              mkbox(L), L.E, u, G, D, wL, pdot);
  else if (variant == 1)
    ax_launch((ax_local_kernel<N, T, GT, 0, S::min_waves>), dim3(grid), dim3(S::block), s, mkbox(L),
                       L.E, u, G, D, wL, pdot);
  else if (variant == 2)
    ax_launch((ax_local_kernel<N, T, GT, 1, S::min_waves>), dim3(grid), dim3(S::block), s, mkbox(L),
                       L.E, u, G, D, wL, pdot);
  else
    ax_launch((ax_local_kernel<N, T, GT, 1, 1>), dim3(grid), dim3(S::block), s, mkbox(L), L.E, u, G,
                       D, wL, pdot);
}

template <int N, typename T, bool DOT>
void launch_ax_tri_n(const Level &L, const T *u, const T *tri, const T *gxw, const T *D, T *wL, int variant,
                     hipStream_t s, double *pdot) {
  using S = AxShape<N>;
  const unsigned grid = (unsigned)((L.E + S::epb - 1) / S::epb);
  // the pencil form holds whole lines and the column's edge sums: FP64 asks for 2 waves per
  // SIMD so they fit without spilling
  constexpr int kPencilOcc = sizeof(T) == 8 ? 2 : S::min_waves;
  // the plane loop with the p . Ap sums would spill in FP64 at order 7 with 4 waves, and would lose
  // its third wave at order 12: 3 for both
  constexpr int kLoopOcc = DOT && (N == 7 || N == 12) ? 3 : S::min_waves;
  // from order 10 on launches with the sums take the plane loop of variant 0: the pencils would spill
  // 40 to 93 registers (order 10, 5832 elements, 505 -> 485 us per FP64 iteration; order 12, 4096
  // elements, 743 -> 645), and variant 1 leave order 12 two waves (mixed, 553 -> 506 us)
  if constexpr (!(DOT && N >= 10)) {
    if (variant == 2) {
      hipLaunchKernelGGL((ax_tri_kernel<N, T, kPencilOcc, 1, DOT>), dim3(grid), dim3(S::block), 0, s, mkbox(L), L.E,
                         u, tri, gxw, D, wL, pdot);
      return;
    }
    if (variant == 1) {
      hipLaunchKernelGGL((ax_tri_kernel<N, T, 1, 0, DOT>), dim3(grid), dim3(S::block), 0, s, mkbox(L), L.E, u, tri,
                         gxw, D, wL, pdot);
      return;
    }
  }
  hipLaunchKernelGGL((ax_tri_kernel<N, T, kLoopOcc, 0, DOT>), dim3(grid), dim3(S::block), 0, s, mkbox(L), L.E, u, tri,
                     gxw, D, wL, pdot);
}

template <typename T>
bool launch_ax_tri(const Level &L, const T *u, const T *tri, const T *gxw, const T *D, T *wL, hipStream_t s,
                   double *pdot = nullptr) {
  const int variant = sizeof(T) == 8 ? L.ax_variant64 : L.ax_variant32;
  switch (L.N) {
#define SEMCHEB_AXT_CASE(n) \
  case n:                                                                                     \
    if constexpr (sizeof(T) == 8) {                                                           \
      if (pdot) {                                                                             \
        launch_ax_tri_n<n, T, true>(L, u, tri, gxw, D, wL, variant, s, pdot);                 \
        return true;                                                                          \
      }                                                                                       \
    }                                                                                         \
    launch_ax_tri_n<n, T, false>(L, u, tri, gxw, D, wL, variant, s, nullptr);                 \
    return true;
    SEMCHEB_AXT_CASE(1) SEMCHEB_AXT_CASE(2) SEMCHEB_AXT_CASE(3) SEMCHEB_AXT_CASE(4)
    SEMCHEB_AXT_CASE(5) SEMCHEB_AXT_CASE(6) SEMCHEB_AXT_CASE(7) SEMCHEB_AXT_CASE(8)
    SEMCHEB_AXT_CASE(9) SEMCHEB_AXT_CASE(10) SEMCHEB_AXT_CASE(11) SEMCHEB_AXT_CASE(12)
#undef SEMCHEB_AXT_CASE
    default: return false;
  }
}

template <typename T, typename GT>
bool launch_ax_t(const Level &L, const T *u, const GT *G, const T *D, T *wL, hipStream_t s,
                 double *pdot = nullptr) {
  const int variant = sizeof(T) == 8 ? L.ax_variant64 : L.ax_variant32;
  switch (L.N) {
#define SEMCHEB_AX_CASE(n) \
  case n: launch_ax_n<n, T, GT>(L, u, G, D, wL, variant, s, pdot); return true;
    SEMCHEB_AX_CASE(1) SEMCHEB_AX_CASE(2) SEMCHEB_AX_CASE(3) SEMCHEB_AX_CASE(4)
    SEMCHEB_AX_CASE(5) SEMCHEB_AX_CASE(6) SEMCHEB_AX_CASE(7) SEMCHEB_AX_CASE(8)
    SEMCHEB_AX_CASE(9) SEMCHEB_AX_CASE(10) SEMCHEB_AX_CASE(11) SEMCHEB_AX_CASE(12)
#undef SEMCHEB_AX_CASE
    default: return false;
  }
}

template <int N>
void launch_adj_n(const Level &L, const double *lam, const double *u, double *dG, hipStream_t s) {
  using S = AxShape<N>;
  const unsigned grid = (unsigned)((L.E + S::epb - 1) / S::epb);
  hipLaunchKernelGGL((adjoint_kernel<N>), dim3(grid), dim3(S::block), 0, s, mkbox(L), L.E, lam, u, L.D64, dG);
}

}  // namespace

int ax_elems_per_block(int N) {
  switch (N) {
#define SEMCHEB_EPB(n) \
  case n: return AxShape<n>::epb;
    SEMCHEB_EPB(1) SEMCHEB_EPB(2) SEMCHEB_EPB(3) SEMCHEB_EPB(4) SEMCHEB_EPB(5) SEMCHEB_EPB(6)
    SEMCHEB_EPB(7) SEMCHEB_EPB(8) SEMCHEB_EPB(9) SEMCHEB_EPB(10) SEMCHEB_EPB(11) SEMCHEB_EPB(12)
#undef SEMCHEB_EPB
    default: return 1;
  }
}

// ------------------------------------------------------------------ launchers
bool launch_ax(const Level &L, const double *u, double *wL, hipStream_t s) {
  if (L.tri64) return launch_ax_tri<double>(L, u, L.tri64, L.gxw64, L.D64, wL, s);
  return launch_ax_t<double, double>(L, u, L.G64, L.D64, wL, s);
}
bool launch_ax(const Level &L, const float *u, float *wL, hipStream_t s) {
  if (L.tri32) return launch_ax_tri<float>(L, u, L.tri32, L.gxw32, L.D32, wL, s);
  return launch_ax_t<float, uint16_t>(L, u, L.Gbf, L.D32, wL, s);
}

void set_ax_launch_events(hipEvent_t start, hipEvent_t stop) {
  t_ax_start = start;
  t_ax_stop = stop;
}

int launch_ax_dot(const Level &L, const double *u, double *wL, double *partials, hipStream_t s) {
  if (L.type != LVL_SEM || !(L.tri64 || L.G64)) return 0;
  if (L.tri64 ? !launch_ax_tri<double>(L, u, L.tri64, L.gxw64, L.D64, wL, s, partials)
              : !launch_ax_t<double, double>(L, u, L.G64, L.D64, wL, s, partials))
    return 0;
  return (int)((L.E + ax_elems_per_block(L.N) - 1) / ax_elems_per_block(L.N));
}

int update_r_dss_blocks(int64_t n) { return (int)nblk((n + 1) / 2); }

int launch_update_r_dss(const Level &L, double *scal, const double *r, const double *wL, double *rnew,
                        double *partials, float *r32, hipStream_t s) {
  const int nb = update_r_dss_blocks(L.n);
  hipLaunchKernelGGL((update_r_dss_kernel<2>), dim3(nb), dim3(256), 0, s, mkbox(L), L.n, scal, r, wL, rnew, partials,
                     r32);
  return nb;
}

template <typename T>
void launch_dss(const Level &L, const T *wL, T *out, hipStream_t s) {
  constexpr int VEC = sizeof(T) == 8 ? 2 : 4;
  hipLaunchKernelGGL((dss_kernel<T, T, VEC>), dim3((unsigned)((L.n + 256 * VEC - 1) / (256 * VEC))), dim3(256), 0, s,
                     mkbox(L), L.n, wL, out);
}
template void launch_dss<double>(const Level &, const double *, double *, hipStream_t);
template void launch_dss<float>(const Level &, const float *, float *, hipStream_t);

int dss_dot_blocks(int64_t n) { return (int)nblk((n + 1) / 2); }

int launch_dss_dot(const Level &L, const double *wL, double *out, const double *p, double *partials,
                   hipStream_t s) {
  const int nb = dss_dot_blocks(L.n);
  if (al16(out) && al16(p))
    hipLaunchKernelGGL((dss_dot_kernel<double, 2>), dim3(nb), dim3(256), 0, s, mkbox(L), L.n, wL, out, p,
                       partials);
  else
    hipLaunchKernelGGL((dss_dot_kernel<double, 1>), dim3((unsigned)nblk(L.n)), dim3(256), 0, s, mkbox(L), L.n, wL,
                       out, p, partials);
  return al16(out) && al16(p) ? nb : (int)nblk(L.n);
}


template <typename T, int VEC>
void launch_cheb_v(const Level &L, const T *wsrc, const T *b, const T *r_in, T *r_out, T *d, T *x,
                   const T *invdiag, double a, double bc, double c, int flags, int mode, hipStream_t s,
                   double cprev) {
  const unsigned grid = nblk((L.n + VEC - 1) / VEC);
  if (L.type == LVL_SEM)
    hipLaunchKernelGGL((cheb_kernel<T, true, VEC>), dim3(grid), dim3(256), 0, s, mkbox(L), L.n, wsrc, b, r_in,
                       r_out, d, x, invdiag, (T)a, (T)bc, (T)c, flags, mode, (T)cprev);
  else
    hipLaunchKernelGGL((cheb_kernel<T, false, VEC>), dim3(grid), dim3(256), 0, s, mkbox(L), L.n, wsrc, b, r_in,
                       r_out, d, x, invdiag, (T)a, (T)bc, (T)c, flags, mode, (T)cprev);
}

template <typename T>
void launch_cheb(const Level &L, const T *wsrc, const T *b, const T *r_in, T *r_out, T *d, T *x,
                 const T *invdiag, double a, double bc, double c, int flags, int mode, hipStream_t s,
                 double cprev) {
  if (L.type == LVL_GEN) {
    launch_cheb_lists<T>(L, wsrc, b, r_in, r_out, d, x, invdiag, a, bc, c, flags, mode, s, cprev);
    return;
  }
  // 16-byte packs need every streamed vector 16-byte aligned (device allocations are)
  const bool ok = al16(b) && al16(r_in) && al16(r_out) && al16(d) && al16(x) && al16(invdiag) &&
                  (L.type == LVL_SEM || al16(wsrc));
  if (ok) launch_cheb_v<T, 16 / sizeof(T)>(L, wsrc, b, r_in, r_out, d, x, invdiag, a, bc, c, flags, mode, s, cprev);
  else launch_cheb_v<T, 1>(L, wsrc, b, r_in, r_out, d, x, invdiag, a, bc, c, flags, mode, s, cprev);
}
template void launch_cheb<double>(const Level &, const double *, const double *, const double *, double *,
                                  double *, double *, const double *, double, double, double, int, int,
                                  hipStream_t, double);
template void launch_cheb<float>(const Level &, const float *, const float *, const float *, float *, float *,
                                 float *, const float *, double, double, double, int, int, hipStream_t, double);

template <typename T>
void launch_resid_weight(const Level &L, const T *wL, const T *b, T *rw, hipStream_t s) {
  if (L.type == LVL_GEN) {
    launch_resid_lists<T>(L, wL, b, rw, s);
    return;
  }
  constexpr int VEC = 16 / sizeof(T);
  if (al16(b) && al16(rw))
    hipLaunchKernelGGL((resid_weight_kernel<T, VEC>), dim3(nblk((L.n + VEC - 1) / VEC)), dim3(256), 0, s,
                       mkbox(L), L.n, wL, b, rw);
  else
    hipLaunchKernelGGL((resid_weight_kernel<T, 1>), dim3(nblk(L.n)), dim3(256), 0, s, mkbox(L), L.n, wL, b, rw);
}
template void launch_resid_weight<double>(const Level &, const double *, const double *, double *, hipStream_t);
template void launch_resid_weight<float>(const Level &, const float *, const float *, float *, hipStream_t);

template <typename T, int A, int B, int EX>
void restrict_rows(const Level &F, const Level &C, const T *rw, const T *J, T *rcL, const T *wL, const T *b,
                   hipStream_t s) {
  const unsigned grid = (unsigned)(((F.nex + EX - 1) / EX) * (int64_t)F.ney * F.nez);
  hipLaunchKernelGGL((restrict_rows_kernel<T, A, B, EX>), dim3(grid), dim3(256), 0, s, mkbox(F), mkbox(C), rw, J, rcL,
                     wL, b);
}
template <typename T>
bool launch_restrict_rows(const Level &F, const Level &C, const T *rw, const T *J, T *rcL, const T *wL, const T *b,
                          hipStream_t s) {
#define SEMCHEB_PICK(A, B)                                                                              \
  if (F.N == A && C.N == B) {                                                                           \
    constexpr int ex = rows_ex<A, B, T>();                                                              \
    if (short_runs(F, ex)) restrict_rows<T, A, B, short_ex<ex>()>(F, C, rw, J, rcL, wL, b, s);          \
    else restrict_rows<T, A, B, ex>(F, C, rw, J, rcL, wL, b, s);                                        \
    return true;                                                                                        \
  }
  SEMCHEB_TRANSFER_PAIRS(SEMCHEB_PICK)
#undef SEMCHEB_PICK
  return false;
}

template <typename T>
void launch_restrict(const Level &F, const Level &C, const T *rw, const T *J, T *rcL, hipStream_t s) {
  const int nf = F.N + 1, nc = C.N + 1;
  const size_t lds = sizeof(T) * (size_t)(nf * nc + nf * nf * nf + nf * nf * nc);
  if (launch_restrict_rows<T>(F, C, rw, J, rcL, nullptr, nullptr, s)) return;
  hipLaunchKernelGGL((restrict_kernel<T, 0, 0>), dim3((unsigned)F.E), dim3(128), lds, s, mkbox(F), mkbox(C), F.E,
                     rw, J, rcL);
}

template <typename T>
bool launch_restrict_resid(const Level &F, const Level &C, const T *wL, const T *b, const T *J, T *rcL,
                           hipStream_t s) {
  return launch_restrict_rows<T>(F, C, nullptr, J, rcL, wL, b, s);
}
template bool launch_restrict_resid<double>(const Level &, const Level &, const double *, const double *,
                                            const double *, double *, hipStream_t);
template bool launch_restrict_resid<float>(const Level &, const Level &, const float *, const float *,
                                           const float *, float *, hipStream_t);
template void launch_restrict<double>(const Level &, const Level &, const double *, const double *, double *,
                                      hipStream_t);
template void launch_restrict<float>(const Level &, const Level &, const float *, const float *, float *,
                                     hipStream_t);

template <typename T, int A, int B, int EX>
int prolong_rows(const Level &F, const Level &C, const T *xc, const T *J, T *xf, double *zout, hipStream_t s,
                 const double *dr1, const double *dr2, double *partials, int64_t partials_cap, const double *xc64) {
  const unsigned grid = (unsigned)(((F.nex + EX - 1) / EX) * (int64_t)F.ney * F.nez);
  const bool dots = dr1 && partials && (int64_t)grid * (dr2 ? 2 : 1) <= partials_cap;
  if (!dots) dr1 = dr2 = partials = nullptr;
  if constexpr (sizeof(T) == 4 && B == 1) {
    if (xc64) {
      hipLaunchKernelGGL((prolong_rows_kernel<T, A, B, EX, double>), dim3(grid), dim3(256), 0, s, mkbox(F), mkbox(C),
                         xc64, J, xf, zout, dr1, dr2, partials);
      return dots ? (int)grid : 0;
    }
  }
  hipLaunchKernelGGL((prolong_rows_kernel<T, A, B, EX>), dim3(grid), dim3(256), 0, s, mkbox(F), mkbox(C), xc, J, xf,
                     zout, dr1, dr2, partials);
  return dots ? (int)grid : 0;
}

template <typename T>
int launch_prolong(const Level &F, const Level &C, const T *xc, const T *J, T *xf, double *zout, hipStream_t s,
                   const double *dr1, const double *dr2, double *partials, int64_t partials_cap,
                   const double *xc64) {
  const int nf = F.N + 1, nc = C.N + 1;
  const size_t lds = sizeof(T) * (size_t)(nf * nc + nc * nc * nc + nc * nc * nf + nc * nf * nf);
#define SEMCHEB_PICK(A, B)                                                                                           \
  if (F.N == A && C.N == B) {                                                                                        \
    constexpr int ex = prolong_ex<A, B, T>();                                                                        \
    if (short_runs(F, ex))                                                                                           \
      return prolong_rows<T, A, B, short_ex<ex>()>(F, C, xc, J, xf, zout, s, dr1, dr2, partials, partials_cap, xc64); \
    return prolong_rows<T, A, B, ex>(F, C, xc, J, xf, zout, s, dr1, dr2, partials, partials_cap, xc64);              \
  }
  SEMCHEB_TRANSFER_PAIRS(SEMCHEB_PICK)
#undef SEMCHEB_PICK
  hipLaunchKernelGGL((prolong_kernel<T, 0, 0>), dim3((unsigned)F.E), dim3(128), lds, s, mkbox(F), mkbox(C), F.E, xc,
                     J, xf, zout);
  return 0;
}
template int launch_prolong<double>(const Level &, const Level &, const double *, const double *, double *,
                                    double *, hipStream_t, const double *, const double *, double *, int64_t,
                                    const double *);
template int launch_prolong<float>(const Level &, const Level &, const float *, const float *, float *,
                                   double *, hipStream_t, const double *, const double *, double *, int64_t,
                                   const double *);

bool prolong_rows_available(int nf, int nc) {
#define SEMCHEB_HAS(A, B) \
  if (nf == A && nc == B) return true;
  SEMCHEB_TRANSFER_PAIRS(SEMCHEB_HAS)
#undef SEMCHEB_HAS
  return false;
}

void launch_dss_wide(const Level &L, const float *wL, double *out, hipStream_t s) {
  hipLaunchKernelGGL((dss_kernel<float, double>), dim3(nblk(L.n)), dim3(256), 0, s, mkbox(L), L.n, wL, out);
}

void launch_gemv(int64_t nrows, int64_t ncols, const double *M, const double *x, const double *b, double *y,
                 int sub, hipStream_t s) {
  GemvJob jb{sub ? b : nullptr, y, nrows, 1, {{M, x, ncols, sub ? -1.0 : 1.0}}};
  launch_gemv_jobs(1, &jb, s);
}

void launch_gemv_jobs(int njobs, const GemvJob *jobs, hipStream_t s) {
  GemvJobs J{};
  J.njobs = njobs;
  int64_t rows = 0;
  for (int q = 0; q < njobs; ++q) {
    J.job[q] = jobs[q];
    rows += jobs[q].nrows;
  }
  if (rows == 0) return;
  // two rows per wave (32^3 coarse chain: 0.4 ms less per FP64 solve than one; four rows per
  // wave need 251 VGPRs and were slower)
  constexpr int kRpw = 2;
  const int64_t waves = (jobs[0].nrows + kRpw - 1) / kRpw + (njobs > 1 ? (jobs[1].nrows + kRpw - 1) / kRpw : 0);
  hipLaunchKernelGGL((gemv_jobs_kernel<kRpw>), dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, J);
}

template <typename T>
void launch_dots(int64_t n, int nd, const T *x0, const T *y0, const T *x1, const T *y1, const T *x2,
                 const T *y2, double *partials, int nblocks, hipStream_t s) {
  hipLaunchKernelGGL((dots_kernel<T>), dim3(nblocks), dim3(256), 0, s, n, nd, x0, y0, x1, y1, x2, y2,
                     partials);
}
template void launch_dots<double>(int64_t, int, const double *, const double *, const double *, const double *,
                                  const double *, const double *, double *, int, hipStream_t);

void launch_finalize(int nblocks, int nd, const double *partials, double *scal, int slot, int op,
                     hipStream_t s) {
  hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(kFinThreads), 0, s, nblocks, nd, partials, scal, slot, op);
}


void launch_resid_norm(int64_t n, const double *b, const double *w, double *r, double *partials, int nblocks,
                       float *r32, hipStream_t s) {
  hipLaunchKernelGGL(resid_norm_kernel, dim3(nblocks), dim3(256), 0, s, n, b, w, r, partials, r32);
}

void launch_update_r(int64_t n, double *scal, const double *r, const double *w, double *rnew, double *partials,
                     int nblocks, float *r32, hipStream_t s) {
  hipLaunchKernelGGL(update_r_kernel, dim3(nblocks), dim3(256), 0, s, n, scal, r, w, rnew, partials, r32);
}
void launch_update_xp(int64_t n, const double *scal, double *x, const double *z, double *p, hipStream_t s) {
  hipLaunchKernelGGL(update_xp_kernel, dim3(nblk(n)), dim3(256), 0, s, n, scal, x, z, p);
}
void launch_update_xp32(int64_t n, const double *scal, double *x, const float *z, double *p, hipStream_t s) {
  hipLaunchKernelGGL(update_xp32_kernel, dim3(nblk(n)), dim3(256), 0, s, n, scal, x, z, p);
}
void launch_update_x(int64_t n, const double *scal, double *x, const double *p, hipStream_t s) {
  hipLaunchKernelGGL(update_x_kernel, dim3(nblk(n)), dim3(256), 0, s, n, scal, x, p);
}

void launch_convert(int64_t n, const double *in, float *out, hipStream_t s) {
  hipLaunchKernelGGL((convert_kernel<float, double>), dim3(nblk(n)), dim3(256), 0, s, n, in, out);
}
void launch_convert(int64_t n, const float *in, double *out, hipStream_t s) {
  hipLaunchKernelGGL((convert_kernel<double, float>), dim3(nblk(n)), dim3(256), 0, s, n, in, out);
}

void launch_axpby(int64_t n, double a, const double *x, double b, const double *y, double *out, hipStream_t s) {
  hipLaunchKernelGGL(axpby_kernel, dim3(nblk(n)), dim3(256), 0, s, n, a, x, b, y, out);
}

void launch_multi_dot(int64_t n, int k, const double *V, int64_t ldv, const double *w, double *partials,
                      int nblocks, hipStream_t s) {
  // V and w are the context's own vectors, ldv a multiple of 32: 16-byte aligned
  if (k <= 8) hipLaunchKernelGGL(multi_dot_kernel<8>, dim3(nblocks), dim3(256), 0, s, n, k, V, ldv, w, partials);
  else if (k <= 16)
    hipLaunchKernelGGL(multi_dot_kernel<16>, dim3(nblocks), dim3(256), 0, s, n, k, V, ldv, w, partials);
  else hipLaunchKernelGGL(multi_dot_kernel<32>, dim3(nblocks), dim3(256), 0, s, n, k, V, ldv, w, partials);
}
void launch_finalize_many(int nblocks, int nd, const double *partials, double *out, hipStream_t s) {
  hipLaunchKernelGGL(finalize_many_kernel, dim3(nd), dim3(256), 0, s, nblocks, nd, partials, out);
}
void launch_multi_axpy(int64_t n, int k, const double *V, int64_t ldv, const double *c, double sign, double *y,
                       double *partials, int nblocks, hipStream_t s) {
  if (al16(V) && al16(y))
    hipLaunchKernelGGL(multi_axpy_kernel<2>, dim3(nblocks), dim3(256), 0, s, n, k, V, ldv, c, sign, y, partials);
  else
    hipLaunchKernelGGL(multi_axpy_kernel<1>, dim3(nblocks), dim3(256), 0, s, n, k, V, ldv, c, sign, y, partials);
}
void launch_scale_inv_sqrt(int64_t n, const double *x, const double *nrm2, double *y, float *y32, hipStream_t s) {
  hipLaunchKernelGGL(scale_inv_sqrt_kernel, dim3(nblk(n)), dim3(256), 0, s, n, x, nrm2, y, y32);
}

// two entries per thread up to the fixed grid: small vectors are then not reduced over a thousand
// partials of which most are zero (16,129 unknowns, 10 vectors: 7.7 -> 4.4 us for the projections)
int reduce_blocks(int64_t n) { return (int)std::min<int64_t>(kReduceBlocks, std::max<int64_t>(1, (n + 511) / 512)); }

template <int N, typename T>
void launch_schwarz_local_n(const Level &L, const T *v, const T *Sm, const T *Dinv, T *ye, hipStream_t s) {
  if (L.sw_kind == SW_RAS)
    hipLaunchKernelGGL((schwarz_local_kernel<N, T, true>), dim3((unsigned)L.E), dim3(SwShape<N>::block), 0, s,
                       mkbox(L), L.E, v, Sm, Dinv, ye);
  else
    hipLaunchKernelGGL((schwarz_local_kernel<N, T, false>), dim3((unsigned)L.E), dim3(SwShape<N>::block), 0, s,
                       mkbox(L), L.E, v, Sm, Dinv, ye);
}
template <typename T>
void launch_schwarz_local(const Level &L, const T *v, const T *Sm, const T *Dinv, T *ye, hipStream_t s) {
  switch (L.N) {
#define SEMCHEB_SW_CASE(n) \
  case n: launch_schwarz_local_n<n, T>(L, v, Sm, Dinv, ye, s); break;
    SEMCHEB_SW_CASE(3) SEMCHEB_SW_CASE(4) SEMCHEB_SW_CASE(5) SEMCHEB_SW_CASE(6) SEMCHEB_SW_CASE(7)
    SEMCHEB_SW_CASE(8) SEMCHEB_SW_CASE(9) SEMCHEB_SW_CASE(10) SEMCHEB_SW_CASE(11) SEMCHEB_SW_CASE(12)
#undef SEMCHEB_SW_CASE
    default: break;
  }
}
template void launch_schwarz_local<double>(const Level &, const double *, const double *, const double *, double *,
                                           hipStream_t);
template void launch_schwarz_local<float>(const Level &, const float *, const float *, const float *, float *,
                                          hipStream_t);

template <typename T>
void launch_schwarz_gather(const Level &L, const T *ye, int gmode, T *z, T *r, T *d, T *x, double a, double bc,
                           double c, int flags, hipStream_t s) {
  constexpr int VEC = 16 / sizeof(T);
  const unsigned grid = nblk((L.n + VEC - 1) / VEC);
  if (L.sw_kind == SW_RAS)
    hipLaunchKernelGGL((schwarz_gather_kernel<T, VEC, true>), dim3(grid), dim3(256), 0, s, mkbox(L), L.n, ye, gmode, z,
                       r, d, x, (T)a, (T)bc, (T)c, flags);
  else
    hipLaunchKernelGGL((schwarz_gather_kernel<T, VEC, false>), dim3(grid), dim3(256), 0, s, mkbox(L), L.n, ye, gmode,
                       z, r, d, x, (T)a, (T)bc, (T)c, flags);
}
template void launch_schwarz_gather<double>(const Level &, const double *, int, double *, double *, double *,
                                            double *, double, double, double, int, hipStream_t);
template void launch_schwarz_gather<float>(const Level &, const float *, int, float *, float *, float *,
                                           float *, double, double, double, int, hipStream_t);

template <typename T>
void launch_zero(int64_t n, T *out, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(zero_kernel<T>, dim3(nblk(n)), dim3(256), 0, s, n, out);
}
template void launch_zero<double>(int64_t, double *, hipStream_t);
template void launch_zero<float>(int64_t, float *, hipStream_t);

void launch_mul(int64_t n, const double *a, const double *b, double *out, hipStream_t s) {
  hipLaunchKernelGGL(mul_kernel, dim3(nblk(n)), dim3(256), 0, s, n, a, b, out);
}

bool launch_adjoint(const Level &L, const double *lam, const double *u, double *dG, hipStream_t s) {
  switch (L.N) {
#define SEMCHEB_ADJ_CASE(n) \
  case n: launch_adj_n<n>(L, lam, u, dG, s); return true;
    SEMCHEB_ADJ_CASE(1) SEMCHEB_ADJ_CASE(2) SEMCHEB_ADJ_CASE(3) SEMCHEB_ADJ_CASE(4)
    SEMCHEB_ADJ_CASE(5) SEMCHEB_ADJ_CASE(6) SEMCHEB_ADJ_CASE(7) SEMCHEB_ADJ_CASE(8)
    SEMCHEB_ADJ_CASE(9) SEMCHEB_ADJ_CASE(10) SEMCHEB_ADJ_CASE(11) SEMCHEB_ADJ_CASE(12)
#undef SEMCHEB_ADJ_CASE
    default: return false;
  }
}

}  // namespace semcheb

// ------------------------------------------------------------------ batched launchers
namespace semcheb {
namespace {
inline unsigned tgrid(const LaunchTable &t) { return (unsigned)t.begin[t.count]; }
template <int N>
void b_ax32_n(const LaunchTable &t, const BatchSysDev *sys, int level, int src, int v, hipStream_t s) {
  const dim3 g(tgrid(t)), b(AxShape<N>::block);
  switch (v) {
    case 1: hipLaunchKernelGGL((b_ax32_kernel<N, 1>), g, b, 0, s, t, sys, level, src); break;
    case 2: hipLaunchKernelGGL((b_ax32_kernel<N, 2>), g, b, 0, s, t, sys, level, src); break;
    case 3: hipLaunchKernelGGL((b_ax32_kernel<N, 3>), g, b, 0, s, t, sys, level, src); break;
    case 4: hipLaunchKernelGGL((b_ax32_kernel<N, 4>), g, b, 0, s, t, sys, level, src); break;
    case 5: hipLaunchKernelGGL((b_ax32_kernel<N, 5>), g, b, 0, s, t, sys, level, src); break;
    default: hipLaunchKernelGGL((b_ax32_kernel<N, 0>), g, b, 0, s, t, sys, level, src); break;
  }
}
template <int N>
void b_ax64_n(const LaunchTable &t, const BatchSysDev *sys, int v, double *pdot, hipStream_t s) {
  const dim3 g(tgrid(t)), b(AxShape<N>::block);
  switch (v) {
    case 1: hipLaunchKernelGGL((b_ax64_kernel<N, 1>), g, b, 0, s, t, sys, pdot); break;
    case 2: hipLaunchKernelGGL((b_ax64_kernel<N, 2>), g, b, 0, s, t, sys, pdot); break;
    case 3: hipLaunchKernelGGL((b_ax64_kernel<N, 3>), g, b, 0, s, t, sys, pdot); break;
    case 4: hipLaunchKernelGGL((b_ax64_kernel<N, 4>), g, b, 0, s, t, sys, pdot); break;
    case 5: hipLaunchKernelGGL((b_ax64_kernel<N, 5>), g, b, 0, s, t, sys, pdot); break;
    default: hipLaunchKernelGGL((b_ax64_kernel<N, 0>), g, b, 0, s, t, sys, pdot); break;
  }
}
}  // namespace

int batch_ax_elements_per_block(int N) {
  switch (N) {
#define SEMCHEB_EPB(n) \
  case n: return AxShape<n>::epb;
    SEMCHEB_EPB(1) SEMCHEB_EPB(2) SEMCHEB_EPB(3) SEMCHEB_EPB(4) SEMCHEB_EPB(5) SEMCHEB_EPB(6)
    SEMCHEB_EPB(7) SEMCHEB_EPB(8) SEMCHEB_EPB(9) SEMCHEB_EPB(10) SEMCHEB_EPB(11) SEMCHEB_EPB(12)
#undef SEMCHEB_EPB
    default: return 1;
  }
}

int batch_ax_shared(int N, size_t *lds) {
#define SEMCHEB_CASE(A)                                            \
  case A:                                                          \
    *lds = PencilLds<A, float, true, BlockShape<A>>::bytes;        \
    return BlockShape<A>::epb;
  switch (N) {
    SEMCHEB_CASE(2) SEMCHEB_CASE(3) SEMCHEB_CASE(4) SEMCHEB_CASE(5) SEMCHEB_CASE(6) SEMCHEB_CASE(7)
    SEMCHEB_CASE(8) SEMCHEB_CASE(9) SEMCHEB_CASE(10) SEMCHEB_CASE(11) SEMCHEB_CASE(12)
    default: *lds = 0; return 1;
  }
#undef SEMCHEB_CASE
}

BatchTransfer batch_transfer(int N, bool finest) {
#define SEMCHEB_CASE(A, B)                                                                       \
  case A:                                                                                        \
    return {batch_ex<A>(), sizeof(float) * RowsLds<A, B, batch_ex<A>()>::down,                   \
            sizeof(float) * RowsLds<A, B, batch_ex<A>()>::up};
  if (finest) {
    switch (N) { SEMCHEB_BATCH_FINE(SEMCHEB_CASE) default: break; }
  } else {
    switch (N) { SEMCHEB_BATCH_MID(SEMCHEB_CASE) default: break; }
  }
#undef SEMCHEB_CASE
  return {1, 0, 0};
}

// batched orders: finest levels 4..12, the level below 2..6 (the order-1 level is solved densely)
// batched kernel launches issued so far (all contexts; a batched solve reports the difference)
std::atomic<int64_t> g_batched_launches{0};
int64_t batched_launch_count() { return g_batched_launches.load(); }

bool launch_b_ax32(int N, int variant, const LaunchTable &t, const BatchSysDev *sys, int level, int src,
                   hipStream_t s) {
  if (t.count == 0) return true;
  ++g_batched_launches;
  switch (N) {
#define SEMCHEB_BAX(n) \
  case n: b_ax32_n<n>(t, sys, level, src, variant, s); return true;
    SEMCHEB_BAX(2) SEMCHEB_BAX(3) SEMCHEB_BAX(4) SEMCHEB_BAX(5) SEMCHEB_BAX(6)
    SEMCHEB_BAX(7) SEMCHEB_BAX(8) SEMCHEB_BAX(9) SEMCHEB_BAX(10) SEMCHEB_BAX(11) SEMCHEB_BAX(12)
#undef SEMCHEB_BAX
    default: return false;
  }
}

bool launch_b_ax64(int N, int variant, const LaunchTable &t, const BatchSysDev *sys, double *pdot, hipStream_t s) {
  if (t.count == 0) return true;
  ++g_batched_launches;
  switch (N) {
#define SEMCHEB_BAX(n) \
  case n: b_ax64_n<n>(t, sys, variant, pdot, s); return true;
    SEMCHEB_BAX(4) SEMCHEB_BAX(5) SEMCHEB_BAX(6) SEMCHEB_BAX(7) SEMCHEB_BAX(8) SEMCHEB_BAX(9) SEMCHEB_BAX(10)
    SEMCHEB_BAX(11) SEMCHEB_BAX(12)
#undef SEMCHEB_BAX
    default: return false;
  }
}

void launch_b_ax32_all(const LaunchTable &t, const BatchSysDev *sys, int level, int src, size_t lds, hipStream_t s) {
  if (t.count == 0) return;
  ++g_batched_launches;
  if (level == 0) hipLaunchKernelGGL((b_ax32_all_kernel<true>), dim3(tgrid(t)), dim3(256), lds, s, t, sys, src);
  else hipLaunchKernelGGL((b_ax32_all_kernel<false>), dim3(tgrid(t)), dim3(256), lds, s, t, sys, src);
}
void launch_b_cheb(const LaunchTable &t, const BatchSysDev *sys, int level, int pp, int step, int flags, int mode,
                   hipStream_t s) {
  if (t.count) {
    ++g_batched_launches;
    hipLaunchKernelGGL(b_cheb_kernel, dim3(tgrid(t)), dim3(256), 0, s, t, sys, level, pp, step, flags, mode);
  }
}
void launch_b_restrict(const LaunchTable &t, const BatchSysDev *sys, int level, size_t lds, hipStream_t s) {
  if (t.count) {
    ++g_batched_launches;
    if (level == 0) hipLaunchKernelGGL((b_restrict_kernel<true>), dim3(tgrid(t)), dim3(256), lds, s, t, sys);
    else hipLaunchKernelGGL((b_restrict_kernel<false>), dim3(tgrid(t)), dim3(256), lds, s, t, sys);
  }
}
void launch_b_dss(const LaunchTable &t, const BatchSysDev *sys, int level, hipStream_t s) {
  if (t.count) {
    ++g_batched_launches;
    hipLaunchKernelGGL(b_dss_kernel, dim3(tgrid(t)), dim3(256), 0, s, t, sys, level);
  }
}
void launch_b_prolong(const LaunchTable &t, const BatchSysDev *sys, int level, size_t lds, hipStream_t s) {
  if (t.count) {
    ++g_batched_launches;
    if (level == 0) hipLaunchKernelGGL((b_prolong_kernel<true>), dim3(tgrid(t)), dim3(256), lds, s, t, sys);
    else hipLaunchKernelGGL((b_prolong_kernel<false>), dim3(tgrid(t)), dim3(256), lds, s, t, sys);
  }
}
void launch_b_coarse(const LaunchTable &t, const BatchSysDev *sys, hipStream_t s) {
  if (t.count) {
    ++g_batched_launches;
    hipLaunchKernelGGL(b_coarse_kernel, dim3(tgrid(t)), dim3(256), 0, s, t, sys);
  }
}
void launch_b_finalize(const LaunchTable &t, const BatchSysDev *sys, const double *partials, int nd, int slot, int op,
                       hipStream_t s) {
  if (t.count) {
    ++g_batched_launches;
    hipLaunchKernelGGL(b_finalize_kernel, dim3((unsigned)t.count), dim3(1024), 0, s, t, sys, partials, nd, slot, op);
  }
}
void launch_b_start(const LaunchTable &t, const BatchSysDev *sys, double *partials, hipStream_t s) {
  if (t.count) {
    ++g_batched_launches;
    hipLaunchKernelGGL(b_start_kernel, dim3(tgrid(t)), dim3(256), 0, s, t, sys, partials);
  }
}
void launch_b_update_r(const LaunchTable &t, const BatchSysDev *sys, int par, double *partials, hipStream_t s) {
  if (t.count) {
    ++g_batched_launches;
    hipLaunchKernelGGL(b_update_r_kernel, dim3(tgrid(t)), dim3(256), 0, s, t, sys, par, partials);
  }
}
void launch_b_dots(const LaunchTable &t, const BatchSysDev *sys, int par, int two, double *partials, hipStream_t s) {
  if (t.count) {
    ++g_batched_launches;
    hipLaunchKernelGGL(b_dots_kernel, dim3(tgrid(t)), dim3(256), 0, s, t, sys, par, two, partials);
  }
}
void launch_b_update_xp(const LaunchTable &t, const BatchSysDev *sys, int op, hipStream_t s) {
  if (t.count) {
    ++g_batched_launches;
    hipLaunchKernelGGL(b_update_xp_kernel, dim3(tgrid(t)), dim3(256), 0, s, t, sys, op);
  }
}
}  // namespace semcheb
