// Kernels of unstructured hexahedral meshes. As on a box, operator results stay element-local
// ([e][k][j][i]) and the kernel that uses them sums the copies of an unknown, here through copy
// lists (see CopyLists) in increasing local index: no atomics, reproducible sums, and no launch
// that only sums. Inputs of the operator and of the transfers are gathered through the
// local-to-global map. 12^3 elements at N = 7, mixed solve: 53 launches and 295 us per iteration
// with separate summation, gather and interpolation launches, 32 launches and 180 us with them
// inside the kernels that use their results.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_ops.h"

namespace semcheb {
namespace {
using namespace dev;

inline unsigned nblk(int64_t n, int bs = 256) { return (unsigned)((n + bs - 1) / bs); }

// Operator: the pencil body with the column gathered through the map (the lattice fields of b are
// unused); 12^3 elements at N = 7: BF16 factors 13.2 -> 7.9 us, FP64 16.7 -> 13.4 us per launch
// against the plane loop of ax_body.
template <int N>
__global__ void __launch_bounds__(AxShape<N>::block, PencilShape<N>::occ)
ax_map64_kernel(Box b, int64_t E, const int32_t *__restrict__ map, const double *__restrict__ u,
                const double *__restrict__ G, const double *__restrict__ Dm, double *__restrict__ wL,
                double *__restrict__ pdot) {
  ax_body_pencil<N, double, double, GEO_REG, PencilShape<N>::pfk, true>(blockIdx.x, b, E, u, G, Dm, wL, map, pdot);
}
template <int N>
__global__ void __launch_bounds__(AxShape<N>::block, AxShape<N>::min_waves)
ax_map32_kernel(Box b, int64_t E, const int32_t *__restrict__ map, const float *__restrict__ u,
                const uint16_t *__restrict__ G, const float *__restrict__ Dm, float *__restrict__ wL) {
  ax_body_pencil<N, float, uint16_t, GEO_DMA, 0, true>(xcd_block(blockIdx.x, gridDim.x), b, E, u, G, Dm, wL, map);
}

// Sum of the copies of unknown g. Two thirds of the unknowns of a high-order element are interior and
// have one copy, so the further ones are read only where a second exists: two copies' second together
// with the slots of more, then the slots' values. The slots of consecutive shared unknowns are
// consecutive: as one list per unknown (7 entries at its own offset) they made cycles of 0.3 M
// unknowns 3 to 12 % slower; as slots of every unknown they took 32 bytes or more of each (order 7,
// 12^3 elements, FP64 cycle 123.0 -> 120.0 us with these).
template <typename T>
__device__ __forceinline__ T list_sum(const T *__restrict__ w, const CopyLists &S, int64_t g) {
  const int32_t i0 = S.first[g], i1 = S.second[g];
  T s = w[i0];
  if (i1 != -1) {
    const bool shared = i1 < 0;
    int32_t j[kCopySlots];
    T v[kCopySlots];
#pragma unroll
    for (int k = 0; k < kCopySlots; ++k) j[k] = shared ? S.more[k * S.ld + (-2 - i1)] : -1;
    const T v1 = shared ? T(0) : w[i1];
    s += v1;
#pragma unroll
    for (int k = 0; k < kCopySlots; ++k) v[k] = j[k] >= 0 ? w[j[k]] : T(0);
#pragma unroll
    for (int k = 0; k < kCopySlots; ++k) s += v[k];
    if (j[kCopySlots - 1] < -1) {
      const int32_t *t = S.tail + (-2 - j[kCopySlots - 1]);
      int32_t i;
      do {
        i = *t++;
        s += w[i >= 0 ? i : ~i];
      } while (i >= 0);
    }
  }
  return s;
}

template <typename T, typename TO>
__global__ void __launch_bounds__(256)
sum_lists_kernel(int64_t n, CopyLists S, const T *__restrict__ wL, TO *__restrict__ out) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < n) out[g] = (TO)list_sum(wL, S, g);
}

// Chebyshev step with the summation of A d (the flags of cheb_kernel)
template <typename T, int VEC>
__global__ void __launch_bounds__(256)
cheb_lists_kernel(int64_t n, CopyLists S, const T *__restrict__ wL, const T *__restrict__ bvec,
                  const T *__restrict__ r_in, T *__restrict__ r_out, T *__restrict__ d, T *__restrict__ x,
                  const T *__restrict__ invdiag, T a, T bc, T c, int flags, int mode, T cprev) {
  const int64_t g0 = strided_first<VEC>(blockIdx.x);
  if (g0 >= n) return;
  const T *rsrc = (flags & CHEB_R_FROM_B) ? bvec : r_in;
  T sv[VEC], rr[VEC], dd[VEC], xx[VEC], ad[VEC];
#pragma unroll
  for (int q = 0; q < VEC; ++q) {
    const int64_t g = g0 + 64 * q;
    const bool ok = g < n;
    sv[q] = ok ? invdiag[g] : T(0);
    rr[q] = ok ? rsrc[g] : T(0);
    dd[q] = (ok && !(flags & CHEB_D_INIT)) ? d[g] : T(0);
    xx[q] = (ok && !(flags & (CHEB_X_INIT | CHEB_X_FROM_D))) ? x[g] : T(0);
    ad[q] = (ok && (flags & CHEB_SUB_AD)) ? list_sum(wL, S, g) : T(0);
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

// rw = (b - sum of the copies of wL) / number of copies, or b / number of copies without wL: what
// the restriction gathers
template <typename T>
__global__ void __launch_bounds__(256)
resid_lists_kernel(int64_t n, CopyLists S, const T *__restrict__ wL, const T *__restrict__ b,
                   const T *__restrict__ winv, T *__restrict__ rw) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  T v = b[g];
  const T wi = winv[g];
  if (wL) v -= list_sum(wL, S, g);
  rw[g] = v * wi;
}

// r_new = r - alpha * sum of the copies of A p, its norm's partials and its single-precision copy
// (see update_r_dss_kernel)
__global__ void __launch_bounds__(256)
update_r_lists_kernel(int64_t n, CopyLists S, double *__restrict__ scal, const double *__restrict__ r,
                      const double *__restrict__ wL, double *__restrict__ rnew, double *__restrict__ partials,
                      float *__restrict__ r32) {
  const double alpha = scal[S_RZ] / scal[S_PW];
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double acc = 0.0;
  if (g < n) {
    const double v = r[g] - alpha * list_sum(wL, S, g);
    rnew[g] = v;
    if (r32) r32[g] = (float)v;
    acc = v * v;
  }
  block_sum_store(acc, partials + blockIdx.x);
  if (blockIdx.x == 0 && threadIdx.x == 0) scal[S_ALPHA] = alpha;
}

// ------------------------------------------------------------------ order transfers, one element per block
constexpr int kTransferThreads = 128;

// Restriction: the weighted residual gathered through the fine map, contracted with J^T along i,
// j, k into element-local coarse values. NF, NC > 0: orders known at compile time.
template <typename T, int NF, int NC>
__global__ void __launch_bounds__(kTransferThreads)
restrict_map_kernel(int Nf, int Nc, const int32_t *__restrict__ map, const T *__restrict__ rw,
                    const T *__restrict__ Jm, T *__restrict__ rcL) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int nf = NF > 0 ? NF + 1 : Nf + 1, nc = NC > 0 ? NC + 1 : Nc + 1;
  T *sJ = reinterpret_cast<T *>(smem_raw);  // nf * nc
  T *sf = sJ + nf * nc;                     // nf^3, later nf * nc * nc
  T *t1 = sf + nf * nf * nf;                // nf * nf * nc
  const int64_t e = blockIdx.x;
  for (int q = threadIdx.x; q < nf * nc; q += kTransferThreads) sJ[q] = Jm[q];
  for (int q = threadIdx.x; q < nf * nf * nf; q += kTransferThreads) {
    const int32_t g = map[e * nf * nf * nf + q];
    const T v = rw[g >= 0 ? g : 0];
    sf[q] = g >= 0 ? v : T(0);
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nf * nf * nc; q += kTransferThreads) {
    const int a = q % nc, kj = q / nc;
    T s = 0;
    for (int i = 0; i < nf; ++i) s += sJ[i * nc + a] * sf[kj * nf + i];
    t1[kj * nc + a] = s;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nf * nc * nc; q += kTransferThreads) {
    const int a = q % nc, bq = (q / nc) % nc, k = q / (nc * nc);
    T s = 0;
    for (int j = 0; j < nf; ++j) s += sJ[j * nc + bq] * t1[(k * nf + j) * nc + a];
    sf[(k * nc + bq) * nc + a] = s;
  }
  __syncthreads();
  T *out = rcL + e * nc * nc * nc;
  for (int q = threadIdx.x; q < nc * nc * nc; q += kTransferThreads) {
    const int ba = q % (nc * nc), c = q / (nc * nc);
    T s = 0;
    for (int k = 0; k < nf; ++k) s += sJ[k * nc + c] * sf[k * nc * nc + ba];
    out[q] = s;
  }
}

// Prolongation x += P x_c: every element interpolates the coarse values and updates the unknowns it
// owns (omap: the unknown where this element holds its first copy, -1 elsewhere; the other copies
// interpolate the same values). zout: the widened result instead of x. dr1, dr2: the partial sums
// of the result with these vectors, one (two) per block.
template <typename T, int NF, int NC, typename TC>
__global__ void __launch_bounds__(kTransferThreads)
prolong_map_kernel(int Nf, int Nc, const int32_t *__restrict__ cmap, const int32_t *__restrict__ omap,
                   const TC *__restrict__ xc, const T *__restrict__ Jm, T *__restrict__ xf, double *__restrict__ zout,
                   const double *__restrict__ dr1, const double *__restrict__ dr2, double *__restrict__ partials) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int nf = NF > 0 ? NF + 1 : Nf + 1, nc = NC > 0 ? NC + 1 : Nc + 1;
  T *sJ = reinterpret_cast<T *>(smem_raw);  // nf * nc
  T *sc = sJ + nf * nc;                     // nc^3
  T *t1 = sc + nc * nc * nc;                // nc * nc * nf
  T *t2 = t1 + nc * nc * nf;                // nc * nf * nf
  const int64_t e = blockIdx.x;
  const int n3 = nf * nf * nf;
  for (int q = threadIdx.x; q < nf * nc; q += kTransferThreads) sJ[q] = Jm[q];
  for (int q = threadIdx.x; q < nc * nc * nc; q += kTransferThreads) {
    const int32_t g = cmap[e * nc * nc * nc + q];
    const T v = (T)xc[g >= 0 ? g : 0];
    sc[q] = g >= 0 ? v : T(0);
  }
  // the owned unknowns of a thread's share, requested before the contractions
  constexpr int kIt = NF > 0 ? ((NF + 1) * (NF + 1) * (NF + 1) + kTransferThreads - 1) / kTransferThreads : 1;
  constexpr bool kPre = NF > 0 && kIt <= 8;
  [[maybe_unused]] int32_t go[kPre ? kIt : 1];
  [[maybe_unused]] T xo[kPre ? kIt : 1];
  if constexpr (kPre) {
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
      const int q = threadIdx.x + kTransferThreads * it;
      go[it] = q < n3 ? omap[e * n3 + q] : -1;
    }
#pragma unroll
    for (int it = 0; it < kIt; ++it) xo[it] = xf[go[it] >= 0 ? go[it] : 0];
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nc * nc * nf; q += kTransferThreads) {
    const int i = q % nf, cb = q / nf;
    T s = 0;
    for (int a = 0; a < nc; ++a) s += sJ[i * nc + a] * sc[cb * nc + a];
    t1[cb * nf + i] = s;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nc * nf * nf; q += kTransferThreads) {
    const int i = q % nf, j = (q / nf) % nf, c = q / (nf * nf);
    T s = 0;
    for (int bq = 0; bq < nc; ++bq) s += sJ[j * nc + bq] * t1[(c * nc + bq) * nf + i];
    t2[(c * nf + j) * nf + i] = s;
  }
  __syncthreads();
  double d1 = 0.0, d2 = 0.0;
  auto finish = [&](int q, int32_t g, T xl) {
    const int ji = q % (nf * nf), k = q / (nf * nf);
    T s = 0;
    for (int c = 0; c < nc; ++c) s += sJ[k * nc + c] * t2[c * nf * nf + ji];
    const T xv = xl + s;
    if (zout) zout[g] = (double)xv;
    else xf[g] = xv;
    if (dr1) d1 += (double)xv * dr1[g];
    if (dr2) d2 += (double)xv * dr2[g];
  };
  if constexpr (kPre) {
#pragma unroll
    for (int it = 0; it < kIt; ++it)
      if (go[it] >= 0) finish(threadIdx.x + kTransferThreads * it, go[it], xo[it]);
  } else {
    for (int q = threadIdx.x; q < n3; q += kTransferThreads) {
      const int32_t g = omap[e * n3 + q];
      if (g >= 0) finish(q, g, xf[g]);
    }
  }
  if (dr1) {
    const int nd = dr2 ? 2 : 1;
    block_sum_store(d1, partials + (int64_t)blockIdx.x * nd);
    if (dr2) {
      __syncthreads();  // block_sum_store reuses its LDS
      block_sum_store(d2, partials + (int64_t)blockIdx.x * nd + 1);
    }
  }
}

template <int N>
void ax_map64(const Level &L, const double *u, double *wL, double *pdot, hipStream_t s) {
  using S = AxShape<N>;
  const Box b{N, 1, 1, 1, 1, 1, 1, make_fastdiv(N)};
  hipLaunchKernelGGL((ax_map64_kernel<N>), dim3((unsigned)((L.E + S::epb - 1) / S::epb)), dim3(S::block), 0, s, b, L.E,
                     L.map, u, L.G64, L.D64, wL, pdot);
}
template <int N>
void ax_map32(const Level &L, const float *u, float *wL, hipStream_t s) {
  using S = AxShape<N>;
  const Box b{N, 1, 1, 1, 1, 1, 1, make_fastdiv(N)};
  hipLaunchKernelGGL((ax_map32_kernel<N>), dim3((unsigned)((L.E + S::epb - 1) / S::epb)), dim3(S::block), 0, s, b, L.E,
                     L.map, u, L.Gbf, L.D32, wL);
}
#define SEMCHEB_ORDERS(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12)

bool launch_map64(const Level &L, const double *u, double *wL, double *pdot, hipStream_t s) {
  switch (L.N) {
#define SEMCHEB_CASE(n) \
  case n: ax_map64<n>(L, u, wL, pdot, s); return true;
    SEMCHEB_ORDERS(SEMCHEB_CASE)
#undef SEMCHEB_CASE
    default: return false;
  }
}

}  // namespace

bool launch_ax_map(const Level &L, const double *u, double *wL, hipStream_t s) {
  return launch_map64(L, u, wL, nullptr, s);
}
int launch_ax_map_dot(const Level &L, const double *u, double *wL, double *partials, hipStream_t s) {
  if (!launch_map64(L, u, wL, partials, s)) return 0;
  const int epb = ax_elems_per_block(L.N);
  return (int)((L.E + epb - 1) / epb);
}
bool launch_ax_map(const Level &L, const float *u, float *wL, hipStream_t s) {
  switch (L.N) {
#define SEMCHEB_CASE(n) \
  case n: ax_map32<n>(L, u, wL, s); return true;
    SEMCHEB_ORDERS(SEMCHEB_CASE)
#undef SEMCHEB_CASE
    default: return false;
  }
}

template <typename T, typename TO>
void launch_sum_lists(const Level &L, const T *wL, TO *out, hipStream_t s) {
  hipLaunchKernelGGL((sum_lists_kernel<T, TO>), dim3(nblk(L.n)), dim3(256), 0, s, L.n, L.copies, wL, out);
}
template void launch_sum_lists<double, double>(const Level &, const double *, double *, hipStream_t);
template void launch_sum_lists<float, float>(const Level &, const float *, float *, hipStream_t);
template void launch_sum_lists<float, double>(const Level &, const float *, double *, hipStream_t);

template <typename T>
void launch_cheb_lists(const Level &L, const T *wL, const T *b, const T *r_in, T *r_out, T *d, T *x, const T *invdiag,
                       double a, double bc, double c, int flags, int mode, hipStream_t s, double cprev) {
  // two unknowns per thread once one per thread fills the chip (2.4 M unknowns of order 9: FP64 cycle
  // 333 -> 328 us; 3 M of orders 10 and 12 and 2.7 M of order 7 within 0.7 %, never slower)
  const bool two = L.n >= (int64_t)2048 * 1024;
  if (two)
    hipLaunchKernelGGL((cheb_lists_kernel<T, 2>), dim3(nblk((L.n + 1) / 2)), dim3(256), 0, s, L.n, L.copies, wL, b,
                       r_in, r_out, d, x, invdiag, (T)a, (T)bc, (T)c, flags, mode, (T)cprev);
  else
    hipLaunchKernelGGL((cheb_lists_kernel<T, 1>), dim3(nblk(L.n)), dim3(256), 0, s, L.n, L.copies, wL, b, r_in, r_out,
                       d, x, invdiag, (T)a, (T)bc, (T)c, flags, mode, (T)cprev);
}
template void launch_cheb_lists<double>(const Level &, const double *, const double *, const double *, double *,
                                        double *, double *, const double *, double, double, double, int, int,
                                        hipStream_t, double);
template void launch_cheb_lists<float>(const Level &, const float *, const float *, const float *, float *, float *,
                                       float *, const float *, double, double, double, int, int, hipStream_t, double);

template <typename T>
void launch_resid_lists(const Level &L, const T *wL, const T *b, T *rw, hipStream_t s) {
  const T *winv;
  if constexpr (sizeof(T) == 8) winv = L.winv64;
  else winv = L.winv32;
  hipLaunchKernelGGL((resid_lists_kernel<T>), dim3(nblk(L.n)), dim3(256), 0, s, L.n, L.copies, wL, b, winv, rw);
}
template void launch_resid_lists<double>(const Level &, const double *, const double *, double *, hipStream_t);
template void launch_resid_lists<float>(const Level &, const float *, const float *, float *, hipStream_t);

template <typename T>
void launch_restrict_map(const Level &F, const Level &C, const T *rw, const T *J, T *rcL, hipStream_t s) {
  const int nf = F.N + 1, nc = C.N + 1;
  const size_t lds = sizeof(T) * (size_t)(nf * nc + nf * nf * nf + nf * nf * nc);
#define SEMCHEB_PICK(A, B)                                                                                         \
  if (F.N == A && C.N == B) {                                                                                      \
    hipLaunchKernelGGL((restrict_map_kernel<T, A, B>), dim3((unsigned)F.E), dim3(kTransferThreads), lds, s, F.N,   \
                       C.N, F.map, rw, J, rcL);                                                                    \
    return;                                                                                                        \
  }
  SEMCHEB_TRANSFER_PAIRS(SEMCHEB_PICK)
#undef SEMCHEB_PICK
  hipLaunchKernelGGL((restrict_map_kernel<T, 0, 0>), dim3((unsigned)F.E), dim3(kTransferThreads), lds, s, F.N, C.N,
                     F.map, rw, J, rcL);
}
template void launch_restrict_map<double>(const Level &, const Level &, const double *, const double *, double *,
                                          hipStream_t);
template void launch_restrict_map<float>(const Level &, const Level &, const float *, const float *, float *,
                                         hipStream_t);

template <typename T>
int launch_prolong_map(const Level &F, const Level &C, const T *xc, const T *J, T *xf, double *zout, hipStream_t s,
                       const double *dr1, const double *dr2, double *partials, int64_t partials_cap,
                       const double *xc64) {
  const int nf = F.N + 1, nc = C.N + 1;
  const size_t lds = sizeof(T) * (size_t)(nf * nc + nc * nc * nc + nc * nc * nf + nc * nf * nf);
  const bool dots = dr1 && partials && F.E * (dr2 ? 2 : 1) <= partials_cap;
  const double *r1 = dots ? dr1 : nullptr, *r2 = dots ? dr2 : nullptr;
  auto launch = [&](auto kernel, const auto *x) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)F.E), dim3(kTransferThreads), lds, s, F.N, C.N, C.map, F.omap, x, J, xf,
                       zout, r1, r2, dots ? partials : nullptr);
    return dots ? (int)F.E : 0;
  };
#define SEMCHEB_PICK(A, B)                                                              \
  if (F.N == A && C.N == B) {                                                           \
    if constexpr (sizeof(T) == 4 && B == 1) {                                           \
      if (xc64) return launch(prolong_map_kernel<T, A, B, double>, xc64);               \
    }                                                                                   \
    return launch(prolong_map_kernel<T, A, B, T>, xc);                                  \
  }
  SEMCHEB_TRANSFER_PAIRS(SEMCHEB_PICK)
#undef SEMCHEB_PICK
  if (sizeof(T) == 4 && xc64) return launch(prolong_map_kernel<T, 0, 0, double>, xc64);
  return launch(prolong_map_kernel<T, 0, 0, T>, xc);
}
template int launch_prolong_map<double>(const Level &, const Level &, const double *, const double *, double *,
                                        double *, hipStream_t, const double *, const double *, double *, int64_t,
                                        const double *);
template int launch_prolong_map<float>(const Level &, const Level &, const float *, const float *, float *, double *,
                                       hipStream_t, const double *, const double *, double *, int64_t, const double *);

int launch_update_r_lists(const Level &L, double *scal, const double *r, const double *wL, double *rnew,
                          double *partials, float *r32, hipStream_t s) {
  hipLaunchKernelGGL(update_r_lists_kernel, dim3(nblk(L.n)), dim3(256), 0, s, L.n, L.copies, scal, r, wL, rnew,
                     partials, r32);
  return (int)nblk(L.n);
}

}  // namespace semcheb
