// Kernels of the sparse levels (2D finite-difference problem, lattice multigrid below order 1) and of
// the nested-dissection coarse solve. Sparse matrices are in FP64, stored by entries (ELL): entry k of
// row r at k * ld + r, rows shorter than the widest padded with zero values, so that the loads of
// consecutive rows are contiguous and none of a row's loads waits for another (no row pointers).
// Levels of these problems are small: they are bound by the number of dependent launches and memory
// latencies, not by bytes. So a Chebyshev step is one launch (the product A d fused with the update, d
// double-buffered), the first two steps from a zero guess are one launch (d_0 is formed from b where
// it is gathered), and the finite-difference levels of at most 1024 unknowns run in one launch of one
// block.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace semcheb {
namespace {

// Row sum of the stored entries times f(column), entries in order; W > 0: width known at compile
// time (every load in flight at once), W = 0: chunks of eight.
template <int W, typename F>
__device__ __forceinline__ double ell_row(int64_t r, const EllArgs &A, F f) {
  double s = 0.0;
  if constexpr (W > 0) {
    int32_t c[W];
    double v[W], x[W];
#pragma unroll
    for (int k = 0; k < W; ++k) c[k] = A.col[k * A.ld + r];
#pragma unroll
    for (int k = 0; k < W; ++k) v[k] = A.val[k * A.ld + r];
#pragma unroll
    for (int k = 0; k < W; ++k) x[k] = f(c[k]);
#pragma unroll
    for (int k = 0; k < W; ++k) s += v[k] * x[k];
  } else {
    for (int k0 = 0; k0 < A.width; k0 += 8) {
      int32_t c[8];
      double v[8], x[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {  // past the width: the last entry, not summed
        const int q = k0 + k < A.width ? k0 + k : A.width - 1;
        c[k] = A.col[q * A.ld + r];
        v[k] = A.val[q * A.ld + r];
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = f(c[k]);
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k0 + k < A.width) s += v[k] * x[k];
    }
  }
  return s;
}

// y = A x (mode 0), y = b - A x (mode 1), y += A x (mode 2); one thread per row.
template <int W>
__global__ void __launch_bounds__(256)
ell_kernel(EllArgs A, const double *__restrict__ x, const double *__restrict__ b, double *__restrict__ y, int mode) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= A.nrows) return;
  const double own = mode == 1 ? b[r] : mode == 2 ? y[r] : 0.0;
  const double s = ell_row<W>(r, A, [&](int32_t c) { return x[c]; });
  y[r] = mode == 1 ? own - s : own + s;
}

// The same product with 16 lanes per row for wide rows (restrictions by 8 hold 225 entries per
// row: one thread would chain 28 pairs of memory latencies). Lane sums in a fixed shuffle order.
__global__ void __launch_bounds__(256)
ell_wide_kernel(EllArgs A, const double *__restrict__ x, const double *__restrict__ b, double *__restrict__ y,
                int mode) {
  const int lane = threadIdx.x & 15;
  const int64_t r = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  const int64_t rc = r < A.nrows ? r : 0;
  double s = 0.0;
  for (int k0 = lane; k0 < A.width; k0 += 64) {
    int32_t c[4];
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = k0 + 16 * q < A.width ? k0 + 16 * q : A.width - 1;
      c[q] = A.col[k * A.ld + rc];
      v[q] = A.val[k * A.ld + rc];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (k0 + 16 * q < A.width) s += v[q] * x[c[q]];
  }
  for (int off = 8; off > 0; off >>= 1) s += __shfl_down(s, off, 16);
  if (lane == 0 && r < A.nrows) {
    if (mode == 0) y[r] = s;
    else if (mode == 1) y[r] = b[r] - s;
    else y[r] += s;
  }
}

// One Chebyshev step with its product: ad = A u, u = d (or x with ELL_FROM_X, the first step of a
// smoothing that starts from x; or d_0 = c0 inv b formed from b with ELL_FIRST2, the first two
// steps from a zero guess). Then, with the flags and modes of cheb_kernel (4: 4th kind, 1: 1st
// kind with the residual scaled by inv),
//   r = (R_FROM_B ? b : r) - ad,  d = a d + bc (inv) r,  x = x + c d
// The new d goes to dn: neighbours still read the old one. x is not stored by a first step that
// gathers it (NO_X); the next step then adds that step's cprev d too (ELL_X_PLUS_D). Lattice level of
// 12,075 unknowns, 27 entries per row: 4.6 us, where the product alone took 12.1 us with one thread per
// CSR row.
template <int W>
__global__ void __launch_bounds__(256)
ell_cheb_kernel(EllArgs A, const double *__restrict__ b, double *__restrict__ r_io, const double *__restrict__ d,
                double *__restrict__ dn_out, double *__restrict__ x, const double *__restrict__ inv, double a,
                double bc, double c, double c0, double cprev, int flags, int mode) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= A.nrows) return;
  const bool first2 = flags & ELL_FIRST2, fromx = flags & ELL_FROM_X;
  const double sv = inv[r];
  double rr = (first2 || fromx) ? b[r] : r_io[r];
  const double xo = first2 ? 0.0 : x[r];
  const double dp = first2 ? c0 * (sv * rr) : fromx ? 0.0 : d[r];
  const double ad = first2 ? ell_row<W>(r, A, [&](int32_t q) { return c0 * (inv[q] * b[q]); })
                           : ell_row<W>(r, A, [&](int32_t q) { return fromx ? x[q] : d[q]; });
  if (mode == 1) rr = ((first2 || fromx) ? sv * rr : rr) - sv * ad;
  else rr -= ad;
  const double dn = a * dp + bc * (mode == 4 ? sv * rr : rr);
  if (!(flags & CHEB_LAST)) {
    r_io[r] = rr;
    dn_out[r] = dn;
  }
  if (!(flags & CHEB_NO_X)) {
    const double xp = first2 ? __dmul_rn(cprev, dp) : (flags & ELL_X_PLUS_D) ? xo + cprev * dp : xo;
    x[r] = xp + c * dn;
  }
}

// ------------------------------------------------------------------ the small levels in one block
// All finite-difference levels of at most kTailRows unknowns of a cycle, down to the dense solve of the
// last one, in one block of kTailRows threads, one row per thread: the level vectors live in LDS, a
// row's matrix entries (at most kTailWidth) in registers, and a Chebyshev step costs two barriers
// instead of two launches. FD problem with 128 intervals under GMRES(20): three levels (961, 225 and 49
// unknowns) take 14.4 us instead of 23 launches of about 3 us.
template <int G>
__device__ __forceinline__ double lanes_sum(double s) {
#pragma unroll
  for (int off = G / 2; off > 0; off >>= 1) s += __shfl_down(s, off, G);
  return s;
}

// rows of a matrix applied to an LDS vector with G lanes per row; store(row, value)
template <int G, typename S>
__device__ __forceinline__ void tail_rows(int nrows, const EllArgs &A, const double *xs, S store) {
  const int lane = threadIdx.x % G;
  for (int r0 = 0; r0 < nrows; r0 += kTailRows / G) {
    const int r = r0 + threadIdx.x / G;
    const int rc = r < nrows ? r : 0;
    double s = 0.0;
    for (int k = lane; k < A.width; k += G) s += A.val[(int64_t)k * A.ld + rc] * xs[A.col[(int64_t)k * A.ld + rc]];
    s = lanes_sum<G>(s);
    if (lane == 0 && r < nrows) store(r, s);
  }
}

__global__ void __launch_bounds__(kTailRows) ell_tail_kernel(TailArgs T, const double *__restrict__ b,
                                                             double *__restrict__ x) {
  extern __shared__ double sm[];
  const int t = threadIdx.x;
  double *tmp = sm;  // largest level: the vector a product gathers
  double *vec = sm + T.lev[0].n;  // per level: b, then x (the last level too)
  if (t < T.lev[0].n) vec[t] = b[t];
  const double *beta[2] = {T.beta_pre, T.beta_post};
  int32_t col[kTailWidth];
  double val[kTailWidth];
  // one smoothing of level q: from zero (pp = 0) or from x (pp = 1); returns the thread's x
  auto smooth = [&](const TailLevel &L, const double *bs, double *xs, int pp) {
    const int k = pp ? T.post : T.pre;
    const bool own = t < L.n;
    const int tc = own ? t : 0;
    const double sv = L.inv[tc], bv = bs[tc];
    double r = T.mode == 1 ? sv * bv : bv, d = 0.0, xv = pp ? xs[tc] : 0.0;
    auto product = [&](const double *src) {
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < kTailWidth; ++q) s += val[q] * src[col[q]];
      return s;
    };
    if (pp) {
      const double ad = product(xs);
      r = T.mode == 1 ? r - sv * ad : r - ad;
    }
    const double theta = L.theta[pp], delta = L.delta[pp];
    double rho = delta / theta;
    for (int i = 0; i < k; ++i) {
      double a = 0.0, bc, c = 1.0;
      if (T.mode == 4) {
        a = i ? (2.0 * i - 1.0) / (2.0 * i + 3.0) : 0.0;
        bc = (i ? (8.0 * i + 4.0) / (2.0 * i + 3.0) : 4.0 / 3.0) * L.rlmax;
        c = beta[pp][i];
      } else if (i == 0) {
        bc = 1.0 / theta;
      } else {
        const double rn = 1.0 / (2.0 * (theta / delta) - rho);
        a = rn * rho;
        bc = 2.0 * rn / delta;
        rho = rn;
      }
      if (i) {
        if (own) tmp[t] = d;
        __syncthreads();
        const double ad = product(tmp);
        __syncthreads();
        r = T.mode == 1 ? r - sv * ad : r - ad;
      }
      d = a * d + bc * (T.mode == 4 ? sv * r : r);
      xv += c * d;
    }
    __syncthreads();  // every gather of xs happened
    if (own) xs[t] = xv;
    __syncthreads();
  };
  auto load_rows = [&](const TailLevel &L) {
#pragma unroll
    for (int q = 0; q < kTailWidth; ++q) {
      const bool in = q < L.A.width && t < L.n;
      col[q] = in ? L.A.col[(int64_t)q * L.A.ld + t] : 0;
      val[q] = in ? L.A.val[(int64_t)q * L.A.ld + t] : 0.0;
    }
  };
  __syncthreads();
  double *bs = vec;  // the current level's b, its x behind it
  for (int q = 0; q + 1 < T.nlev; ++q) {
    const TailLevel &L = T.lev[q];
    double *xs = bs + L.n, *bn = bs + 2 * L.n;
    load_rows(L);
    if (T.pre > 0) {
      smooth(L, bs, xs, 0);
    } else {
      if (t < L.n) xs[t] = 0.0;
      __syncthreads();
    }
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kTailWidth; ++k) s += val[k] * xs[col[k]];
    if (t < L.n) tmp[t] = bs[t] - s;
    __syncthreads();
    auto put = [&](int r, double v) { bn[r] = v; };
    const int nc = T.lev[q + 1].n;
    if (nc <= 16) tail_rows<64>(nc, L.R, tmp, put);
    else if (nc <= 64) tail_rows<16>(nc, L.R, tmp, put);
    else if (nc <= 256) tail_rows<4>(nc, L.R, tmp, put);
    else tail_rows<1>(nc, L.R, tmp, put);
    __syncthreads();
    bs = bn;
  }
  {  // exact solve of the last level with its dense inverse, eight lanes per row
    const int n = T.lev[T.nlev - 1].n;
    double *xs = bs + n;
    const int lane = t & 7;
    for (int r0 = 0; r0 < n; r0 += kTailRows / 8) {
      const int r = r0 + (t >> 3);
      const int rc = r < n ? r : 0;
      double s = 0.0;
      for (int c = lane; c < n; c += 8) s += T.Minv[(int64_t)rc * n + c] * bs[c];
      s = lanes_sum<8>(s);
      if (lane == 0 && r < n) xs[r] = s;
    }
    __syncthreads();
  }
  for (int q = T.nlev - 2; q >= 0; --q) {
    const TailLevel &L = T.lev[q];
    const double *xc = bs + T.lev[q + 1].n;
    bs -= 2 * L.n;
    double *xs = bs + L.n;
    if (t < L.n) {
      double s = 0.0;
      for (int k = 0; k < L.P.width; ++k) s += L.P.val[(int64_t)k * L.P.ld + t] * xc[L.P.col[(int64_t)k * L.P.ld + t]];
      xs[t] += s;
    }
    __syncthreads();
    if (T.post > 0) {
      load_rows(L);
      smooth(L, bs, xs, 1);
    }
  }
  if (t < T.lev[0].n) x[t] = vec[T.lev[0].n + t];
}

// One step of the nested-dissection solve: out[row] = base + sum val * src(col), one group of rows
// that share their columns per block (WPG = 4 wavefronts splitting the columns) or per wavefront
// (WPG = 1). The gathered vector entries serve all rows of the group, and a wave keeps four times
// the factor bytes in flight: a step is a chain of three memory latencies (group, factors and
// columns, vector entries), not a stream. The factors are FP64 or their single-precision copies.
// one batch of kU columns per lane from column q0 on (64 WPG apart), every load requested before
// the first use; past the end: the last entry, not summed; a missing row repeats the first, not stored
template <int kU, int WPG, typename V>
__device__ __forceinline__ void nd_batch(const NdGroup &g, int q0, const V *__restrict__ v0,
                                         const uint32_t *__restrict__ c0, const double *b, const double *y,
                                         const double *x, double (&s)[kNdRows]) {
  const int len = g.len;
  uint32_t c[kU];
  V v[kNdRows][kU];
  double xv[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const int q = q0 + 64 * WPG * u, qc = q < len ? q : len - 1;
    c[u] = c0[qc];
#pragma unroll
    for (int r = 0; r < kNdRows; ++r) v[r][u] = v0[(r < g.nrows ? r : 0) * len + qc];
  }
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const uint32_t w = c[u] >> 30;
    xv[u] = (w == kNdY ? y : w == kNdB ? b : x)[c[u] & 0x3fffffffu];
    if (q0 + 64 * WPG * u >= len) xv[u] = 0.0;
  }
#pragma unroll
  for (int r = 0; r < kNdRows; ++r)
#pragma unroll
    for (int u = 0; u < kU; ++u) s[r] += (double)v[r][u] * xv[u];
}

template <int WPG, typename V>
__global__ void __launch_bounds__(256)
nd_step_kernel(int64_t group0, int64_t ngroups, const NdGroup *__restrict__ groups, const uint32_t *__restrict__ col,
               const V *__restrict__ val, const double *b, const double *y, const double *x, double *out, int up) {
  __shared__ double part[4][kNdRows];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t i = WPG > 1 ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(wave);
  if (WPG == 1 && i >= ngroups) return;
  const NdGroup &g = groups[group0 + i];
  const int len = g.len;
  const V *v0 = val + g.val;
  const uint32_t *c0 = col + g.col;
  double s[kNdRows] = {0.0, 0.0, 0.0, 0.0};
  for (int q0 = WPG > 1 ? wave * 64 : 0; q0 < len; q0 += 64 * 8 * WPG) {
    const int left = (len - q0 + 64 * WPG - 1) / (64 * WPG);  // wave-uniform
    if (left > 4) nd_batch<8, WPG, V>(g, q0 + lane, v0, c0, b, y, x, s);
    else if (left > 2) nd_batch<4, WPG, V>(g, q0 + lane, v0, c0, b, y, x, s);
    else nd_batch<2, WPG, V>(g, q0 + lane, v0, c0, b, y, x, s);
  }
#pragma unroll
  for (int r = 0; r < kNdRows; ++r)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s[r] += __shfl_down(s[r], off, 64);
  if constexpr (WPG > 1) {
    if (lane == 0)
#pragma unroll
      for (int r = 0; r < kNdRows; ++r) part[wave][r] = s[r];
    __syncthreads();
    const int r = threadIdx.x;
    if (r >= g.nrows) return;
    double t = part[0][r];
#pragma unroll
    for (int w = 1; w < WPG; ++w) t += part[w][r];
    out[g.row[r]] = up ? b[g.row[r]] + t : t;
  } else if (lane == 0) {
#pragma unroll
    for (int r = 0; r < kNdRows; ++r)
      if (r < g.nrows) out[g.row[r]] = up ? b[g.row[r]] + s[r] : s[r];
  }
}

// blocks of 64 rows while the level is too small to fill the chip with blocks of 256
inline int ell_block(int64_t n) { return n < 256 * 256 ? 64 : 256; }
inline unsigned blocks(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

#define SEMCHEB_ELL_WIDTHS(X) X(4) X(5) X(8) X(9) X(27)

void launch_ell(const EllArgs &A, const double *x, const double *b, double *y, int mode, hipStream_t s) {
  if (A.nrows == 0) return;
  const int bs = ell_block(A.nrows);
  const dim3 grid(blocks(A.nrows, bs)), block(bs);
  switch (A.width) {
#define SEMCHEB_ELL(w) \
  case w: hipLaunchKernelGGL((ell_kernel<w>), grid, block, 0, s, A, x, b, y, mode); return;
    SEMCHEB_ELL_WIDTHS(SEMCHEB_ELL)
#undef SEMCHEB_ELL
    default: break;
  }
  if (A.width > 32)
    hipLaunchKernelGGL(ell_wide_kernel, dim3(blocks(A.nrows, 16)), dim3(256), 0, s, A, x, b, y, mode);
  else
    hipLaunchKernelGGL((ell_kernel<0>), grid, block, 0, s, A, x, b, y, mode);
}

void launch_ell_cheb(const EllArgs &A, const double *b, double *r, const double *d, double *dn, double *x,
                     const double *inv, double a, double bc, double c, double c0, double cprev, int flags, int mode,
                     hipStream_t s) {
  if (A.nrows == 0) return;
  const int bs = ell_block(A.nrows);
  const dim3 grid(blocks(A.nrows, bs)), block(bs);
  switch (A.width) {
#define SEMCHEB_ELL(w)                                                                                          \
  case w:                                                                                                       \
    hipLaunchKernelGGL((ell_cheb_kernel<w>), grid, block, 0, s, A, b, r, d, dn, x, inv, a, bc, c, c0, cprev,    \
                       flags, mode);                                                                            \
    return;
    SEMCHEB_ELL_WIDTHS(SEMCHEB_ELL)
#undef SEMCHEB_ELL
    default:
      hipLaunchKernelGGL((ell_cheb_kernel<0>), grid, block, 0, s, A, b, r, d, dn, x, inv, a, bc, c, c0, cprev, flags,
                         mode);
  }
}

void launch_nd_step(const CoarseSolver &C, const NdStep &st, const double *b, double *x, bool f32, hipStream_t s) {
  double *out = st.up ? C.y : x;
  if (st.ngroups == 0) return;
  // four wavefronts per group while the groups alone would leave the chip short of wavefronts
  // (eight were no faster: 31^3 unknowns, 698 groups of 2791 columns, 22.1 against 22.2 us)
  const bool wide = st.ngroups < 4096;
  const dim3 grid((unsigned)(wide ? st.ngroups : (st.ngroups + 3) / 4)), block(256);
#define SEMCHEB_ND(w, V, vals)                                                                                  \
  hipLaunchKernelGGL((nd_step_kernel<w, V>), grid, block, 0, s, st.group0, st.ngroups, C.nd_groups, C.nd_col,   \
                     vals, b, C.y, x, out, st.up ? 1 : 0)
  if (f32) {
    if (wide) SEMCHEB_ND(4, float, C.nd_val32);
    else SEMCHEB_ND(1, float, C.nd_val32);
  } else {
    if (wide) SEMCHEB_ND(4, double, C.nd_val);
    else SEMCHEB_ND(1, double, C.nd_val);
  }
#undef SEMCHEB_ND
}

void launch_ell_tail(const TailArgs &T, const double *b, double *x, hipStream_t s) {
  size_t lds = (size_t)T.lev[0].n;
  for (int q = 0; q < T.nlev; ++q) lds += 2 * (size_t)T.lev[q].n;
  hipLaunchKernelGGL(ell_tail_kernel, dim3(1), dim3(kTailRows), lds * sizeof(double), s, T, b, x);
}

}  // namespace semcheb
