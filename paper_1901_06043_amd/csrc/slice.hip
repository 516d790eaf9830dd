// Hyperslice pre/post-processing (paper Sec. 3.5) and the factor side of
// reconstruction through per-mode linear operators (paper Sec. 8).
//
// Geometry: the hyperslices of mode n are the rows a < J of the mode-n
// unfolding; element (l, a, r) of the tensor sits at l + L*a + L*J*r with
// L = prod_{k<n} J_k and r < Rt = prod_{k>n} J_k.  Every kernel here is an
// HBM-bound single pass over the tensor.
//
// Statistics take one pass.  The sum of squared deviations, which needs the
// mean, is gathered from batches: a thread holds 16 (8) values in registers,
// sums the squares about the batch's own mean, and merges batch and running
// moments (Chan, Golub and LeVeque's pairwise update), so nothing is
// subtracted from anything larger than the spread of the data.  Two mappings,
// chosen so that global loads are contiguous across a wave:
//  * row mapping (L >= 64, or a period L*J above 1024 elements): a workgroup
//    owns one slice and a range of its columns; threads walk the columns, so
//    a wave reads runs of L contiguous values, 16 bytes per lane where L and
//    the base allow it;
//  * period mapping (L < 64 and L*J <= 1024): the tensor is Rt periods of
//    L*J values; a workgroup reads G of them at a time (G*L*J <= 1024) and
//    thread t always meets positions t, t+256, ... (fixed slices per
//    thread), so every load instruction of a wave reads 64 consecutive values.
// Partial results are written per (slice, split) and merged by a second
// kernel in a fixed order, so the statistics do not depend on scheduling.
// Bound: HBM.  Standardising the 33 variables of a 672x672x33x64 float32
// tensor (3.8 GB) took two passes of 1.77 ms each with one 4-byte load in
// flight per thread; the single pass takes 0.96 ms (4.0 TB/s).
#include <cmath>

#include "common.hpp"
#include "kernels.hpp"

namespace tk {

namespace {

constexpr int kST = 256;
constexpr int kPeriodMax = 4 * kST;  // positions of one period held by a workgroup (4 per thread)

// Moments of a set of values: count, mean, sum of squared deviations from the
// mean, sum, extremes, 1-norm and sum of squares.
struct Mom {
  double cnt, mean, m2, sum, mn, mx, n1, n2;
};
constexpr int kMW = 8;  // doubles of a Mom

__device__ __forceinline__ void mom_init(Mom& s) {
  s.cnt = s.mean = s.m2 = s.sum = s.n1 = s.n2 = 0.0;
  s.mn = INFINITY;
  s.mx = -INFINITY;
}

// The union of two sets; an empty one leaves the other as it is (no product
// of a zero count with an infinite mean).
__device__ __forceinline__ void mom_merge(Mom& s, const Mom& o) {
  if (o.cnt > 0.0) {
    const double n = s.cnt + o.cnt, w = o.cnt / n, d = o.mean - s.mean;
    s.mean = (s.cnt > 0.0) ? s.mean + d * w : o.mean;
    s.m2 = (s.cnt > 0.0) ? s.m2 + (o.m2 + d * d * (s.cnt * w)) : o.m2;
    s.cnt = n;
  }
  s.sum += o.sum;
  s.mn = fmin(s.mn, o.mn);
  s.mx = fmax(s.mx, o.mx);
  s.n1 += o.n1;
  s.n2 += o.n2;
}

// Adds the first nb > 0 of B values.  A full batch of equal values has
// exactly zero deviations (B is a power of two and the sum a balanced tree).
template <int B, typename T>
__device__ __forceinline__ void mom_batch(Mom& s, const T (&x)[B], int nb) {
  Mom o;
  double t[B];
  o.mn = INFINITY;
  o.mx = -INFINITY;
  o.n1 = o.n2 = o.m2 = 0.0;
#pragma unroll
  for (int j = 0; j < B; ++j) {
    const double v = (j < nb) ? (double)x[j] : 0.0;
    t[j] = v;
    o.n1 += fabs(v);
    o.n2 += v * v;
    o.mn = (j < nb) ? fmin(o.mn, v) : o.mn;
    o.mx = (j < nb) ? fmax(o.mx, v) : o.mx;
  }
#pragma unroll
  for (int w = B / 2; w > 0; w >>= 1)
#pragma unroll
    for (int j = 0; j < w; ++j) t[j] += t[j + w];
  o.cnt = nb;
  o.sum = t[0];
  o.mean = t[0] / o.cnt;
#pragma unroll
  for (int j = 0; j < B; ++j) {
    const double d = (double)x[j] - o.mean;
    o.m2 += (j < nb) ? d * d : 0.0;
  }
  mom_merge(s, o);
}

__device__ __forceinline__ void mom_store(double* p, const Mom& s) {
  p[0] = s.cnt;
  p[1] = s.mean;
  p[2] = s.m2;
  p[3] = s.sum;
  p[4] = s.mn;
  p[5] = s.mx;
  p[6] = s.n1;
  p[7] = s.n2;
}
__device__ __forceinline__ Mom mom_load(const double* p) {
  return Mom{p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]};
}

// Tree merge of one Mom per thread over NT threads (fixed order); the result
// is valid in thread 0.  `active` (uniform): threads from it on hold an empty
// Mom, and the tree's levels above it are left out.  One row of LDS per
// member: with a Mom's members side by side the lanes of a wave met in four
// banks.
template <int NT>
__device__ __forceinline__ Mom block_merge(Mom s, double (*sh)[NT], uint64_t active) {
  const int tid = threadIdx.x;
  auto put = [&](const Mom& m) __attribute__((always_inline)) {
    const double v[kMW] = {m.cnt, m.mean, m.m2, m.sum, m.mn, m.mx, m.n1, m.n2};
#pragma unroll
    for (int k = 0; k < kMW; ++k) sh[k][tid] = v[k];
  };
  put(s);
  __syncthreads();
  for (int w = NT / 2; w > 0; w >>= 1) {
    if ((uint64_t)w >= active) continue;
    if (tid < w) {
      const int o = tid + w;
      mom_merge(s, Mom{sh[0][o], sh[1][o], sh[2][o], sh[3][o], sh[4][o], sh[5][o], sh[6][o], sh[7][o]});
      put(s);
    }
    __syncthreads();
  }
  return s;
}

// The statistics of slice a: stats[s*J + a] for mean, standard deviation, min,
// max, 1-norm, 2-norm.
__device__ __forceinline__ void mom_stats(const Mom& t, uint64_t a, uint64_t J, double* __restrict__ stats) {
  stats[0 * J + a] = t.sum / t.cnt;
  stats[1 * J + a] = sqrt(t.m2 / t.cnt);
  stats[2 * J + a] = t.mn;
  stats[3 * J + a] = t.mx;
  stats[4 * J + a] = t.n1;
  stats[5 * J + a] = sqrt(t.n2);
}

// Row mapping: workgroup (a, s) reduces columns [s*cper, (s+1)*cper) of
// slice a.  Column c of the unfolding is (r, l) = divmod(c, L).  V values per
// load (V > 1: L and cper multiples of V, Y aligned to V values), 16 values
// per thread in flight.  Slices in one piece (nsplit = 1: many, or short ones)
// get their statistics here, without a second launch (10 us for 5000 slices).
// NT threads: one wave where that holds a split's values, so that a CU reduces
// four times as many of them at once (5000 slices of 198 floats: 37 us with four
// waves, 14 us with one).
template <typename T, int V, int NT>
__global__ __launch_bounds__(NT) void slice_rows_kernel(const T* __restrict__ Y, uint64_t L, uint64_t J,
                                                         uint64_t Rt, int64_t nsplit, uint64_t cper,
                                                         double* __restrict__ part, double* __restrict__ stats) {
  constexpr int B = 16, NL = B / V;
  typedef T vec __attribute__((ext_vector_type(V)));
  __shared__ double sh[kMW][NT];
  const uint64_t a = blockIdx.x / nsplit;
  const uint64_t s = blockIdx.x - a * nsplit;
  const uint64_t K = L * Rt;
  const uint64_t c0 = s * cper;
  const uint64_t c1 = (c0 + cper < K) ? c0 + cper : K;
  Mom acc;
  mom_init(acc);
  constexpr uint64_t kStep = (uint64_t)NT * V;
  uint64_t c = c0 + (uint64_t)threadIdx.x * V;
  uint64_t r = c / L, l = c - r * L;
  const uint64_t dr = kStep / L;
  const uint64_t dl = kStep - dr * L;  // < L
  const T* __restrict__ base = Y + L * a;
  const uint64_t rs = L * J;
  while (c < c1) {
    T x[B];
    int nb = 0;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      if (c < c1) {
        const T* p = base + l + rs * r;
        if constexpr (V == 1) {
          x[j] = *p;
        } else {
          const vec v = *reinterpret_cast<const vec*>(p);
#pragma unroll
          for (int u = 0; u < V; ++u) x[V * j + u] = v[u];
        }
        nb += V;
      } else {
#pragma unroll
        for (int u = 0; u < V; ++u) x[V * j + u] = (T)0;
      }
      c += kStep;
      l += dl;
      r += dr;
      if (l >= L) {
        l -= L;
        ++r;
      }
    }
    mom_batch<B>(acc, x, nb);
  }
  acc = block_merge<NT>(acc, sh, (c1 - c0 + V - 1) / V);
  if (threadIdx.x != 0) return;
  if (nsplit == 1) mom_stats(acc, a, J, stats);
  else mom_store(part + (a * nsplit + s) * kMW, acc);
}

// Period mapping: workgroup w reduces the groups of G periods [w*gper,
// (w+1)*gper); thread t reads positions t + 256k (k < 4) of every group,
// position p being element p % L of slice (p / L) % J.  G is a power of two.
template <typename T>
__global__ __launch_bounds__(kST) void slice_period_kernel(const T* __restrict__ Y, uint32_t L, uint32_t J,
                                                           uint64_t Rt, uint32_t G, uint64_t gper,
                                                           double* __restrict__ part) {
  constexpr int B = 8;
  __shared__ double sp[kPeriodMax][kMW];
  const int tid = threadIdx.x;
  const uint32_t P = L * J, PG = P * G;
  const uint64_t total = (uint64_t)P * Rt;
  const uint64_t e0 = (uint64_t)blockIdx.x * gper * PG;
  const uint64_t e1 = (e0 + gper * PG < total) ? e0 + gper * PG : total;
  Mom acc[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) mom_init(acc[k]);
  for (uint64_t e = e0; e < e1; e += (uint64_t)B * PG) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t p = tid + kST * k;
      if (p >= PG) break;
      T x[B];
      int nb = 0;
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const uint64_t at = e + (uint64_t)j * PG + p;
        const bool ok = at < e1;
        x[j] = ok ? Y[at] : (T)0;
        nb += ok ? 1 : 0;
      }
      if (nb > 0) mom_batch<B>(acc[k], x, nb);
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t p = tid + kST * k;
    if (p < PG) mom_store(sp[p], acc[k]);
  }
  __syncthreads();
  // the periods of a group, pairwise, then the L values of each slice
  for (uint32_t h = G / 2; h > 0; h >>= 1) {
    for (uint32_t p = tid; p < h * P; p += kST) {
      Mom t = mom_load(sp[p]);
      mom_merge(t, mom_load(sp[p + h * P]));
      mom_store(sp[p], t);
    }
    __syncthreads();
  }
  // (short ones one after the other, on up to 256 slices at once; 63 merges of one
  // slice took 5 us that way)
  if (L < 8) {
    for (uint32_t a = tid; a < J; a += kST) {
      Mom t = mom_load(sp[a * L]);
      for (uint32_t l = 1; l < L; ++l) mom_merge(t, mom_load(sp[a * L + l]));
      mom_store(part + ((uint64_t)blockIdx.x * J + a) * kMW, t);
    }
    return;
  }
  for (uint32_t n = L; n > 1; n = (n + 1) / 2) {
    const uint32_t h = (n + 1) / 2;
    for (uint32_t i = tid; i < J * h; i += kST) {
      const uint32_t a = i / h, l = i - a * h;
      if (l + h < n) {
        Mom t = mom_load(sp[a * L + l]);
        mom_merge(t, mom_load(sp[a * L + l + h]));
        mom_store(sp[a * L + l], t);
      }
    }
    __syncthreads();
  }
  for (uint32_t a = tid; a < J; a += kST)
    mom_store(part + ((uint64_t)blockIdx.x * J + a) * kMW, mom_load(sp[a * L]));
}

// One wave per slice: the partials (stride sa between slices, ss between
// splits) in a fixed order.
__global__ __launch_bounds__(64) void slice_finalize_kernel(const double* __restrict__ part, uint64_t J,
                                                            int64_t nsplit, uint64_t sa, uint64_t ss,
                                                            double* __restrict__ stats) {
  __shared__ double sh[kMW][64];
  const uint64_t a = blockIdx.x;
  Mom t;
  mom_init(t);
  for (int64_t s = threadIdx.x; s < nsplit; s += 64) mom_merge(t, mom_load(part + a * sa + s * ss));
  t = block_merge<64>(t, sh, (uint64_t)nsplit);
  if (threadIdx.x == 0) mom_stats(t, a, J, stats);
}

__global__ __launch_bounds__(kST) void scaling_vectors_kernel(const double* __restrict__ stats, uint64_t J,
                                                              int method, double* __restrict__ shift,
                                                              double* __restrict__ scale) {
  const uint64_t a = (uint64_t)blockIdx.x * kST + threadIdx.x;
  if (a >= J) return;
  double sh, sc;
  if (method == 0) {  // standardization: shift by the mean, scale by the standard deviation
    sh = stats[0 * J + a];
    sc = stats[1 * J + a];
  } else {  // max rescaling
    sh = 0.0;
    sc = fmax(fabs(stats[2 * J + a]), fabs(stats[3 * J + a]));
  }
  shift[a] = sh;
  scale[a] = (sc == 0.0) ? 1.0 : sc;
}

// Power-of-two divisor per slice for the reduced-precision Gram: pscale[a] =
// 2^e with max|x| of the slice in [2^(e-1), 2^e), so that every scaled value
// x / 2^e has magnitude below 1 and the largest at least 1/2 (1 for an
// all-zero or non-finite slice).  Division by a power of two is exact.
__global__ __launch_bounds__(kST) void slice_pow2_kernel(const double* __restrict__ stats, uint64_t J,
                                                         double* __restrict__ pscale) {
  const uint64_t a = (uint64_t)blockIdx.x * kST + threadIdx.x;
  if (a >= J) return;
  const double mx = fmax(fabs(stats[2 * J + a]), fabs(stats[3 * J + a]));
  int e = 0;
  if (mx > 0.0 && isfinite(mx)) (void)frexp(mx, &e);
  pscale[a] = ldexp(1.0, e);
}

// S_ab *= pscale_a pscale_b (exact: powers of two), undoing the per-slice scaling.
__global__ __launch_bounds__(kST) void gram_unscale_kernel(double* __restrict__ S, int64_t J,
                                                           const double* __restrict__ pscale) {
  const int64_t e = (int64_t)blockIdx.x * kST + threadIdx.x;
  if (e >= J * J) return;
  const int64_t a = e / J, b = e - a * J;
  S[e] = S[e] * (pscale[a] * pscale[b]);
}

template <typename TI, typename TO, bool INV>
__device__ __forceinline__ TO affine(TI x, double sh, double sc) {
  const double v = (double)x;
  return (TO)(INV ? fma(v, sc, sh) : (v - sh) / sc);
}

// Y = (X - shift_a) / scale_a (or the inverse fma(X, scale_a, shift_a)) with
// a the slice of each element.  A thread takes U groups of 4 consecutive
// elements per iteration, all loaded before the first is used, and carries
// (l, a) of each group's first element incrementally.  One group per iteration
// takes 2.02 ms on the 672x672x33x64 float32 tensor (3.8 TB/s read and written),
// four 1.57 ms (4.9 TB/s), where the scaling is looked up again only where the
// slice changes.  That branch is taken in most groups of short odd slices: there,
// and for few groups per thread, one group, each element looking up its own
// (5x200x30000 floats: 44 us, with four groups 59 us).
// X and Y may be the same buffer (in place; each thread reads its elements
// before writing them).
template <typename TI, typename TO, bool INV, int U>
__global__ __launch_bounds__(kST) void slice_transform_kernel(const TI* X, TO* Y,
                                                              uint64_t total, uint64_t L, uint64_t J,
                                                              const double* __restrict__ shift,
                                                              const double* __restrict__ scale) {
  const uint64_t nvec = total / 4;
  const uint64_t stride = (uint64_t)gridDim.x * kST;
  uint64_t v = (uint64_t)blockIdx.x * kST + threadIdx.x;
  uint64_t q = (4 * v) / L;
  uint64_t l = 4 * v - q * L;
  uint64_t a = q % J;
  const uint64_t S = 4 * stride;
  const uint64_t dq = S / L, dl = S - dq * L, da = dq % J;
  auto step = [&]() __attribute__((always_inline)) {
    l += dl;
    a += da;
    if (l >= L) {
      l -= L;
      ++a;
    }
    while (a >= J) a -= J;
  };
  if constexpr (U == 1) {
    for (; v < nvec; v += stride) {
      TI x[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = X[4 * v + j];
      uint64_t lc = l, ac = a;
      TO y[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        y[j] = affine<TI, TO, INV>(x[j], shift[ac], scale[ac]);
        if (++lc == L) {
          lc = 0;
          ac = (ac + 1 == J) ? 0 : ac + 1;
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) Y[4 * v + j] = y[j];
      step();
    }
  } else {
    while (v < nvec) {
      TI x[U][4];
      uint64_t lv[U], av[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        lv[u] = l;
        av[u] = a;
        const uint64_t at = v + u * stride;
        if (at < nvec) {
#pragma unroll
          for (int j = 0; j < 4; ++j) x[u][j] = X[4 * at + j];
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) x[u][j] = (TI)0;
        }
        step();
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint64_t at = v + u * stride;
        if (at >= nvec) break;
        uint64_t lc = lv[u], ac = av[u];
        TO y[4];
        double sh = shift[ac], sc = scale[ac];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          y[j] = affine<TI, TO, INV>(x[u][j], sh, sc);
          if (++lc == L && j < 3) {
            lc = 0;
            ac = (ac + 1 == J) ? 0 : ac + 1;
            sh = shift[ac];
            sc = scale[ac];
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) Y[4 * at + j] = y[j];
      }
      v += U * stride;
    }
  }
  // the last total % 4 elements
  if (blockIdx.x == 0 && threadIdx.x < total - 4 * nvec) {
    const uint64_t e = 4 * nvec + threadIdx.x;
    const uint64_t ae = (e / L) % J;
    Y[e] = affine<TI, TO, INV>(X[e], shift[ae], scale[ae]);
  }
}

// Factor of one mode of a reconstruction: W = C^T diag(s) U (K x R, row-major,
// element (k, r) at W[k*R + r]) for U the I x R column-major factor and the
// operator kinds of tucker_op_kind; s may be null (no scaling).  One thread
// per (k, r); the sum runs over increasing row index.
__global__ __launch_bounds__(kST) void op_factor_kernel(int kind, int64_t begin, int64_t end, int64_t step,
                                                        const double* __restrict__ Ct, int64_t I, int64_t K,
                                                        int64_t R, const double* __restrict__ U,
                                                        const double* __restrict__ s, double* __restrict__ W) {
  const int64_t idx = (int64_t)blockIdx.x * kST + threadIdx.x;
  if (idx >= K * R) return;
  const int64_t k = idx / R, r = idx - k * R;
  const double* __restrict__ u = U + r * I;
  double acc = 0.0;
  switch (kind) {
    case 0:  // identity
    case 1: {  // strided selection
      const int64_t i = (kind == 0) ? k : begin + k * step;
      acc = u[i] * (s ? s[i] : 1.0);
      break;
    }
    case 2: {  // average of rows [begin + k*step, min(begin + (k+1)*step, end))
      const int64_t lo = begin + k * step;
      const int64_t hi = (lo + step < end) ? lo + step : end;
      for (int64_t i = lo; i < hi; ++i) acc += u[i] * (s ? s[i] : 1.0);
      acc /= (double)(hi - lo);
      break;
    }
    case 3:
    case 4: {  // sum / mean of rows [begin, end)
      for (int64_t i = begin; i < end; ++i) acc += u[i] * (s ? s[i] : 1.0);
      if (kind == 4) acc /= (double)(end - begin);
      break;
    }
    default: {  // dense C^T, K x I row-major
      const double* __restrict__ c = Ct + k * I;
      for (int64_t i = 0; i < I; ++i) acc += c[i] * u[i] * (s ? s[i] : 1.0);
      break;
    }
  }
  W[idx] = acc;
}

__global__ __launch_bounds__(kST) void fill_kernel(double* __restrict__ p, uint64_t n, double v) {
  const uint64_t i = (uint64_t)blockIdx.x * kST + threadIdx.x;
  if (i < n) p[i] = v;
}

// dst (sizes g.dst[0..N)) <- the leading part of src (sizes g.src[k] >=
// g.dst[k]), both natural descending.  One wave per run of dst[0]
// contiguous elements; runs r = 0 .. prod_{k>0} dst[k] - 1.
__global__ __launch_bounds__(kST) void compact_kernel(const double* __restrict__ src, double* __restrict__ dst,
                                                      CompactGeo g, int N, int64_t nruns) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * kST + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * kST) >> 6;
  const int64_t e0 = g.dst[0];
  for (int64_t r = wave; r < nruns; r += nwaves) {
    int64_t rem = r, off = 0, stride = g.src[0];
    for (int k = 1; k < N; ++k) {
      const int64_t i = rem % g.dst[k];
      rem /= g.dst[k];
      off += i * stride;
      stride *= g.src[k];
    }
    for (int64_t i = lane; i < e0; i += 64) dst[r * e0 + i] = src[off + i];
  }
}

// coef[e] = prod_m v_m[e_m] over the multi-index of e in sizes K_lo..K_{hi-1}
// (natural descending); vec holds the vectors one after another.
__global__ __launch_bounds__(kST) void outer_coef_kernel(const double* __restrict__ vec, OuterGeo g, int lo, int hi,
                                                         uint64_t count, double* __restrict__ coef) {
  const uint64_t e = (uint64_t)blockIdx.x * kST + threadIdx.x;
  if (e >= count) return;
  uint64_t rem = e;
  double c = 1.0;
  for (int m = lo; m < hi; ++m) {
    const uint64_t km = rem % (uint64_t)g.K[m];
    rem /= (uint64_t)g.K[m];
    c *= vec[g.voff[m] + km];
  }
  coef[e] = c;
}

// out[o*inner + i] += outer[o] * inner[i], in FP64, rounded once to TO.
template <typename TO>
__global__ __launch_bounds__(kST) void add_outer_kernel(TO* __restrict__ out, uint64_t inner, uint64_t outer,
                                                        const double* __restrict__ ci,
                                                        const double* __restrict__ co) {
  for (uint64_t o = blockIdx.y; o < outer; o += gridDim.y) {
    const double c = co[o];
    TO* __restrict__ row = out + o * inner;
    for (uint64_t i = (uint64_t)blockIdx.x * kST + threadIdx.x; i < inner; i += (uint64_t)gridDim.x * kST)
      row[i] = (TO)((double)row[i] + c * ci[i]);
  }
}

struct StatPlan {
  bool period;
  int64_t nsplit;   // row mapping: splits per slice; period mapping: workgroups
  uint64_t per;     // columns per split / groups of periods per workgroup
  uint32_t G;       // period mapping: periods per group (a power of two)
};

StatPlan plan_stats(uint64_t L, uint64_t J, uint64_t Rt) {
  StatPlan p{};
  const uint64_t K = L * Rt;
  p.G = 1;
  p.period = (L < 64 && L * J <= (uint64_t)kPeriodMax);
  if (p.period) {
    // at least 8 groups (about 8 K elements) per workgroup, about 2048 workgroups
    const uint64_t P = L * J;
    while (2 * p.G * P <= (uint64_t)kPeriodMax) p.G *= 2;
    const uint64_t groups = ceil_div(Rt, p.G);
    p.per = std::max<uint64_t>(8, ceil_div(ceil_div(groups, 2048), 8) * 8);
    p.nsplit = (int64_t)ceil_div(groups, p.per);
  } else {
    uint64_t ns = std::max<uint64_t>(1, ceil_div(2048, J));
    ns = std::min<uint64_t>(ns, std::max<uint64_t>(1, K / 4096));
    p.per = ceil_div(ceil_div(K, ns), 4) * 4;  // whole 16-byte loads where L allows them
    p.nsplit = (int64_t)ceil_div(K, p.per);
  }
  return p;
}

}  // namespace

int64_t slice_stats_work_doubles(uint64_t L, uint64_t J, uint64_t Rt) {
  const StatPlan p = plan_stats(L, J, Rt);
  return (int64_t)(J * p.nsplit * kMW);
}

template <typename T>
hipError_t launch_slice_stats(const T* Y, uint64_t L, uint64_t J, uint64_t Rt, double* work, double* stats,
                              hipStream_t s) {
  const StatPlan p = plan_stats(L, J, Rt);
  if (p.period) {
    hipLaunchKernelGGL((slice_period_kernel<T>), dim3(p.nsplit), dim3(kST), 0, s, Y, (uint32_t)L, (uint32_t)J, Rt,
                       p.G, p.per, work);
  } else {
    constexpr int V = 16 / sizeof(T);
    const dim3 grid(J * p.nsplit);
    const bool vec = L % V == 0 && reinterpret_cast<uintptr_t>(Y) % 16 == 0;
#define SR_LAUNCH(VV, NTV)                                                                                       \
  hipLaunchKernelGGL((slice_rows_kernel<T, VV, NTV>), grid, dim3(NTV), 0, s, Y, L, J, Rt, p.nsplit, p.per, work, \
                     stats)
    if (p.per <= 16 * 64) {
      if (vec) SR_LAUNCH(V, 64);
      else SR_LAUNCH(1, 64);
    } else {
      if (vec) SR_LAUNCH(V, kST);
      else SR_LAUNCH(1, kST);
    }
#undef SR_LAUNCH
    if (p.nsplit == 1) return hipGetLastError();
  }
  const uint64_t sa = p.period ? kMW : (uint64_t)p.nsplit * kMW, ss = p.period ? J * kMW : kMW;
  hipLaunchKernelGGL(slice_finalize_kernel, dim3(J), dim3(64), 0, s, work, J, p.nsplit, sa, ss, stats);
  return hipGetLastError();
}

hipError_t launch_scaling_vectors(const double* stats, uint64_t J, int method, double* shift, double* scale,
                                  hipStream_t s) {
  hipLaunchKernelGGL(scaling_vectors_kernel, dim3((unsigned)ceil_div(J, kST)), dim3(kST), 0, s, stats, J, method,
                     shift, scale);
  return hipGetLastError();
}

hipError_t launch_slice_pow2(const double* stats, uint64_t J, double* pscale, hipStream_t s) {
  hipLaunchKernelGGL(slice_pow2_kernel, dim3((unsigned)ceil_div(J, kST)), dim3(kST), 0, s, stats, J, pscale);
  return hipGetLastError();
}

hipError_t launch_gram_unscale(double* S, int64_t J, const double* pscale, hipStream_t s) {
  hipLaunchKernelGGL(gram_unscale_kernel, dim3((unsigned)ceil_div(J * J, kST)), dim3(kST), 0, s, S, J, pscale);
  return hipGetLastError();
}

template <typename TI, typename TO>
hipError_t launch_slice_transform(const TI* X, TO* Y, uint64_t total, uint64_t L, uint64_t J, const double* shift,
                                  const double* scale, bool inverse, hipStream_t s) {
  const uint64_t nvec = total / 4;
  const int64_t grid = std::max<int64_t>(1, std::min<int64_t>(ceil_div((int64_t)nvec, kST), 8192));
  // the time of one group at a time over that of four, 33 slices of floats: 4.0e8
  // elements, L = 64 (whole groups) 1.32, 255 1.17, 129 0.98, 65 0.86; L = 64, 2.4e7
  // elements (3 groups a thread) 0.88, 3.4e7 (4) 1.01, 5.0e7 1.27; of doubles (or to
  // them) 1.2e7 (1.5) 0.98, 2.4e7 1.09
  const bool four = (L % 4 == 0 || L >= 192) && 2 * nvec >= (uint64_t)((sizeof(TI) + sizeof(TO) > 8 ? 5 : 8) * grid * kST);
#define ST_LAUNCH(INV, U)                                                                                        \
  hipLaunchKernelGGL((slice_transform_kernel<TI, TO, INV, U>), dim3(grid), dim3(kST), 0, s, X, Y, total, L, J, shift, \
                     scale)
  if (inverse && four) ST_LAUNCH(true, 4);
  else if (inverse) ST_LAUNCH(true, 1);
  else if (four) ST_LAUNCH(false, 4);
  else ST_LAUNCH(false, 1);
#undef ST_LAUNCH
  return hipGetLastError();
}

hipError_t launch_op_factor(int kind, int64_t begin, int64_t end, int64_t step, const double* Ct, int64_t I, int64_t K,
                            int64_t R, const double* U, const double* scl, double* W, hipStream_t s) {
  hipLaunchKernelGGL(op_factor_kernel, dim3((unsigned)ceil_div(K * R, kST)), dim3(kST), 0, s, kind, begin, end, step,
                     Ct, I, K, R, U, scl, W);
  return hipGetLastError();
}

hipError_t launch_fill(double* p, uint64_t n, double v, hipStream_t s) {
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)ceil_div((int64_t)n, kST)), dim3(kST), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_compact(const double* src, double* dst, const CompactGeo& g, int N, hipStream_t s) {
  int64_t nruns = 1;
  for (int k = 1; k < N; ++k) nruns *= g.dst[k];
  if (nruns <= 0 || g.dst[0] <= 0) return hipSuccess;
  const int64_t grid = std::min<int64_t>(ceil_div(nruns, kST / 64), 8192);
  hipLaunchKernelGGL(compact_kernel, dim3((unsigned)grid), dim3(kST), 0, s, src, dst, g, N, nruns);
  return hipGetLastError();
}

hipError_t launch_outer_coef(const double* vec, const OuterGeo& g, int lo, int hi, uint64_t count, double* coef,
                             hipStream_t s) {
  hipLaunchKernelGGL(outer_coef_kernel, dim3((unsigned)ceil_div((int64_t)count, kST)), dim3(kST), 0, s, vec, g, lo, hi,
                     count, coef);
  return hipGetLastError();
}

template <typename TO>
hipError_t launch_add_outer(TO* out, uint64_t inner, uint64_t outer, const double* ci, const double* co,
                            hipStream_t s) {
  const unsigned gx = (unsigned)std::min<int64_t>(ceil_div((int64_t)inner, kST), 64);
  const unsigned gy = (unsigned)std::min<uint64_t>(outer, 65535);
  hipLaunchKernelGGL((add_outer_kernel<TO>), dim3(gx, gy), dim3(kST), 0, s, out, inner, outer, ci, co);
  return hipGetLastError();
}

template hipError_t launch_slice_stats<float>(const float*, uint64_t, uint64_t, uint64_t, double*, double*,
                                              hipStream_t);
template hipError_t launch_slice_stats<double>(const double*, uint64_t, uint64_t, uint64_t, double*, double*,
                                               hipStream_t);
template hipError_t launch_slice_transform<float, float>(const float*, float*, uint64_t, uint64_t, uint64_t,
                                                         const double*, const double*, bool, hipStream_t);
template hipError_t launch_slice_transform<float, double>(const float*, double*, uint64_t, uint64_t, uint64_t,
                                                          const double*, const double*, bool, hipStream_t);
template hipError_t launch_slice_transform<double, float>(const double*, float*, uint64_t, uint64_t, uint64_t,
                                                          const double*, const double*, bool, hipStream_t);
template hipError_t launch_slice_transform<double, double>(const double*, double*, uint64_t, uint64_t, uint64_t,
                                                           const double*, const double*, bool, hipStream_t);
template hipError_t launch_add_outer<float>(float*, uint64_t, uint64_t, const double*, const double*, hipStream_t);
template hipError_t launch_add_outer<double>(double*, uint64_t, uint64_t, const double*, const double*, hipStream_t);

}  // namespace tk
