// Gram matrix S = Y_(n) Y_(n)^T (Alg. 2; flop count Sec. 7) for mode sizes
// above the whole-triangle kernel's range: FP64 products of float or double
// input, or, for float input, FP32 MFMA products (the FP32 form) or the
// three-piece bf16 split products of the BF16X6 form (b0 = bf16(x),
// b1 = bf16(x - b0), b2 = bf16(x - b0 - b1); b2 c0 + b0 c2 + b1 c1 +
// b1 c0 + b0 c1 + b0 c0 with v_mfma_f32_16x16x32_bf16), each summed in FP32
// over a 32-column chunk and in FP64 across chunks.
//
// Work items: a pair of 128-row tiles (ta <= tb) and a contiguous range of
// column chunks.  Eight waves per workgroup; wave w multiplies the 16 rows of
// block w of tile ta with up to eight blocks of tile tb (all of them for an
// off-diagonal pair; four or five for a diagonal one, chosen so that the
// waves share its 36 blocks evenly: gram_dma.hpp), in FP64 MFMA accumulators.
// 128 registers per lane leave four waves per SIMD from two workgroups, which
// cover each other's operand reads, load issue and barriers.  Four waves of
// 64 x 64 (two per SIMD) covered them less, and the reduced forms, which keep
// FP32 sums or bf16 pieces beside the FP64 accumulators, fitted only one such
// workgroup on a CU; with eight waves they have two per SIMD in one workgroup,
// or, with 4-byte loads, four in two.
// J^2 K flops over the time, before and after: FP64 672x448x33x64 doubles,
// mode 0: 46.7 -> 58 TF, mode 1 of 448x672x33x64: 45.6 -> 55 TF (FP64 MFMA
// bound, 71 to 79% busy, with 3.4 TB/s of tile reads beyond L2 close behind);
// FP32 mode 0 of 672x448x33x64: 52 -> 83 TF; 161x161x160x11x25 (unaligned columns, on the
// register-staged kernel before): FP32 20.6 -> 49, BF16X6 15.9 -> 46 TF.
// Blocks of rows at or beyond J are skipped, so a ragged last tile costs only
// its rows.  About 8192 items: the faster diagonal and ragged items then even
// out over the run (with two items per workgroup slot the run ended on a long
// tail of slow items).
//
// Staging: the chunk images (gram_dma.hpp) are written straight from global
// memory into LDS (global_load_lds, 64 lanes x 16 bytes per instruction, or 4
// bytes where the rows or columns are not 16-byte aligned), with no registers
// in between, from pointers advanced by a fixed stride per chunk.  Rows >= J
// feed only rows and columns of S that are dropped, and the columns past the
// end of the unfolding (or of a slab of L columns) are zeroed in LDS.  Each
// workgroup double-buffers its chunks (64 or 80 KB); the loads of the next
// chunk run during the MFMAs of the current one (chunk_loop).
//
// Output: every item writes its FP64 partial blocks in the layout of the
// tile-pair reduction (gram_mixed.hip), which sums the splits in a fixed
// order.  ||Y||^2 is the trace of S with FP64 products (its diagonal entries
// are FP64 sums of squares of the values as loaded); with reduced products the
// diagonal items sum the squares of their tile's rows in FP64 from LDS.
#include "common.hpp"
#include "gram_dma.hpp"
#include "kernels.hpp"

namespace tk {

namespace {

using dma::Img;

constexpr int kDW = 8;           // waves per workgroup
constexpr int kDNT = 64 * kDW;   // threads per workgroup

typedef __attribute__((address_space(3))) void lds_void;

struct DmaParams {
  const char* Y;   // the tensor's bytes
  int J;
  int64_t L;       // layout 0: 1
  int64_t K;       // columns of the unfolding
  int64_t CL;      // layout 1: chunks per slab of L columns
  int64_t nchunks, nsplit, total;
  int64_t cps;     // chunks per split
  int ntiles, npairs;
  double* part;
  double* sq;  // PREC 1: one sum of squares per item
};

__device__ __forceinline__ void decode_pair_dma(int p, int ntiles, int& ta, int& tb) {
  int t = 0;
  while (p >= ntiles - t) {
    p -= ntiles - t;
    ++t;
  }
  ta = t;
  tb = t + p;
}

template <int W>
__device__ __forceinline__ void load_lds(const char* src, char* dst) {
  if constexpr (W == 16) __builtin_amdgcn_global_load_lds(static_cast<const void*>(src), (lds_void*)dst, 16, 0, 0);
  else __builtin_amdgcn_global_load_lds(static_cast<const void*>(src), (lds_void*)dst, 4, 0, 0);
}

// Per-lane state of an item's loads: one pointer per tile image.  Instruction
// jj of an image covers its bytes [64 W jj, 64 W (jj + 1)), W bytes per lane;
// a wave issues every eighth one, and the swizzles repeat over those, so that
// they differ by a distance common to the wave (whole columns in layout 0,
// rows in layout 1).  Layout 0: rows >= J are clamped into the tensor; layout
// 1: they are left out.
template <typename T, int LAY, int W>
struct Loader {
  using I = Img<sizeof(T), LAY>;
  static constexpr int ES = sizeof(T);
  static constexpr int IPS = I::TB / (64 * W);         // instructions per tile image
  static constexpr int NI = (IPS + kDW - 1) / kDW;     // per wave and image
  static constexpr int RS = kDW * 64 * W / 128;        // layout 1: rows between a wave's instructions
  const char* p[2];
  int64_t step;   // bytes between a wave's instructions of one image
  int rows[2];    // layout 1: rows from the lane's first row to J, per image
  bool whole;     // layout 1: all rows of both tiles lie in the tensor
  int64_t cc;     // layout 1: chunk within its slab
  int64_t left;   // layout 0: columns from the next chunk's first to K
  int ncol;       // valid columns of the chunk to be loaded next

  // the wave's first instruction of image s (20 per image: 4 waves issue 3 of
  // the first image and 2 of the second, the others 2 and 3)
  __device__ __forceinline__ static int first(int s, int wave) { return (s && IPS % kDW) ? (wave ^ 4) : wave; }

  __device__ __forceinline__ void init(const DmaParams& g, int64_t ch, int r0a, int r0b, int wave, int lane) {
    int64_t base;  // element offset of the chunk's first column
    if constexpr (LAY == 0) {
      base = ch * I::KC * g.J;
      left = g.K - ch * I::KC;
      ncol = (int)min((int64_t)I::KC, left);
      step = (int64_t)(kDW * 64 * W / I::CB) * g.J * ES;
    } else {
      const int64_t m = ch / g.CL;
      cc = ch - m * g.CL;
      base = m * g.L * g.J + cc * I::KC;
      ncol = (int)min((int64_t)I::KC, g.L - cc * I::KC);
      step = (int64_t)RS * g.L * ES;
      whole = max(r0a, r0b) + dma::kTileRows <= g.J;
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      int r, c, b;
      I::inv(first(s, wave) * (64 * W) + lane * W, r, c, b);
      const int r0 = s ? r0b : r0a;
      // (layout 0: a unit holds E rows, and J is a multiple of E where W = 16)
      const int row = min(r0 + r, (LAY == 0 && W == 16) ? g.J - I::E : g.J - 1);
      p[s] = g.Y + (base + ((LAY == 0) ? (int64_t)row + (int64_t)g.J * c : (int64_t)row * g.L + c)) * ES + b;
      rows[s] = g.J - r0 - r;
    }
  }

  // The column of the chunk that this lane's part of instruction jj holds.
  __device__ __forceinline__ static int column(int jj, int lane) {
    int r, c, b;
    I::inv(jj * (64 * W) + lane * W, r, c, b);
    return c;
  }

  // TEST: columns past the chunk's end and rows past J are left out.
  template <bool TEST>
  __device__ __forceinline__ void issue_all(char* buf, int nslots, int wave, int lane) const {
    if constexpr (TEST) asm volatile("" : "+v"(lane));
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if (s >= nslots) break;  // uniform
#pragma unroll
      for (int k = 0; k < NI; ++k) {
        const int jj = first(s, wave) + kDW * k;
        if (jj >= IPS) break;  // uniform
        if (!TEST || ((LAY == 0 || RS * k < rows[s]) && column(jj, lane) < ncol))
          load_lds<W>(p[s] + k * step, buf + s * I::TB + jj * (64 * W));
      }
    }
  }
  // Loads the next chunk into buf.
  __device__ __forceinline__ void issue(char* buf, int nslots, int wave, int lane) const {
    if (ncol >= I::KC && (LAY == 0 || whole)) issue_all<false>(buf, nslots, wave, lane);
    else issue_all<true>(buf, nslots, wave, lane);
  }
  // Zeros the positions of that chunk's columns past its end (the last chunk of
  // the unfolding, or of a slab of L columns when KC does not divide L), then
  // moves on.  Called once the wave's own loads have landed; no load ever
  // targets these positions.
  __device__ __forceinline__ void finish(const DmaParams& g, char* buf, int nslots, int wave, int lane) {
    if (ncol < I::KC) {
      asm volatile("" : "+v"(lane));
#pragma unroll 1
      for (int s = 0; s < nslots; ++s)
#pragma unroll 1
        for (int jj = first(s, wave); jj < IPS; jj += kDW)
          if (column(jj, lane) >= ncol) {
            char* at = buf + s * I::TB + jj * (64 * W) + lane * W;
            if constexpr (W == 16) *reinterpret_cast<uint4*>(at) = uint4{0u, 0u, 0u, 0u};
            else *reinterpret_cast<uint32_t*>(at) = 0u;
          }
    }
    int64_t d;  // bytes to the next chunk
    if constexpr (LAY == 0) {
      d = (int64_t)I::KC * g.J * ES;
      left -= I::KC;
      ncol = (int)min((int64_t)I::KC, left);
    } else {
      d = I::KC * ES;
      if (++cc == g.CL) {
        cc = 0;
        d = (g.L * g.J - (g.CL - 1) * I::KC) * ES;
      }
      ncol = (int)min((int64_t)I::KC, g.L - cc * I::KC);
    }
    p[0] += d;
    p[1] += d;
  }
};

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// The bf16 pieces of eight FP32 values: b0 = bf16(x), b1 = bf16(x - b0)
// (x - b0 is exact in FP32) and b2 = bf16(x - b0 - b1).
__device__ __forceinline__ void split8(const float (&v)[8], bf8 (&p)[3]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float x = v[e];
    const __bf16 b0 = (__bf16)x;
    const float r1 = x - (float)b0;
    const __bf16 b1 = (__bf16)r1;
    p[0][e] = b0;
    p[1][e] = b1;
    p[2][e] = (__bf16)(r1 - (float)b1);
  }
}

// Operand offsets of a lane: row i of block 0 of a tile image, column 0 of
// its lane group (Img::col); d (layout 1): the distance to its second unit.
template <int ES, int LAY>
__device__ __forceinline__ int blk_off(int o, int b) {
  return LAY == 0 ? (o ^ (b * 16 * ES)) : o + b * 16 * 128;
}

// The eight FP32 values of one operand block that lane (i, q) supplies to the
// chunk's products: slot e holds column Img::col(e, q).
template <int LAY>
__device__ __forceinline__ void read8(const char* buf, int off, int d, float (&v)[8]) {
  if constexpr (LAY == 0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = *reinterpret_cast<const float*>(buf + off + e * 4 * Img<4, 0>::CB);
  } else {
    const float4 u0 = *reinterpret_cast<const float4*>(buf + off);
    const float4 u1 = *reinterpret_cast<const float4*>(buf + off + d);
    v[0] = u0.x; v[1] = u0.y; v[2] = u0.z; v[3] = u0.w;
    v[4] = u1.x; v[5] = u1.y; v[6] = u1.z; v[7] = u1.w;
  }
}

// MK: the compile-time block mask (gram_dma.hpp), or kGeneric for a mask
// known only at run time (ragged last tiles), tested block by block.
constexpr unsigned kGeneric = 0x100u;

// The products of one chunk: A block `oa` (already the wave's) with the B
// blocks of the slots in the mask; slot y's block is b0 + y (mod 8).
// PREC 0: FP64 products and accumulation, step by step over all slots.
// PREC 1 (FP32 MFMA) and 3 (BF16X6), float input: slot by slot, each slot's
// products summed in FP32 over the chunk's 32 columns (BF16X6: smallest terms
// first), then added to its FP64 accumulator; AHEAD: FP32 slots overlap.
template <unsigned MK, typename T, int LAY, int PREC, bool AHEAD>
__device__ __forceinline__ void compute_chunk(const char* abuf, const char* bbuf, int oa, int ob, int d, int b0,
                                              d4 (&acc)[8], unsigned mask) {
  using I = Img<sizeof(T), LAY>;
  constexpr int ES = sizeof(T);
  // (derived offsets are formed again for each chunk rather than held in
  // registers for both buffers, which spilled)
  asm volatile("" : "+v"(oa), "+v"(ob), "+v"(d));
  auto on = [&](int y) __attribute__((always_inline)) {
    return (MK == kGeneric) ? ((mask >> y) & 1u) : ((MK >> y) & 1u);
  };
  auto boff = [&](int y) __attribute__((always_inline)) { return blk_off<ES, LAY>(ob, (b0 + y) & 7); };
  if constexpr (PREC == 0 && LAY == 0) {
#pragma unroll
    for (int s = 0; s < I::KC / 4; ++s) {
      __builtin_amdgcn_sched_barrier(0);  // one step's operands at a time
      const double a = (double)*reinterpret_cast<const T*>(abuf + oa + s * 4 * I::CB);
      T b[8];
#pragma unroll
      for (int y = 0; y < 8; ++y)
        if (on(y)) b[y] = *reinterpret_cast<const T*>(bbuf + boff(y) + s * 4 * I::CB);
#pragma unroll
      for (int y = 0; y < 8; ++y)
        if (on(y)) acc[y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (double)b[y], acc[y], 0, 0, 0);
    }
  } else if constexpr (PREC == 0) {
    typedef T V __attribute__((ext_vector_type(I::E)));
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      __builtin_amdgcn_sched_barrier(0);
      const V a = *reinterpret_cast<const V*>(abuf + oa + (g ? d : 0));
      V b[8];
#pragma unroll
      for (int y = 0; y < 8; ++y)
        if (on(y)) b[y] = *reinterpret_cast<const V*>(bbuf + boff(y) + (g ? d : 0));
#pragma unroll
      for (int s = 0; s < I::E; ++s)
#pragma unroll
        for (int y = 0; y < 8; ++y)
          if (on(y)) acc[y] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[s], (double)b[y][s], acc[y], 0, 0, 0);
    }
  } else if constexpr (PREC == 1 && AHEAD && MK != kGeneric) {
    // the next slot's operands are read before, and a slot's sums added to the
    // FP64 accumulators under, the products of another slot
    float a[8], b[2][8];
    f4 c[2];
    read8<LAY>(abuf, oa, d, a);
    read8<LAY>(bbuf, boff(__builtin_ctz(MK)), d, b[0]);
    int n = 0, prev = -1;
#pragma unroll
    for (int y = 0; y < 8; ++y) {
      if (!on(y)) continue;
#pragma unroll
      for (int z = y + 1; z < 8; ++z)
        if (on(z)) {
          read8<LAY>(bbuf, boff(z), d, b[(n + 1) & 1]);
          break;
        }
      __builtin_amdgcn_sched_barrier(0);
      c[n & 1] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 8; ++s) c[n & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[n & 1][s], c[n & 1], 0, 0, 0);
      if (prev >= 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[prev][v] += (double)c[(n + 1) & 1][v];
      }
      prev = y;
      ++n;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[prev][v] += (double)c[(n + 1) & 1][v];
  } else {
    float a[8];
    read8<LAY>(abuf, oa, d, a);
    bf8 ap[3];
    if constexpr (PREC == 3) split8(a, ap);
#pragma unroll
    for (int y = 0; y < 8; ++y) {
      if (!on(y)) continue;
      __builtin_amdgcn_sched_barrier(0);  // one slot's operands at a time
      float b[8];
      read8<LAY>(bbuf, boff(y), d, b);
      f4 c = f4{0.f, 0.f, 0.f, 0.f};
      if constexpr (PREC == 3) {
        bf8 bp[3];
        split8(b, bp);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap[2], bp[0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap[0], bp[2], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap[1], bp[1], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap[1], bp[0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap[0], bp[1], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap[0], bp[0], c, 0, 0, 0);
      } else {
#pragma unroll
        for (int s = 0; s < 8; ++s) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[s], c, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[y][v] += (double)c[v];
    }
  }
}

// FP64 sum of squares of the rows of a diagonal item's tile image (float
// input, PREC 1): rows >= J hold stale data and are skipped, columns past the
// chunk's end were zeroed.
template <int LAY>
__device__ __forceinline__ double chunk_sq(const char* buf, int r0, int J, int tid) {
  using I = Img<4, LAY>;
  double s = 0.0;
  for (int u = tid; u < I::TB / 16; u += kDNT) {
    int r, c, b;
    I::inv(16 * u, r, c, b);
    const float4 v = *reinterpret_cast<const float4*>(buf + 16 * u);
    const float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      // layout 1: the unit's elements share row r; layout 0: rows r .. r + 3
      const int row = r0 + r + (LAY == 0 ? h : 0);
      if (row < J) s += (double)e[h] * (double)e[h];
    }
  }
  return s;
}

// The chunks of one item: chunk t sits in buffer t & 1.  The loads of chunk
// t + 1 are issued right after the barrier that makes chunk t available, so
// they run during chunk t's MFMAs; then the wave waits for them, zeros any
// columns past the chunk's end and meets the others at the next barrier,
// after which the buffer of chunk t is free for chunk t + 2.
template <unsigned MK, typename T, int LAY, int PREC, int W>
__device__ __forceinline__ void chunk_loop(const DmaParams& g, Loader<T, LAY, W>& ld, int64_t niter, char* buf0,
                                           char* buf1, int nslots, int r0a, int wave, int lane, int oa, int ob, int d,
                                           int b0, d4 (&acc)[8], unsigned mask, double& sq) {
  // reduced forms: diagonal items also sum the squares of their tile's rows
  const bool dsq = (PREC >= 1) && nslots == 1;
  const int pb = (nslots - 1) * Img<sizeof(T), LAY>::TB;  // B operand's tile image
  const int tid = 64 * wave + lane;
  if (niter <= 0) return;
  ld.issue(buf0, nslots, wave, lane);
  __builtin_amdgcn_s_waitcnt(0);
  ld.finish(g, buf0, nslots, wave, lane);
  __syncthreads();
  // (one exit from the loop: with two, the accumulators were copied between
  // register sets in every round)
  auto step = [&](char* cur, char* nxt, bool more) __attribute__((always_inline)) {
    if (more) ld.issue(nxt, nslots, wave, lane);  // uniform
    if constexpr (PREC >= 1)
      if (dsq) sq += chunk_sq<LAY>(cur, r0a, g.J, tid);
    compute_chunk<MK, T, LAY, PREC, W == 16>(cur, cur + pb, oa, ob, d, b0, acc, mask);
    if (more) {
      __builtin_amdgcn_s_waitcnt(0);
      ld.finish(g, nxt, nslots, wave, lane);
      __syncthreads();
    }
  };
  int64_t t = 0;
  for (; t + 1 < niter; t += 2) {
    step(buf0, buf1, true);
    step(buf1, buf0, t + 2 < niter);
  }
  if (t < niter) step(buf0, buf1, false);
}

// The whole item of one mask class: accumulators zeroed, all chunks, then the
// partial blocks (one copy per class, so that no accumulator is merged across
// classes).  MFMA result, lane l, register v: FP64 D[(l >> 4) + 4 v][l & 15],
// FP32 D[4 (l >> 4) + v][l & 15].  A diagonal pair's block (w, b) with b < w
// is the transpose of block (b, w).
template <unsigned MK, typename T, int LAY, int PREC, int W>
__device__ __forceinline__ double item_body(const DmaParams& g, Loader<T, LAY, W>& ld, int64_t niter, char* buf0,
                                            char* buf1, bool diag, int r0a, int wave, int lane, int oa, int ob, int d,
                                            unsigned mask, double* __restrict__ P) {
  d4 acc[8];
#pragma unroll
  for (int y = 0; y < 8; ++y) acc[y] = d4{0.0, 0.0, 0.0, 0.0};
  double sq = 0.0;
  const int b0 = diag ? wave : 0;
  chunk_loop<MK, T, LAY, PREC, W>(g, ld, niter, buf0, buf1, diag ? 1 : 2, r0a, wave, lane, oa, ob, d, b0, acc, mask,
                                  sq);
  const int i = lane & 15, q = lane >> 4;
#pragma unroll
  for (int y = 0; y < 8; ++y) {
    if ((MK == kGeneric) ? ((mask >> y) & 1u) : ((MK >> y) & 1u)) {
      const int b = (b0 + y) & 7;
      const bool flip = diag && b < wave;
      const int qb = diag ? dma::tri_index(min(b, wave), max(b, wave)) : wave * 8 + b;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = (PREC == 0) ? q + 4 * v : 4 * q + v;
        P[(int64_t)qb * 256 + (flip ? i * 16 + r : r * 16 + i)] = acc[y][v];
      }
    }
  }
  return sq;
}

// The reduced forms with 16-byte loads run one workgroup per CU: the pieces of
// two operand blocks (BF16X6), or two slots' operands and sums (FP32, AHEAD),
// beside the accumulators spill at 128 registers (mode 0 of 256x256x256x11x5:
// BF16X6 3.6 against 4.2 ms with two workgroups, FP32 3.0 against 3.3 ms with
// two and no overlap of slots, 3.4 with it); with 4-byte loads, whose issue
// needs covering, two workgroups are the faster (mode 0 of 161x161x160x11x25:
// BF16X6 4.0 against 5.6 ms, FP32 3.7 against 4.8 ms).
template <typename T, int LAY, int PREC, int W>
__global__ __launch_bounds__(kDNT, PREC != 0 && W == 16 ? 2 : 4) void gram_dma_kernel(DmaParams g) {
  static_assert(PREC == 0 || sizeof(T) == 4, "the reduced forms read float input");
  using I = Img<sizeof(T), LAY>;
  __shared__ __attribute__((aligned(16))) char buf0[2 * I::TB];
  __shared__ __attribute__((aligned(16))) char buf1[2 * I::TB];
  const int64_t item = xcd_remap(blockIdx.x, gridDim.x, g.total);
  if (item < 0) return;
  const int64_t split = (uint32_t)item / (uint32_t)g.npairs;  // total < 2^31
  const int pair = (int)(item - split * g.npairs);
  int ta, tb;
  decode_pair_dma(pair, g.ntiles, ta, tb);
  const bool diag = (ta == tb);
  const int r0a = 128 * ta, r0b = 128 * tb;
  // split s takes the contiguous chunks [s cps, (s + 1) cps)
  const int64_t ch0 = split * g.cps, niter = min(g.cps, g.nchunks - ch0);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, q = lane >> 4;
  const unsigned mask = __builtin_amdgcn_readfirstlane(dma::wave_mask(wave, diag, r0a, r0b, g.J));
  const int o0 = I::at(i, I::col(0, q));
  const int oa = blk_off<sizeof(T), LAY>(o0, wave);
  const int d = (LAY == 1) ? I::at(i, I::col(I::E, q)) - o0 : 0;
  Loader<T, LAY, W> ld;
  ld.init(g, ch0, r0a, r0b, wave, lane);
  double sq = 0.0;
#define DMA_ITEM(MK)                                                                                              \
  sq = item_body<MK, T, LAY, PREC, W>(g, ld, niter, buf0, buf1, diag, r0a, wave, lane, oa, o0, d, mask,           \
                                      g.part + item * (int64_t)64 * 256)
  // (waves without blocks still load and meet the barriers)
  if (mask == dma::kMaskFull) DMA_ITEM(dma::kMaskFull);
  else if (mask == dma::kMaskDiag5) DMA_ITEM(dma::kMaskDiag5);
  else if (mask == dma::kMaskDiag4) DMA_ITEM(dma::kMaskDiag4);
  else DMA_ITEM(kGeneric);
#undef DMA_ITEM
  if constexpr (PREC >= 1) {
    // the item's sum of squares (zero unless diagonal), in wave order
    __shared__ double sred[kDW];
    const double sw = wave_sum(sq);
    if (lane == 0) sred[wave] = sw;
    __syncthreads();
    if (tid == 0)
      g.sq[item] = ((sred[0] + sred[1]) + (sred[2] + sred[3])) + ((sred[4] + sred[5]) + (sred[6] + sred[7]));
  }
}

// trace(S) in a fixed order: one workgroup.
__global__ __launch_bounds__(256) void gram_trace_kernel(const double* __restrict__ S, int J,
                                                         double* __restrict__ out) {
  __shared__ double red[256];
  double s = 0.0;
  for (int a = threadIdx.x; a < J; a += 256) s += S[(int64_t)a * J + a];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}


}  // namespace

// 16-byte loads: the base and the stride between consecutive columns (unit
// stride) or rows (row segments) are multiples of 16 bytes; 4-byte loads
// otherwise.
static bool gram_dma_w16(int J, uint64_t L, int elem_size, const void* Y) {
  return ((L == 1 ? (uint64_t)J : L) * (uint64_t)elem_size) % 16 == 0 && reinterpret_cast<uintptr_t>(Y) % 16 == 0;
}

// Work items: tile pairs by splits of at least 16 chunks, up to about 8192.
static int64_t gram_dma_chunks(uint64_t L, uint64_t K, int elem_size) {
  const int64_t KC = (L == 1 && elem_size == 8) ? Img<8, 0>::KC : 128 / elem_size;
  return (L == 1) ? ceil_div((int64_t)K, KC) : (int64_t)(K / L) * ceil_div((int64_t)L, KC);
}
static int64_t gram_dma_splits(int64_t npairs, int64_t nchunks) {
  return std::min<int64_t>(std::max<int64_t>(1, 8192 / npairs), std::max<int64_t>(1, nchunks / 16));
}

// The block products of the register-staged tile pairs, which multiply the
// blocks past J of a ragged last tile too, over those of this kernel, which
// leaves them out but takes its chunks slab by slab, so that a last chunk that
// a short slab does not fill is work as well.  A pair of few blocks takes the
// time of 24, that of its loads.
static double gram_dma_gain(int J, uint64_t L, int elem_size) {
  const int64_t KC = 128 / elem_size, nt = ceil_div(J, 128);
  double cost = 0.0;
  for (int64_t a = 0; a < nt; ++a) {
    const int64_t ba = std::min<int64_t>(8, ceil_div(J - 128 * a, 16));
    const int64_t bl = std::min<int64_t>(8, ceil_div(J - 128 * (nt - 1), 16));
    cost += (double)std::max<int64_t>(24, ba * (ba + 1) / 2);
    if (a < nt - 1) cost += (double)((nt - 2 - a) * 8 * ba) + (double)std::max<int64_t>(24, ba * bl);
  }
  const double fill = L == 1 ? 1.0 : (double)L / (double)(ceil_div((int64_t)L, KC) * KC);
  return 32.0 * (double)(nt * (nt + 1)) * fill / cost;
}

// FP64, and the reduced forms on unit stride, with 16-byte loads are taken here
// whatever the shape (FP64 of doubles on row segments at least 1.04 times as fast
// as the register-staged tile pairs, of floats in slabs that fill three quarters
// of their chunks, at a gain of 0.83 to 0.91, 0.93 to 0.97).  With 4-byte loads,
// whose issue the products no longer cover, and for the reduced forms on row
// segments two things decide:
//  * the number of items: with few a Gram is one item's chain of 16 chunks long,
//    which takes 40 to 120 us here, and the other kernel splits finer.  300 rows
//    of floats in slabs of 65, FP64, us, register-staged against here: 1000
//    columns (12 items) 38 / 126, 10000 (174) 67 / 101, 30000 (516) 134 / 136, 70000
//    (1218) 290 / 252;
//  * the gain, with the lines where the two measured the same.  In us, 200000 or
//    300000 columns in slabs of L, J at gain:
//      FP64 of doubles: L = 65 384 at 1.04 1292 / 1407, L = 67 256 at 1.18 656 / 660,
//        L = 129 384 at 1.15 1283 / 1264, L = 129 256 at 1.26 654 / 611
//      FP64 of floats:  L = 65 626 at 0.79 3045 / 3469, L = 129 384 at 1.03 1239 / 1214
//      FP32:    L = 67 257 at 1.22 290 / 368, 16-byte loads 626 at 1.17 1.0 / 1.05
//      BF16X6:  L = 161 257 at 1.47 290 / 356
//    and in 400000 columns (ms)
//      FP32:    L = 447 200 at 1.88 0.45 / 0.35, 336 at 1.48 0.87 / 0.86, 626 at 1.17 2.13 / 2.83
//      BF16X6:  L = 447 161 at 2.27 0.40 / 0.33, 200 at 1.88 0.42 / 0.38, 336 at 1.48 0.85 / 0.96
static bool gram_dma_pays(int J, uint64_t L, uint64_t K, int elem_size, bool w16, int prec) {
  if (w16 && (prec == 0 || L == 1)) return true;
  const int64_t nt = ceil_div(J, 128), npairs = nt * (nt + 1) / 2;
  if (gram_dma_splits(npairs, gram_dma_chunks(L, K, elem_size)) * npairs < 1024) return false;
  const double gain = gram_dma_gain(J, L, elem_size);
  if (L == 1) return prec != 3 || gain >= 1.2;
  if (prec == 0) return gain >= (elem_size == 8 ? 1.2 : 1.1);
  const int64_t KC = 128 / elem_size;
  return gain >= 1.86 || (prec == 1 && w16 && gain >= 1.2 && 20 * L >= 19 * (uint64_t)(ceil_div((int64_t)L, KC) * KC));
}

bool gram_dma_eligible(int J, uint64_t L, uint64_t K, int elem_size, const void* Y, int prec) {
  const uint64_t KC = 128 / elem_size;
  return J > 128 && J <= (1 << 20) && reinterpret_cast<uintptr_t>(Y) % elem_size == 0 &&
         (L == 1 || L >= 64 || L % KC == 0) && gram_dma_pays(J, L, K, elem_size, gram_dma_w16(J, L, elem_size, Y), prec);
}

GramPlan plan_gram_dma(int J, uint64_t L, uint64_t K, int elem_size, int prec) {
  GramPlan p{};
  p.tile = 128;
  p.nchunks = gram_dma_chunks(L, K, elem_size);
  p.ntiles = (int)ceil_div(J, 128);
  p.npairs = p.ntiles * (p.ntiles + 1) / 2;
  // about 16 items per workgroup slot (two slots per CU), at least 16 chunks
  // each: items of different speed (diagonal and ragged pairs are faster)
  // then even out over the run; 128 KB of partial blocks per item
  p.cps = ceil_div(p.nchunks, gram_dma_splits(p.npairs, p.nchunks));
  p.nsplit = ceil_div(p.nchunks, p.cps);
  p.part_elems = p.nsplit * p.npairs * 64 * 256;
  p.sq_elems = (prec >= 1) ? p.nsplit * p.npairs : 0;
  return p;
}

template <typename T>
hipError_t launch_gram_dma(const T* Y, int J, uint64_t L, uint64_t K, int prec, const GramPlan& p, double* part,
                           double* sq, double* S, double* norm2, hipStream_t stream, hipEvent_t after_main) {
  if (!gram_dma_eligible(J, L, K, (int)sizeof(T), Y, prec)) return hipErrorInvalidValue;
  if (prec != 0 && ((prec != 1 && prec != 3) || sizeof(T) != 4 || sq == nullptr)) return hipErrorInvalidValue;
  DmaParams g{};
  g.Y = reinterpret_cast<const char*>(Y);
  g.J = J;
  g.L = (int64_t)L;
  g.K = (int64_t)K;
  const int64_t KC = 128 / (int64_t)sizeof(T);
  g.CL = ceil_div((int64_t)L, KC);
  g.nchunks = p.nchunks;
  g.nsplit = p.nsplit;
  g.cps = p.cps;
  g.ntiles = p.ntiles;
  g.npairs = p.npairs;
  g.total = p.nsplit * p.npairs;
  g.part = part;
  g.sq = sq;
  const int64_t grid = ceil_div(g.total, kXcds) * kXcds;
  const bool w16 = gram_dma_w16(J, L, (int)sizeof(T), Y);
#define DMA_W(LAY, PREC)                                                                                          \
  do {                                                                                                            \
    if (w16) hipLaunchKernelGGL((gram_dma_kernel<T, LAY, PREC, 16>), dim3(grid), dim3(kDNT), 0, stream, g);       \
    else hipLaunchKernelGGL((gram_dma_kernel<T, LAY, PREC, 4>), dim3(grid), dim3(kDNT), 0, stream, g);            \
  } while (0)
#define DMA_L(PREC)             \
  do {                          \
    if (L == 1) DMA_W(0, PREC); \
    else DMA_W(1, PREC);        \
  } while (0)
  if constexpr (sizeof(T) == 4) {
    if (prec == 1) DMA_L(1);
    else if (prec == 3) DMA_L(3);
  }
  if (prec == 0) DMA_L(0);
#undef DMA_L
#undef DMA_W
  if (after_main) (void)hipEventRecord(after_main, stream);
  launch_gram_pair_reduce(part, p.ntiles, p.npairs, p.nsplit, J, S, stream);
  if (norm2) {
    // FP64: the trace of S is the FP64 sum of squares; reduced forms: the
    // diagonal items' FP64 sums of squares, in item order
    if (prec == 0) hipLaunchKernelGGL(gram_trace_kernel, dim3(1), dim3(256), 0, stream, S, J, norm2);
    else hipLaunchKernelGGL(sum_fixed_kernel, dim3(1), dim3(256), 0, stream, sq, g.total, norm2);
  }
  return hipGetLastError();
}

template hipError_t launch_gram_dma<float>(const float*, int, uint64_t, uint64_t, int, const GramPlan&, double*,
                                           double*, double*, double*, hipStream_t, hipEvent_t);
template hipError_t launch_gram_dma<double>(const double*, int, uint64_t, uint64_t, int, const GramPlan&, double*,
                                            double*, double*, double*, hipStream_t, hipEvent_t);

}  // namespace tk
