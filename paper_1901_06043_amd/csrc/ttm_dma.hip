// Mode-n product Z_(n) = M Y_(n) (Sec. 2.2.3, Alg. 3) with FP64 products, for
// more than 64 output rows, on the strided unfolding (element (j, c = l + L m)
// of Y_(n) at l + L j + L J m, element (k, c) of Z_(n) at l + L k + L K m).
//
// Work items: a tile of up to 128 output rows k by 128 columns c, over the
// whole reduction J in chunks of 16.  The row tiles of one column tile are
// consecutive items (same XCD), so their reads of the same Y chunks meet in
// L2 and Y comes from HBM about once.  The ceil(K / 16) blocks of rows are
// split evenly over the row tiles.  Eight waves per workgroup, each holding
// all of the tile's k blocks of one 16-column block in FP64 MFMA accumulators
// (v_mfma_f64_16x16x4f64): a step of four j reads NB + 1 operands from LDS for
// NB MFMAs.  128 registers per lane leave four waves per SIMD from two
// workgroups, which cover each other's operand reads, barriers, load issue
// and stores; four waves of 64 x 64 each (8 operands for 16 MFMAs, two waves
// per SIMD) covered them less, and split a ragged row tile unevenly.  The
// bound is the FP64 MFMA rate (72.8 TF for a large matrix product here):
// 672 -> 448 rows of 672x448x33x64 doubles, L = 1: 57.4 -> 68.2 TF;
// 336 -> 672 of 448x336x33x100, L > 1: 54.3 -> 67.0 TF;
// 626 -> 469 of 672x224x8x626 floats: 46.4 -> 64.6 TF.
// The MFMA's output rows are k (A = M, B = Y) when L > 1, so that a lane
// group stores 16 consecutive columns, and c (A = Y^T, B = M^T) when L = 1, so
// that it stores 16 consecutive rows k; both are contiguous in Z.
//
// Staging: both operands' chunk images (ttm_dma.hpp) are written straight
// from global memory into LDS (global_load_lds, 16 bytes per lane), double
// buffered; two workgroups fit on a CU.  Rows past K and columns past the end
// are clamped into the tensor (their outputs are not stored); indices j >= J
// of the last chunk are zeroed in both images.
#include "common.hpp"
#include "kernels.hpp"
#include "ttm_dma.hpp"

namespace tk {

namespace {

using tdma::kJC;
using tdma::TImg;

constexpr int kTDW = 8;   // waves per workgroup
constexpr int kTDNT = 64 * kTDW;

typedef __attribute__((address_space(3))) void lds_void;

struct TtmDmaParams {
  const char* Y;
  const char* M;
  char* Z;
  int J, K;
  int64_t L, cols;
  int64_t msk, msj;   // M(k, j) at M + k msk + j msj (doubles)
  int64_t nkt, total;
  int khi;             // row tiles with the larger number of blocks
  int64_t Lo;          // L of the output (L unless remapped)
  int64_t Lp, Pp, Rp;  // output remap (TtmOutRemap); Pp == Rp: none
};

// ORI 0 (L > 1): A = M (row form MF = 0, column form MF = 1), B = Y (column
// form).  ORI 1 (L = 1): A = Y (row form), B = M.
// WY: bytes per lane of the Y loads, 16, or 4 where Y's rows or columns are
// not 16-byte aligned (L or J odd, or not a multiple of 4 for floats); M is
// always loaded in 16-byte units (launch_pack_factor makes an aligned copy).
template <typename TY, int ORI, int MF, int WY>
struct Cfg {
  using IM = TImg<MF == 0 ? 0 : 1, 8>;
  using IY = TImg<ORI == 0 ? 1 : 0, sizeof(TY)>;
  static constexpr int MB = IM::BYTES, YB = IY::BYTES;
  static constexpr int BUF = MB + YB;  // one chunk: M image then Y image
  static constexpr int NIM = MB / 1024, NIY = YB / (64 * WY);  // load instructions per image
};

// Per-lane state of the loads of one item (tile at output row k0, column
// c0).  The wave issues instructions jj = w, w + 8, ... of each image, from
// pointers that it advances by a fixed stride per chunk: forming each address
// from (row, j) again, under a test of both, cost about 800 cycles of issue
// per chunk (on four waves) beside 4096 of MFMAs.  Rows and columns outside
// the tensor are clamped into it: their outputs are not stored.
//   16-byte loads: one pointer per instruction;
//   4-byte loads (256 bytes per instruction; Y only), doubles: column form, j
//     = 2 n + (w >> 2) and the lane's rows alternate between two sets with the
//     swizzle of j (bit 0 of n); row form, 2 rows per instruction (16 more per
//     n).  Floats: column form, j = 4 n + (w >> 1), again two sets of rows;
//     row form, 4 rows per instruction (32 more per n).
template <typename TY, int ORI, int MF, int WY>
struct Loader {
  static constexpr int NM = Cfg<TY, ORI, MF, WY>::NIM / kTDW;
  static constexpr int NY = Cfg<TY, ORI, MF, WY>::NIY / kTDW;
  static constexpr int NP = (WY == 16) ? NY : (ORI == 1 ? 1 : 2);
  const char* mp[NM];
  const char* yp[NP];
  int64_t mjstride, yjstride;  // M, Y bytes per reduction index j
  int64_t yrstride;  // 4-byte row form: Y bytes per row
  int yleft;         // 4-byte row form: columns from the lane's first row to the tensor's last
  int yj;            // 4-byte row form: the lane's j
};

template <typename TY, int ORI, int MF, int WY>
__device__ __forceinline__ void loader_init(Loader<TY, ORI, MF, WY>& ld, const TtmDmaParams& g, int k0, int64_t c0,
                                            int wave, int lane) {
  using C = Cfg<TY, ORI, MF, WY>;
  using LD = Loader<TY, ORI, MF, WY>;
  constexpr int ES = sizeof(TY);
#pragma unroll
  for (int n = 0; n < LD::NM; ++n) {
    int r, j;
    C::IM::unit_of(wave + kTDW * n, lane, r, j);
    // (column form: the unit's second row may lie one past the last)
    const int k = min(k0 + r, MF == 0 ? g.K - 1 : (g.K - 1) & ~1);
    ld.mp[n] = g.M + ((int64_t)k * g.msk + (int64_t)j * g.msj) * 8;
  }
  ld.mjstride = g.msj * 8;
  ld.yjstride = (ORI == 0) ? g.L * (int64_t)ES : (int64_t)ES;
  ld.yrstride = (int64_t)g.J * ES;
  // column c of the unfolding sits at l + L J m
  auto colbase = [&](int rr) {
    const int64_t last = (WY == 16) ? (g.cols - 1) / (16 / ES) * (16 / ES) : g.cols - 1;
    const uint32_t c = (uint32_t)min(c0 + rr, last);  // cols < 2^32
    const uint32_t m = c / (uint32_t)g.L, l = c - m * (uint32_t)g.L;
    return g.Y + (l + g.L * (int64_t)g.J * m) * (int64_t)ES;
  };
  if constexpr (WY == 16 && ORI == 0) {
    // the lane's rows are the same for all of the wave's instructions (the
    // swizzle of j = w + 8 n, or of the j that an instruction of floats
    // covers, depends on the wave and lane only)
    int r, j;
    C::IY::unit_of(wave, lane, r, j);
    const char* col = colbase(r);
#pragma unroll
    for (int n = 0; n < LD::NY; ++n) {
      C::IY::unit_of(wave + kTDW * n, lane, r, j);
      ld.yp[n] = col + (int64_t)j * ld.yjstride;
    }
  } else if constexpr (WY == 16) {
#pragma unroll
    for (int n = 0; n < LD::NY; ++n) {
      int r, j;
      C::IY::unit_of(wave + kTDW * n, lane, r, j);
      ld.yp[n] = g.Y + min(c0 + r, g.cols - 1) * ld.yrstride + j * ES;
    }
  } else if constexpr (ORI == 0) {
    if constexpr (ES == 4) {
      // 512 bytes per j: instruction w + 8 n covers half w & 1 of j
      const int r = 4 * (16 * (wave & 1) + (lane >> 2)) + (lane & 3);
#pragma unroll
      for (int p = 0; p < LD::NP; ++p) ld.yp[p] = colbase(r ^ (16 * (2 * p + (wave >> 2)))) + (wave >> 1) * ld.yjstride;
    } else {
      // 1024 bytes per j: instruction w + 8 n covers quarter w & 3 of j
      const int u = 16 * (wave & 3) + (lane >> 2);
#pragma unroll
      for (int p = 0; p < LD::NP; ++p)
        ld.yp[p] = colbase(2 * (u ^ (8 * p)) + ((lane & 3) >> 1)) + (lane & 1) * 4 + (wave >> 2) * ld.yjstride;
    }
  } else {
    // floats: rows 4 w + 32 n + (lane >> 4); doubles: rows 2 w + 16 n + (lane >> 5)
    const int row = (ES == 4) ? 4 * wave + (lane >> 4) : 2 * wave + (lane >> 5);
    const int64_t c = min(c0 + row, g.cols - 1);
    ld.yleft = (int)min((int64_t)tdma::kRows, g.cols - 1 - c);
    ld.yp[0] = g.Y + c * ld.yrstride + (ES == 4 ? 0 : (lane & 1) * 4);
    ld.yj = (ES == 4) ? 4 * (((lane & 15) >> 2) ^ (wave & 3)) + (lane & 3)
                      : 2 * (((lane & 31) >> 2) ^ wave) + ((lane & 3) >> 1);
  }
}

__device__ __forceinline__ void load_lds16(const char* src, char* dst) {
  __builtin_amdgcn_global_load_lds(static_cast<const void*>(src), (lds_void*)dst, 16, 0, 0);
}
__device__ __forceinline__ void load_lds4(const char* src, char* dst) {
  __builtin_amdgcn_global_load_lds(static_cast<const void*>(src), (lds_void*)dst, 4, 0, 0);
}

// Loads the next chunk into buf: M image, then Y image.  `left`: reduction
// indices from the chunk's first to J; fewer than 16 in a ragged last chunk,
// where the lanes of indices past the end load nothing.
template <typename TY, int ORI, int MF, int WY>
__device__ __forceinline__ void issue_chunk(Loader<TY, ORI, MF, WY>& ld, int left, char* buf, int wave, int lane) {
  using C = Cfg<TY, ORI, MF, WY>;
  using LD = Loader<TY, ORI, MF, WY>;
  const bool whole = left >= kJC;  // uniform
  auto yinstr = [&](int n, bool test) __attribute__((always_inline)) {
    char* dst = buf + C::MB + (wave + kTDW * n) * (64 * WY);
    if constexpr (WY == 16) {
      int r, j;
      C::IY::unit_of(wave + kTDW * n, lane, r, j);
      if (!test || j < left) load_lds16(ld.yp[n], dst);
    } else if constexpr (ORI == 0) {
      // (the wave's part of j is in the pointers)
      const int j = (sizeof(TY) == 4) ? 4 * n : 2 * n, jw = (sizeof(TY) == 4) ? (wave >> 1) : (wave >> 2);
      if (!test || j + jw < left) load_lds4(ld.yp[n & 1] + j * ld.yjstride, dst);
    } else {
      const int step = (sizeof(TY) == 4) ? 32 : 16;
      // (columns past the last one are not loaded: they feed no stored output)
      if (!test || (step * n <= ld.yleft && ld.yj < left))
        load_lds4(ld.yp[0] + step * n * ld.yrstride + ld.yj * (int)sizeof(TY), dst);
    }
  };
  if (whole) {
#pragma unroll
    for (int n = 0; n < LD::NM; ++n) load_lds16(ld.mp[n], buf + (wave + kTDW * n) * 1024);
  } else {
#pragma unroll
    for (int n = 0; n < LD::NM; ++n) {
      int r, j;
      C::IM::unit_of(wave + kTDW * n, lane, r, j);
      if (j < left) load_lds16(ld.mp[n], buf + (wave + kTDW * n) * 1024);
    }
  }
  // 4-byte row form: all of the tile's columns inside the tensor
  const bool inside = (WY == 16 || ORI == 0) || __all(ld.yleft >= tdma::kRows - 16);
  if (whole && inside) {
#pragma unroll
    for (int n = 0; n < LD::NY; ++n) yinstr(n, false);
  } else {
#pragma unroll
    for (int n = 0; n < LD::NY; ++n) yinstr(n, true);
  }
#pragma unroll
  for (int n = 0; n < LD::NM; ++n) ld.mp[n] += kJC * ld.mjstride;
#pragma unroll
  for (int n = 0; n < LD::NP; ++n) ld.yp[n] += kJC * ld.yjstride;
}

// Zeros the elements of the indices j >= left of a chunk in both images.
// Each wave clears the slots of its own load instructions (loaded or not),
// once its loads have landed, so that no load of another wave can land on a
// cleared element afterwards.
template <typename TY, int ORI, int MF, int WY>
__device__ __forceinline__ void fill_chunk(const Loader<TY, ORI, MF, WY>& ld, int left, char* buf, int wave,
                                           int lane) {
  using C = Cfg<TY, ORI, MF, WY>;
  if (left >= kJC) return;
  // M: 16-byte units of two doubles; the row form's two elements have j, j + 1
#pragma unroll
  for (int n = 0; n < C::NIM / kTDW; ++n) {
    const int jj = wave + kTDW * n;
    int r, j;
    C::IM::unit_of(jj, lane, r, j);
    double* e = reinterpret_cast<double*>(buf + jj * 1024 + lane * 16);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (j + (MF == 0 ? h : 0) >= left) e[h] = 0.0;
  }
  constexpr int ES = sizeof(TY);
#pragma unroll
  for (int n = 0; n < C::NIY / kTDW; ++n) {
    const int jj = wave + kTDW * n;
    if constexpr (WY == 16) {
      int r, j;
      C::IY::unit_of(jj, lane, r, j);
      TY* e = reinterpret_cast<TY*>(buf + C::MB + jj * 1024 + lane * 16);
#pragma unroll
      for (int h = 0; h < 16 / ES; ++h)
        if (j + (ORI == 1 ? h : 0) >= left) e[h] = (TY)0;
    } else {
      const int jl = (ORI == 1) ? ld.yj : (ES == 4 ? 4 * n + (wave >> 1) : 2 * n + (wave >> 2));
      if (jl >= left) *reinterpret_cast<uint32_t*>(buf + C::MB + jj * 256 + lane * 4) = 0u;
    }
  }
}

// Operand reads of one lane for NB blocks (16 rows each, `bs` bytes apart) of
// an image.  Row form: one pair of values per block serves steps 2 g and 2 g +
// 1, at o (g = 0) or o + d (g = 1); column form: step s at o + (s & 1) CB +
// 8 (s >> 1) CB.
template <int FORM, typename T, int NB>
struct Opnd;

template <typename T, int NB>
struct Opnd<0, T, NB> {  // row form
  typedef T pair __attribute__((ext_vector_type(2)));
  static constexpr int BS = 16 * TImg<0, sizeof(T)>::RB;
  pair u[NB];
  __device__ __forceinline__ void fetch(const char* img, int o, int d, int s) {
    if ((s & 1) == 0) {
#pragma unroll
      for (int x = 0; x < NB; ++x) u[x] = *reinterpret_cast<const pair*>(img + o + (s ? d : 0) + x * BS);
    }
  }
  __device__ __forceinline__ double get(int x, int s) const { return (double)((s & 1) ? u[x].y : u[x].x); }
};

template <typename T, int NB>
struct Opnd<1, T, NB> {  // column form
  static constexpr int CB = tdma::kRows * (int)sizeof(T);
  T v[NB];
  // (a block is 16 rows: 16 sizeof(T) bytes, moved by the swizzle of j, which
  // the lane's o holds for block 0 and flips in the same bits for all)
  __device__ __forceinline__ void fetch(const char* img, int o, int, int s) {
#pragma unroll
    for (int x = 0; x < NB; ++x)
      v[x] = *reinterpret_cast<const T*>(img + (o ^ (x * 16 * (int)sizeof(T))) + (s & 1) * CB + (s >> 1) * 8 * CB);
  }
  __device__ __forceinline__ double get(int x, int) const { return (double)v[x]; }
};

// One chunk of MFMAs (four steps of four j) over NX x NY blocks.  `half`: the
// chunk holds at most 8 j, which steps 0 and 1 cover (j(s, q) = 2 q + (s & 1)
// + 8 (s >> 1)).  `issue` enqueues the next chunk's loads, behind the first
// operand reads.
template <int NX, int NY, int FA, typename TA, int FB, typename TB, typename F>
__device__ __forceinline__ void compute_chunk(const char* abuf, const char* bbuf, int oa, int da, int ob, int db,
                                              d4 (&acc)[NX][NY], bool half, F&& issue) {
  Opnd<FA, TA, NX> a;
  Opnd<FB, TB, NY> b;
#pragma unroll
  for (int s = 0; s < kJC / 4; ++s) {
    if (s >= 2 && half) break;  // uniform
    a.fetch(abuf, oa, da, s);
    b.fetch(bbuf, ob, db, s);
    if (s == 0) issue();
#pragma unroll
    for (int x = 0; x < NX; ++x)
#pragma unroll
      for (int y = 0; y < NY; ++y)
        acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.get(x, s), b.get(y, s), acc[x][y], 0, 0, 0);
  }
}

// Chunk t from one buffer while chunk t + 1 is loaded into the other.
template <int NX, int NY, typename TY, int ORI, int MF, int WY>
__device__ __forceinline__ void chunk_loop(Loader<TY, ORI, MF, WY>& ld, const TtmDmaParams& g, char* buf0, char* buf1,
                                           int oa, int da, int ob, int db, d4 (&acc)[NX][NY], int wave, int lane) {
  using C = Cfg<TY, ORI, MF, WY>;
  // A and B operand images: forms, element types and offsets in a buffer
  constexpr int FM = (MF == 0) ? 0 : 1, FY = (ORI == 0) ? 1 : 0;
  constexpr int FA = (ORI == 0) ? FM : FY, FB = (ORI == 0) ? FY : FM;
  using TA = typename std::conditional<ORI == 0, double, TY>::type;
  using TB = typename std::conditional<ORI == 0, TY, double>::type;
  constexpr int AOFF = (ORI == 0) ? 0 : C::MB, BOFF = (ORI == 0) ? C::MB : 0;
  const int nch = (g.J + kJC - 1) / kJC;
  issue_chunk(ld, g.J, buf0, wave, lane);
  __builtin_amdgcn_s_waitcnt(0);
  fill_chunk(ld, g.J, buf0, wave, lane);
  __syncthreads();
  auto step = [&](int t, char* cur, char* nxt) __attribute__((always_inline)) {
    const int left = g.J - kJC * t;
    const bool more = t + 1 < nch;
    compute_chunk<NX, NY, FA, TA, FB, TB>(cur + AOFF, cur + BOFF, oa, da, ob, db, acc, left <= kJC / 2,
                                          [&]() __attribute__((always_inline)) {
                                            if (more) issue_chunk(ld, left - kJC, nxt, wave, lane);
                                          });
    if (more) {
      __builtin_amdgcn_s_waitcnt(0);
      fill_chunk(ld, left - kJC, nxt, wave, lane);
      __syncthreads();
    }
    return more;
  };
  for (int t = 0;; t += 2)
    if (!step(t, buf0, buf1) || !step(t + 1, buf1, buf0)) break;
}

// Stores the wave's blocks of the tile: blocks of 16 along k from k0 and the
// 16 columns from c0.  MFMA result: lane l, register v -> D[(l >> 4) + 4 v][l & 15].
template <int NB, typename TZ, int ORI, int NX, int NY>
__device__ __forceinline__ void store_tile(const TtmDmaParams& g, const d4 (&acc)[NX][NY], int k0, int64_t c0, int i,
                                           int q) {
  TZ* __restrict__ Z = reinterpret_cast<TZ*>(g.Z);
  if constexpr (ORI == 0) {
    // D rows k = k0 + 16 x + q + 4 v, column c = c0 + i
    const int64_t c = c0 + i;
    if (c >= g.cols) return;
    const int64_t m = (uint32_t)c / (uint32_t)g.L, l = c - m * g.L;  // cols < 2^32
    int64_t lo = l;
    bool zpad = false;  // also write the appended zero slice after this one
    if (g.Pp != g.Rp) {  // uniform
      const int64_t t = (uint32_t)l / (uint32_t)g.Lp, a = l - t * g.Lp;
      const int64_t h = (uint32_t)t / (uint32_t)g.Pp, ip = t - h * g.Pp;
      if (ip >= g.Rp) return;  // a zero slice of the padded mode
      lo = a + g.Lp * (ip + g.Rp * h);
      zpad = g.Rp > g.Pp && ip == g.Pp - 1;
    }
    TZ* zc = Z + lo + g.Lo * ((int64_t)g.K * m + k0 + q);
#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (k0 + 16 * x + q + 4 * v < g.K) {
          *zc = static_cast<TZ>(acc[x][0][v]);
          if (zpad) zc[g.Lp] = static_cast<TZ>(0.0);
        }
        zc += 4 * g.Lo;
      }
  } else {
    // D rows c = c0 + q + 4 v, columns k = k0 + 16 y + i
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t c = c0 + q + 4 * v;
      if (c >= g.cols) continue;
      TZ* zk = Z + (int64_t)g.K * c + k0 + i;
#pragma unroll
      for (int y = 0; y < NB; ++y)
        if (k0 + 16 * y + i < g.K) zk[16 * y] = static_cast<TZ>(acc[0][y][v]);
    }
  }
}

// The whole item with NB blocks along k: accumulators zeroed, all chunks, then
// the stores.
template <int NB, typename TY, typename TZ, int ORI, int MF, int WY>
__device__ __forceinline__ void tile_body(Loader<TY, ORI, MF, WY>& ld, const TtmDmaParams& g, char* buf0, char* buf1,
                                          int oa, int da, int ob, int db, int wave, int lane, int k0, int64_t c0) {
  constexpr int NX = (ORI == 0) ? NB : 1, NY = (ORI == 0) ? 1 : NB;
  d4 acc[NX][NY];
#pragma unroll
  for (int x = 0; x < NX; ++x)
#pragma unroll
    for (int y = 0; y < NY; ++y) acc[x][y] = d4{0.0, 0.0, 0.0, 0.0};
  chunk_loop<NX, NY>(ld, g, buf0, buf1, oa, da, ob, db, acc, wave, lane);
  store_tile<NB, TZ, ORI>(g, acc, k0, c0 + 16 * wave, lane & 15, lane >> 4);
}

// NB: blocks of 16 output rows in the first g.khi row tiles; one fewer in the
// others, so that K is split evenly (469 rows: 8, 8, 7, 7 blocks) and no row
// tile of few blocks pays for a whole chunk's loads and barrier.
template <typename TY, typename TZ, int ORI, int MF, int WY, int NB>
__global__ __launch_bounds__(kTDNT, 4) void ttm_dma_kernel(TtmDmaParams g) {
  using C = Cfg<TY, ORI, MF, WY>;
  __shared__ __attribute__((aligned(16))) char buf0[C::BUF];
  __shared__ __attribute__((aligned(16))) char buf1[C::BUF];
  const int64_t item = xcd_remap(blockIdx.x, gridDim.x, g.total);
  if (item < 0) return;
  const uint32_t ct = (uint32_t)item / (uint32_t)g.nkt;  // total < 2^31
  const int kt = (int)((uint32_t)item - ct * (uint32_t)g.nkt);
  const int k0 = 16 * (kt * NB - max(0, kt - g.khi));
  const int64_t c0 = 128 * (int64_t)ct;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, q = lane >> 4;
  // operand offsets of the lane's first block at step 0 (row form: and the
  // byte distance d to its second unit, whose sign depends on the row's
  // swizzle): all blocks along k, block `wave` along the columns
  using IA = typename std::conditional<ORI == 0, typename C::IM, typename C::IY>::type;
  using IB = typename std::conditional<ORI == 0, typename C::IY, typename C::IM>::type;
  const int ra = (ORI == 0) ? i : 16 * wave + i, rb = (ORI == 0) ? 16 * wave + i : i;
  const int oa = IA::at(ra, IA::jstep(0, q)), ob = IB::at(rb, IB::jstep(0, q));
  const int da = IA::at(ra, IA::jstep(2, q)) - oa, db = IB::at(rb, IB::jstep(2, q)) - ob;
  Loader<TY, ORI, MF, WY> ld;
  loader_init(ld, g, k0, c0, wave, lane);
  if (kt < g.khi) tile_body<NB, TY, TZ, ORI, MF, WY>(ld, g, buf0, buf1, oa, da, ob, db, wave, lane, k0, c0);
  else tile_body<NB - 1, TY, TZ, ORI, MF, WY>(ld, g, buf0, buf1, oa, da, ob, db, wave, lane, k0, c0);
}

}  // namespace

// 16-byte loads of Y need its rows (L = 1: stride J) or slabs (L > 1: the
// element offset L j) 16-byte aligned; otherwise it takes 4-byte loads.
static bool ttm_dma_y16(int J, uint64_t L, int ysize, const void* Y) {
  if (reinterpret_cast<uintptr_t>(Y) % 16) return false;
  if (L == 1) return ((uint64_t)J * ysize) % 16 == 0;
  return L % (16 / ysize) == 0;
}

// M is read in 16-byte units: rows contiguous (msj = 1, row stride a multiple
// of 16 bytes that holds a row) or columns contiguous (msk = 1, column stride likewise; double
// Y only).
static bool ttm_dma_mrow(int J, int64_t msk, int64_t msj) { return msj == 1 && msk % 2 == 0 && msk >= J; }
static bool ttm_dma_m16(int J, int K, int64_t msk, int64_t msj, int ysize, const void* M) {
  if (reinterpret_cast<uintptr_t>(M) % 16) return false;
  return ttm_dma_mrow(J, msk, msj) || (ysize == 8 && msk == 1 && msj % 2 == 0 && msj >= K);
}

// Up to 128 tiles (of 128 x 128) leave half of the CUs without one, and a call
// takes as long as one tile's chain of chunks, in which the register-staged
// kernel of smaller tiles is the faster for float Y, whose values it converts
// once and not at every operand read, from three chunks on.  That kernel
// against this one, in us, rows J -> K of C columns in slabs of 50:
//   626 -> 468: C = 2000 (64 tiles) 64 / 89, 4000 (128) 73 / 91, 8000 (252) 112 / 93
//   336 -> 200: C = 2000 (32) 38 / 44, 8000 (126) 42 / 46, 16000 (250) 70 / 48
//   (slabs of 25) 32 -> 200: C = 1000 (16) 9.5 / 8.8; 16 -> 200: 9.6 / 7.1
// Doubles take this kernel whatever their number.
constexpr int64_t kTDFew = 128;
static int64_t ttm_dma_tiles(int K, uint64_t cols) {
  return ceil_div(ceil_div(K, 16), 8) * ceil_div((int64_t)cols, 128);
}

bool ttm_dma_eligible(int J, uint64_t cols, int K, int64_t msk, int64_t msj, int ysize, const void* Y,
                      const void* M) {
  if (K <= 64 || J < 16 || cols == 0) return false;
  if (ysize == 4 && J > 2 * kJC && ttm_dma_tiles(K, cols) <= kTDFew) return false;
  return ttm_dma_m16(J, K, msk, msj, ysize, M) && reinterpret_cast<uintptr_t>(Y) % ysize == 0;
}

bool ttm_dma_wants_pack(int J, uint64_t cols, int K, int64_t msk, int64_t msj, int ysize, const void* Y,
                        const void* M) {
  if (K <= 64 || J < 16 || cols == 0 || reinterpret_cast<uintptr_t>(Y) % ysize) return false;
  // The launch that lays M out takes 6 us, and moves M twice more: 50 -> 129
  // rows of 2000 columns (2.6e7 flops) 14 us without it and 22 us with it, 50 ->
  // 65 rows of 200000 columns (1.3e9) faster with it; 201 -> 20001 rows of 500
  // columns 126 and 112 us, of 1000 242 and 175 us, but 50 -> 20001 rows of 500
  // slower.  With few tiles it gains nothing even then: 201 -> 201 rows of 8000
  // columns (126 tiles) 31 and 34 us, of 16000 (250) 50 and 35 us.
  if (2.0 * K * J * (double)cols < 1e9 || cols < 1000 || ttm_dma_tiles(K, cols) <= kTDFew) return false;
  return !ttm_dma_m16(J, K, msk, msj, ysize, M);
}

// P(k, j) = M(k, j) for j < J, zero for J <= j < ld, at P[k * ld + j].  Tiles
// of 32 x 32 through LDS, so that both sides run along their contiguous axis.
__global__ __launch_bounds__(256) void pack_factor_kernel(const double* __restrict__ M, int64_t msk, int64_t msj,
                                                          int K, int J, int ld, double* __restrict__ P) {
  __shared__ double t[32][33];
  const int k0 = 32 * blockIdx.y, j0 = 32 * blockIdx.x;
  const int u = threadIdx.x & 31, v = threadIdx.x >> 5;
  const bool alongk = msk < msj;
#pragma unroll
  for (int p = 0; p < 32; p += 8) {
    const int k = alongk ? u : v + p, j = alongk ? v + p : u;
    t[k][j] = (k0 + k < K && j0 + j < J) ? M[(int64_t)(k0 + k) * msk + (int64_t)(j0 + j) * msj] : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 32; p += 8)
    if (k0 + v + p < K && j0 + u < ld) P[(int64_t)(k0 + v + p) * ld + j0 + u] = t[v + p][u];
}

hipError_t launch_pack_factor(const double* M, int64_t msk, int64_t msj, int K, int J, int ld, double* P,
                              hipStream_t stream) {
  if (ld < J || K < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(pack_factor_kernel, dim3(ceil_div(ld, 32), ceil_div(K, 32)), dim3(256), 0, stream, M, msk, msj,
                     K, J, ld, P);
  return hipGetLastError();
}

template <typename TY, typename TZ>
hipError_t launch_ttm_dma(const TY* Y, int J, uint64_t L, uint64_t cols, const double* M, int64_t msk, int64_t msj,
                          int K, TZ* Z, hipStream_t stream, const TtmOutRemap& rm) {
  if (!ttm_dma_eligible(J, cols, K, msk, msj, (int)sizeof(TY), Y, M) || cols >= (uint64_t(1) << 32))
    return hipErrorInvalidValue;
  const bool remap = rm.Pp != rm.Rp;
  if (remap && (L == 1 || rm.Lp < 1 || rm.Rp < 1 || rm.Rp > rm.Pp + 1 || (int64_t)L % (rm.Lp * rm.Pp) != 0))
    return hipErrorInvalidValue;
  TtmDmaParams g{};
  g.Y = reinterpret_cast<const char*>(Y);
  g.M = reinterpret_cast<const char*>(M);
  g.Z = reinterpret_cast<char*>(Z);
  g.J = J;
  g.K = K;
  g.L = (int64_t)L;
  g.cols = (int64_t)cols;
  g.msk = msk;
  g.msj = msj;
  const int nb = (int)ceil_div(K, 16);  // blocks of 16 rows, at least 5
  g.nkt = ceil_div(nb, 8);
  const int nbt = (int)ceil_div(nb, g.nkt);
  g.khi = (int)(nb - (nbt - 1) * g.nkt);
  g.total = g.nkt * ceil_div((int64_t)cols, 128);
  g.Lp = remap ? rm.Lp : 1;
  g.Pp = remap ? rm.Pp : 1;
  g.Rp = remap ? rm.Rp : 1;
  g.Lo = remap ? (int64_t)L / rm.Pp * rm.Rp : (int64_t)L;
  if (g.total >= (int64_t(1) << 31)) return hipErrorInvalidValue;
  const int64_t grid = ceil_div(g.total, kXcds) * kXcds;
  const bool mrow = ttm_dma_mrow(J, msk, msj);
  const bool y16 = ttm_dma_y16(J, L, (int)sizeof(TY), Y);
#define TDMA_R(ORI, MF, WYV, NBV) \
  hipLaunchKernelGGL((ttm_dma_kernel<TY, TZ, ORI, MF, WYV, NBV>), dim3(grid), dim3(kTDNT), 0, stream, g)
#define TDMA_Y(ORI, MF, WYV)                    \
  do {                                          \
    if (nbt == 8) TDMA_R(ORI, MF, WYV, 8);      \
    else if (nbt == 7) TDMA_R(ORI, MF, WYV, 7); \
    else if (nbt == 6) TDMA_R(ORI, MF, WYV, 6); \
    else TDMA_R(ORI, MF, WYV, 5);               \
  } while (0)
#define TDMA_W(ORI, MF)             \
  do {                              \
    if (y16) TDMA_Y(ORI, MF, 16);   \
    else TDMA_Y(ORI, MF, 4);        \
  } while (0)
  if (mrow) {
    if (L == 1) TDMA_W(1, 0);
    else TDMA_W(0, 0);
  } else if constexpr (std::is_same<TY, double>::value) {
    if (L == 1) TDMA_W(1, 1);
    else TDMA_W(0, 1);
  }
#undef TDMA_W
#undef TDMA_Y
#undef TDMA_R
  return hipGetLastError();
}

template hipError_t launch_ttm_dma<double, double>(const double*, int, uint64_t, uint64_t, const double*, int64_t,
                                                   int64_t, int, double*, hipStream_t, const TtmOutRemap&);
template hipError_t launch_ttm_dma<float, double>(const float*, int, uint64_t, uint64_t, const double*, int64_t,
                                                  int64_t, int, double*, hipStream_t, const TtmOutRemap&);
template hipError_t launch_ttm_dma<double, float>(const double*, int, uint64_t, uint64_t, const double*, int64_t,
                                                  int64_t, int, float*, hipStream_t, const TtmOutRemap&);
template hipError_t launch_ttm_dma<float, float>(const float*, int, uint64_t, uint64_t, const double*, int64_t,
                                                 int64_t, int, float*, hipStream_t, const TtmOutRemap&);

}  // namespace tk
