// Device helpers and per-tile shapes shared by the MVM's tile kernels
// (lattice_mvm.hip) and the CG iteration's (cg_tile.h).
#ifndef SGP_TILE_H
#define SGP_TILE_H
#include "sgp_internal.h"

namespace sgp {
namespace {

constexpr int kXcds = 8;

// Logical block for dispatch slot b when blocks are dealt round-robin over
// the XCDs: XCD x runs logical blocks [x*q + min(x, r), ...) contiguously.
__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t nb) {
  const int64_t x = b % kXcds, t = b / kXcds;
  const int64_t q = nb / kXcds, r = nb % kXcds;
  return x * q + (x < r ? x : r) + t;
}

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Column c of a lattice point whose partial rows span the gather ranges g0 ..
// g1: its fragments in range order (the first at `first`), eight in flight
// together: a chain of dependent loads otherwise. 8 CG iterations, 8 columns:
// n = 200,000, d = 6 0.755 -> 0.673 ms, n = 500,000, d = 8 1.015 -> 0.953 ms.
template <typename T>
__device__ __forceinline__ T frag_sum(const T* frag, int64_t first, int64_t g0, int64_t g1, int64_t C, int c) {
  T acc = frag[first];
  for (int64_t g = g0 + 1; g <= g1; g += 8) {
    T v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = frag[(g + u <= g1 ? g + u : g1) * 2 * C + c];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (g + u <= g1) acc += v[u];
  }
  return acc;
}

// 16-byte vectors for LDS and global accesses of lattice and point rows.
typedef double dvec2 __attribute__((ext_vector_type(2)));
typedef float fvec4 __attribute__((ext_vector_type(4)));
template <typename T>
struct Vec16;
template <>
struct Vec16<double> {
  typedef dvec2 T;
  static constexpr int N = 2;
};
template <>
struct Vec16<float> {
  typedef fvec4 T;
  static constexpr int N = 4;
};

// Read (or write) W consecutive elements at p, as 16-byte vectors when W
// elements span whole vectors (p is then 16-byte aligned by construction).
template <typename T, int W>
__device__ __forceinline__ void read_row(const T* p, T (&o)[W]) {
  constexpr int N = Vec16<T>::N;
  if constexpr (W % N == 0) {
#pragma unroll
    for (int i = 0; i < W / N; ++i) {
      const typename Vec16<T>::T x = *(const typename Vec16<T>::T*)(p + i * N);
#pragma unroll
      for (int j = 0; j < N; ++j) o[i * N + j] = x[j];
    }
  } else {
#pragma unroll
    for (int i = 0; i < W; ++i) o[i] = p[i];
  }
}
template <typename T, int W>
__device__ __forceinline__ void write_row(T* p, const T (&v)[W]) {
  constexpr int N = Vec16<T>::N;
  if constexpr (W % N == 0) {
#pragma unroll
    for (int i = 0; i < W / N; ++i) {
      typename Vec16<T>::T x;
#pragma unroll
      for (int j = 0; j < N; ++j) x[j] = v[i * N + j];
      *(typename Vec16<T>::T*)(p + i * N) = x;
    }
  } else {
#pragma unroll
    for (int i = 0; i < W; ++i) p[i] = v[i];
  }
}

// read_row with non-temporal loads
template <typename T, int W>
__device__ __forceinline__ void read_row_nt(const T* p, T (&o)[W]) {
  constexpr int N = Vec16<T>::N;
  if constexpr (W % N == 0) {
#pragma unroll
    for (int i = 0; i < W / N; ++i) {
      const typename Vec16<T>::T x = __builtin_nontemporal_load((const typename Vec16<T>::T*)(p + i * N));
#pragma unroll
      for (int j = 0; j < N; ++j) o[i * N + j] = x[j];
    }
  } else {
#pragma unroll
    for (int i = 0; i < W; ++i) o[i] = __builtin_nontemporal_load(p + i);
  }
}

// write_row with non-temporal stores (streamed past the caches)
template <typename TU, int W>
__device__ __forceinline__ void write_row_nt(TU* p, const TU (&v)[W]) {
  constexpr int N = Vec16<TU>::N;
  if constexpr (W % N == 0) {
#pragma unroll
    for (int i = 0; i < W / N; ++i) {
      typename Vec16<TU>::T x;
#pragma unroll
      for (int j = 0; j < N; ++j) x[j] = v[i * N + j];
      __builtin_nontemporal_store(x, (typename Vec16<TU>::T*)(p + i * N));
    }
  } else {
#pragma unroll
    for (int i = 0; i < W; ++i) __builtin_nontemporal_store(v[i], p + i);
  }
}

// Persistent tile kernels: block b runs on XCD b % 8 and takes work items
// from a contiguous range owned by its XCD, striding over it with the other
// blocks of that XCD.
__device__ __forceinline__ void xcd_items(int64_t items, int64_t* first, int64_t* end, int64_t* step) {
  const int64_t nb = gridDim.x, b = blockIdx.x;
  const int64_t x = b % kXcds, k = b / kXcds;
  const int64_t per = nb / kXcds, rem = nb % kXcds;
  const int64_t before = x * per + (x < rem ? x : rem);
  const int64_t mine = per + (x < rem ? 1 : 0);
  const int64_t lo = items * before / nb;
  const int64_t hi = items * (before + mine) / nb;
  *first = lo + k;
  *end = hi;
  *step = mine;
}

// Per-thread register shapes of the tile kernels (NT threads per block, at
// most 256 points and kMaxTileEntries entries and runs per tile).
constexpr int kMaxTileEntries = 4096;
constexpr int kSplatBlock = 512;   // two blocks per CU
// The slice adds a point's entries by blocks of this many runs of its tile's
// run list; every staged chunk (at most 16 channels) holds a whole number of
// such blocks (RC = 8 NT / G >= 512).
constexpr int kSliceOrderRows = 512;
// Threads per block of k_slice_tile: 1024 (one block per CU), or for narrow
// channel chunks just the lane groups for the 256 points of a tile (LPR =
// G / VW lanes each), so that the lanes are not left idle. The narrow block
// also stages fewer lattice rows per pass (RC = 8 NT / G), so it is taken
// only where a tile's runs mostly fit in one pass.
template <int G>
constexpr int slice_threads_narrow() { return G >= 16 ? 1024 : G == 8 ? 512 : 256; }
template <typename TU, int G, int NT_>
struct TileShape {
  static constexpr int NT = NT_;
  static constexpr int kPts = 256;
  static constexpr int EPT = kMaxTileEntries / NT;  // entries per thread
  static constexpr int VPT = (kPts * G) / NT > 0 ? (kPts * G) / NT : 1;  // point values
  static constexpr int VW = G < 4 ? G : 4;  // channels per lane
  static constexpr int LPR = G / VW;        // lanes per run (splat) or point (slice)
  static constexpr int NG = NT / LPR;
  static constexpr int UPT = 8;             // lattice rows staged per thread in the slice
  static constexpr int RC = UPT * NT / G;   // lattice rows per slice chunk
  static constexpr int PPG = (kPts + NG - 1) / NG;  // points per lane group in the slice
  // LDS row stride in elements: rows of 64 bytes or more get 16 bytes of
  // padding, so lane groups reading different rows spread over the banks
  static constexpr int RS = G * (int)sizeof(TU) >= 64 ? G + 16 / (int)sizeof(TU) : G;
  // point values can be staged as whole 16-byte vectors per thread
  static constexpr bool VEC = VPT >= Vec16<TU>::N && VPT % Vec16<TU>::N == 0;
};

// Lanes of the splat: SLPR lanes of SVW channels sum a piece, so a wave takes
// whole slices of kSlicePieces pieces.
template <int G>
struct SplatLanes {
  static constexpr int LPR = G < 4 ? G : 4;
  static constexpr int VW = G / LPR;
  static constexpr int GPW = 64 / LPR;             // pieces per wave
  static constexpr int SPW = GPW / kSlicePieces;   // slices per wave
};

// The splat's entry lists of a tile in LDS, at byte offsets: weights [maxe]
// (fp32) | row offsets [maxe] (uint16) | partial rows [maxq] (int32) | slices
// [maxq / 16 + 1] (uint32) | next unclaimed batch, then a spare word (int32).
struct SplatLists {
  int w, off, dst, sl, next, end;
};
__host__ __device__ inline SplatLists splat_lists(int base, int maxe, int maxq) {
  SplatLists o;
  int b = (base + 15) & ~15;
  o.w = b;
  b += 4 * maxe;
  o.off = b;
  b += (2 * maxe + 15) & ~15;
  o.dst = b;
  b += 4 * maxq;
  o.sl = b;
  b += 4 * (maxq / kSlicePieces + 1);
  o.next = b;
  o.end = b + 8;
  return o;
}

// The lists of one tile on their way from global memory to LDS: four
// consecutive entries per thread and round. NT * 4 * ROUNDS entries and
// NT * QR pieces travel in registers, the rest of longer lists (tiles with
// very many distinct points) is copied when staged.
template <int NT>
struct SplatFetch {
  static constexpr int ROUNDS = 4096 / (4 * NT);
  static constexpr int QR = NT >= 1024 ? 1 : NT == 512 ? 2 : 4;
  fvec4 w[ROUNDS];
  uint32_t lp[ROUNDS];
  int32_t dst[QR];
  uint32_t sl;
  // Entries are read once per MVM: non-temporal, so that they do not push
  // the partial rows, which the gather reads next, out of the caches.
  __device__ __forceinline__ void load(const float* ew, const uint8_t* elp, const int32_t* run_dst,
                                       const uint32_t* slice, int ne, int nq) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
      const int e4 = tid + u * NT, i = e4 < ne / 4 ? e4 : ne / 4 - 1;
      w[u] = __builtin_nontemporal_load((const fvec4*)ew + i);
      lp[u] = __builtin_nontemporal_load((const uint32_t*)elp + i);
    }
#pragma unroll
    for (int u = 0; u < QR; ++u) {
      const int q = tid + u * NT;
      dst[u] = run_dst[q < nq ? q : nq - 1];
    }
    const int ns = (nq + kSlicePieces - 1) / kSlicePieces;
    sl = slice[tid < ns ? tid : ns - 1];
  }
  // row: bytes of a staged row; pads read the zero row with weight 0
  __device__ __forceinline__ static void put(unsigned char* smem, const SplatLists& l, int i, fvec4 ww, uint32_t p,
                                             int row, int zrow) {
    typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
    u16x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float f = ww[j];
      const bool pad = __float_as_uint(f) == kPadWeight;
      o[j] = (uint16_t)((pad ? zrow : (int)((p >> (8 * j)) & 0xffu)) * row);
      ww[j] = pad ? 0.f : f;
    }
    *(fvec4*)(smem + l.w + 16 * i) = ww;
    *(u16x4*)(smem + l.off + 8 * i) = o;
  }
  __device__ __forceinline__ void stage(unsigned char* smem, const SplatLists& l, const float* ew,
                                        const uint8_t* elp, const int32_t* run_dst, const uint32_t* slice,
                                        int ne, int nq, int row, int zrow) const {
    const int tid = threadIdx.x;
    const int ns = (nq + kSlicePieces - 1) / kSlicePieces;
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
      const int i = tid + u * NT;
      if (i < ne / 4) put(smem, l, i, w[u], lp[u], row, zrow);
    }
    for (int i = tid + ROUNDS * NT; i < ne / 4; i += NT)
      put(smem, l, i, ((const fvec4*)ew)[i], ((const uint32_t*)elp)[i], row, zrow);
#pragma unroll
    for (int u = 0; u < QR; ++u) {
      const int q = tid + u * NT;
      if (q < nq) ((int32_t*)(smem + l.dst))[q] = dst[u];
    }
    for (int q = tid + QR * NT; q < nq; q += NT) ((int32_t*)(smem + l.dst))[q] = run_dst[q];
    if (tid < ns) ((uint32_t*)(smem + l.sl))[tid] = sl;
    for (int q = tid + NT; q < ns; q += NT) ((uint32_t*)(smem + l.sl))[q] = slice[q];
    if (tid == 0) *(int*)(smem + l.next) = NT / 64;  // batches 0 .. NT/64-1 start on a wave each
  }
};

// N entries of a piece, from its lane's position in the lists on: their rows
// are read together and added in entry order.
template <int N, typename TU, int VW>
__device__ __forceinline__ void splat_step(const unsigned char* rows, const uint16_t* po, const float* pw,
                                           TU (&acc)[VW]) {
  TU x[N][VW], w[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    w[u] = (TU)pw[u * kSlicePieces];
    read_row<TU, VW>((const TU*)(rows + po[u * kSlicePieces]), x[u]);
  }
#pragma unroll
  for (int u = 0; u < N; ++u)
#pragma unroll
    for (int i = 0; i < VW; ++i) acc[i] = fma_t(w[u], x[u][i], acc[i]);
}

template <typename TU, int VW>
__device__ __forceinline__ void store_piece(TU* o, const TU (&acc)[VW], int cg, int C, bool cvec) {
  if (cvec && cg + VW <= C) {
    write_row<TU, VW>(o, acc);
  } else {
#pragma unroll
    for (int i = 0; i < VW; ++i)
      if (cg + i < C) o[i] = acc[i];
  }
}

// The pieces of a staged tile: each is summed in entry order and stored as
// its partial row. A wave takes a slice of 16 pieces of about equal length
// (SPW slices where fewer lanes share a piece), claiming its next before it
// sums this one, and steps through the interleaved entries with one address
// per lane. This is bound by instruction issue: with the pieces in run order,
// one lane group per piece, every step waited for whichever of a wave's 16
// groups had just finished a piece to claim, look up and start another, and
// an entry cost ten instructions of addressing and bounds beside its sums.
// A piece's sum does not depend on the wave that takes it.
template <typename TU, int G, int NT>
__device__ __forceinline__ void splat_pieces(const unsigned char* rows, unsigned char* smem, const SplatLists& l,
                                             int nq, TU* part, int C, int c0, bool cvec) {
  using W = SplatLanes<G>;
  const int lane = threadIdx.x & 63, g = lane / W::LPR;
  const int cl = (lane % W::LPR) * W::VW, cg = c0 + cl;
  const uint32_t* lsl = (const uint32_t*)(smem + l.sl);
  const int32_t* ldst = (const int32_t*)(smem + l.dst);
  const unsigned char* lrows = rows + cl * sizeof(TU);
  const int ns = (nq + kSlicePieces - 1) / kSlicePieces;
  int b = (int)(threadIdx.x >> 6);
  while (b * W::SPW < ns) {
    int nx = 0;
    if (lane == 0) nx = atomicAdd((int*)(smem + l.next), 1);
    const int s = b * W::SPW + g / kSlicePieces;
    uint32_t sw = lsl[s < ns ? s : ns - 1];
    if constexpr (W::SPW == 1) sw = __builtin_amdgcn_readfirstlane(sw);
    const int m = s < ns ? (int)(sw >> 16) : 0;
    const int e = (int)(sw & 0xffffu) + g % kSlicePieces;
    const int q = s * kSlicePieces + g % kSlicePieces;
    const int dq = ldst[q < nq ? q : nq - 1];
    const uint16_t* po = (const uint16_t*)(smem + l.off) + e;
    const float* pw = (const float*)(smem + l.w) + e;
    TU acc[W::VW];
#pragma unroll
    for (int i = 0; i < W::VW; ++i) acc[i] = 0;
    int k = 0;
    for (; k + 4 <= m; k += 4, po += 4 * kSlicePieces, pw += 4 * kSlicePieces) splat_step<4>(lrows, po, pw, acc);
    if (k + 2 <= m) {
      splat_step<2>(lrows, po, pw, acc);
      k += 2;
      po += 2 * kSlicePieces;
      pw += 2 * kSlicePieces;
    }
    if (k < m) splat_step<1>(lrows, po, pw, acc);
    if (q < nq && m > 0) store_piece(part + (int64_t)dq * C + cg, acc, cg, C, cvec);
    b = __builtin_amdgcn_readfirstlane(nx);
  }
}

// x of the lane N lanes on within the 16-lane row (0 past its end).
template <int N, typename T>
__device__ __forceinline__ T row_from(T x) {
  if constexpr (sizeof(T) == 8) {
    const long long v = __builtin_bit_cast(long long, x);
    const int lo = __builtin_amdgcn_mov_dpp((int)v, 0x100 + N, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(v >> 32), 0x100 + N, 0xf, 0xf, true);
    return __builtin_bit_cast(T, (long long)hi << 32 | (long long)(unsigned)lo);
  } else {
    return __builtin_bit_cast(T, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x100 + N, 0xf, 0xf, true));
  }
}

// splat_pieces with a piece of more than kShortPiece entries summed by four
// lane groups, kShortPiece entries each, whose sums are added as (0 + 1) +
// (2 + 3) (the four groups share a 16-lane row): the wave that holds a tile's
// longest pieces makes two steps in place of eight and no longer ends last.
// A batch is a quarter of a long slice (a half, or a whole one, with fewer
// lanes per piece), or SPW short slices. A piece's sum depends on its entries
// only, as before.
template <typename TU, int G, int NT>
__device__ __forceinline__ void splat_pieces_split(const unsigned char* rows, unsigned char* smem,
                                                   const SplatLists& l, int nq, TU* part, int C, int c0,
                                                   bool cvec) {
  using W = SplatLanes<G>;
  static_assert(4 * W::LPR <= 16 && 4 * kShortPiece >= kPiece && W::GPW / 4 <= kSlicePieces, "batches of long pieces");
  constexpr int PPB = W::GPW / 4;            // long pieces per batch
  constexpr int BPS = kSlicePieces / PPB;    // batches per long slice
  const int lane = threadIdx.x & 63, g = lane / W::LPR;
  const int cl = (lane % W::LPR) * W::VW, cg = c0 + cl;
  const uint32_t* lsl = (const uint32_t*)(smem + l.sl);
  const int32_t* ldst = (const int32_t*)(smem + l.dst);
  const uint16_t* loff = (const uint16_t*)(smem + l.off);
  const float* lw = (const float*)(smem + l.w);
  const unsigned char* lrows = rows + cl * sizeof(TU);
  const int ns = (nq + kSlicePieces - 1) / kSlicePieces;
  int nl = 0;  // long slices, which come first
  for (int s0 = 0; s0 < ns; s0 += 64) {
    const int s = s0 + lane;
    const unsigned long long bal = __ballot(s < ns && (int)(lsl[s < ns ? s : ns - 1] >> 16) > kShortPiece);
    nl += (int)__popcll(bal);
    if (bal != ~0ull) break;
  }
  const int nbl = nl * BPS;
  const int nb = nbl + (ns - nl + W::SPW - 1) / W::SPW;
  int b = NT / 64 - 1 - (int)(threadIdx.x >> 6);
  while (b < nb) {
    int nx = 0;
    if (lane == 0) nx = atomicAdd((int*)(smem + l.next), 1);
    TU acc[W::VW];
#pragma unroll
    for (int i = 0; i < W::VW; ++i) acc[i] = 0;
    if (b < nbl) {
      const int s = b / BPS, c = (b % BPS) * PPB + g / 4, off = g % 4 * kShortPiece;
      const uint32_t sw = __builtin_amdgcn_readfirstlane(lsl[s]);
      const int m = (int)(sw >> 16) - off;  // a multiple of 4
      const int e = (int)(sw & 0xffffu) + off * kSlicePieces + c;
      const int q = s * kSlicePieces + c;
      const int dq = ldst[q < nq ? q : nq - 1];
      if (m > 0) splat_step<4>(lrows, loff + e, lw + e, acc);
      if (m > 4) splat_step<4>(lrows, loff + e + 4 * kSlicePieces, lw + e + 4 * kSlicePieces, acc);
#pragma unroll
      for (int i = 0; i < W::VW; ++i) acc[i] += row_from<W::LPR>(acc[i]);
#pragma unroll
      for (int i = 0; i < W::VW; ++i) acc[i] += row_from<2 * W::LPR>(acc[i]);
      if (off == 0 && q < nq) store_piece(part + (int64_t)dq * C + cg, acc, cg, C, cvec);
    } else {
      const int s = nl + (b - nbl) * W::SPW + g / kSlicePieces;
      uint32_t sw = lsl[s < ns ? s : ns - 1];
      if constexpr (W::SPW == 1) sw = __builtin_amdgcn_readfirstlane(sw);
      const int m = s < ns ? (int)(sw >> 16) : 0;  // at most kShortPiece
      const int e = (int)(sw & 0xffffu) + g % kSlicePieces;
      const int q = s * kSlicePieces + g % kSlicePieces;
      const int dq = ldst[q < nq ? q : nq - 1];
      const uint16_t* po = loff + e;
      const float* pw = lw + e;
      int k = 0;
      for (; k + 4 <= m; k += 4, po += 4 * kSlicePieces, pw += 4 * kSlicePieces) splat_step<4>(lrows, po, pw, acc);
      if (k + 2 <= m) {
        splat_step<2>(lrows, po, pw, acc);
        k += 2;
        po += 2 * kSlicePieces;
        pw += 2 * kSlicePieces;
      }
      if (k < m) splat_step<1>(lrows, po, pw, acc);
      if (q < nq && m > 0) store_piece(part + (int64_t)dq * C + cg, acc, cg, C, cvec);
    }
    b = __builtin_amdgcn_readfirstlane(nx);
  }
}

// Sum over the 256 rows of a tile's staged fp64 values of the squares of
// column c (rows from np on count as zero), for lane blk of a 16-lane row:
// lane 0 gets the sum. Lane blk adds rows 16 blk + (blk + u) % 16 in turn (16
// padded rows apart they would share an LDS bank), then the lanes' sums are
// added pairwise.
template <int RS>
__device__ __forceinline__ double tile_sumsq(const double* lv, int blk, int c, int np) {
  double v = 0.0;
  asm volatile("" : "+v"(blk));  // keeps the 16 addresses out of the caller's loop-long registers
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int q = blk * 16 + ((blk + u) & 15);
    const double x = lv[q * RS + c];  // rows of an earlier tile are discarded
    const double y = q < np ? x : 0.0;
    v = __builtin_fma(y, y, v);
  }
  v += row_from<8>(v);
  v += row_from<4>(v);
  v += row_from<2>(v);
  v += row_from<1>(v);
  return v;
}

// Sum of squares of column c over rows 16 blk .. 16 blk + 15 (those below
// np), in row order, of a tile's staged fp64 values.
template <int RS, typename TU>
__device__ __forceinline__ double block_sumsq(const TU* lv, int blk, int c, int np) {
  double v = 0.0;
  asm volatile("" : "+v"(blk));  // keeps the 16 addresses out of the caller's loop-long registers
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int q = blk * 16 + u;
    const double x = q < np ? (double)lv[q * RS + c] : 0.0;
    v = __builtin_fma(x, x, v);
  }
  return v;
}

}  // namespace
}  // namespace sgp
#endif  // SGP_TILE_H
