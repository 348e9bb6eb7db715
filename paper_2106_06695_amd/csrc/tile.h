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
  static constexpr int RPT = 2;                      // runs prefetched per thread (splat)
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

// LDS layout of k_splat_tile: values [P+1][G] (TU; row P stays zero) | weights [P*D] (fp32) |
// partial rows [maxq] (int32) | pieces [maxq] (uint32) | entry points [P*D]
// (uint8) | next unclaimed piece (int32).
struct SplatLds {
  size_t w, dst, pc, lp, next, total;
};
template <typename TU>
__host__ __device__ inline SplatLds splat_lds(int P, int D, int maxq, int G) {
  SplatLds o;
  const int rs = G * (int)sizeof(TU) >= 64 ? G + 16 / (int)sizeof(TU) : G;
  size_t b = sizeof(TU) * (size_t)(P + 1) * rs;
  o.w = b;
  b += sizeof(float) * (size_t)P * D;
  o.dst = b;
  b += sizeof(int32_t) * (size_t)maxq;
  o.pc = b;
  b += sizeof(uint32_t) * (size_t)maxq;
  o.lp = b;
  b += ((size_t)P * D + 3) & ~(size_t)3;
  o.next = b;
  b += sizeof(int);
  o.total = (b + 15) & ~(size_t)15;
  return o;
}

// A piece as the build stores it: first entry within its tile, length.
__device__ __forceinline__ int piece_start(uint32_t pc) { return (int)(pc & 0xffffu); }
__device__ __forceinline__ int piece_len(uint32_t pc) { return (int)(pc >> 16); }

// The pieces of a staged tile: each is summed in entry order by LPR lanes of
// VW channels and stored as its partial row. A wave takes 64 / LPR
// consecutive pieces at a time, claiming the next batch (lnext) before it
// sums this one. Pieces are stored longest first, so the pieces of a batch
// are about equally long and the wave runs one uniform loop of passes of
// four entries; with pieces in run order every pass of a wave waited for
// whichever of its 16 groups had just finished a piece to claim, look up and
// start another (a dependent chain of four LDS accesses): at n = 2M, d = 11,
// C = 16 (306 pieces of 1 to 32 entries a tile) that took 4 to 7 us of a
// tile's 14. k_splat_tile there: fp32 156 -> 118 us, fp64 with the direction
// update 287 -> 262 us (now at the copy rate of its HBM bytes).
// Entries past a piece's end read the zero row with weight 0: fma(0, 0, acc)
// is acc exactly, as acc is never -0. A piece's sum does not depend on the
// wave that takes it.
template <typename TU, typename S>
__device__ __forceinline__ void splat_pieces(const TU* lv, int zrow, const float* lw, const uint8_t* llp,
                                             const uint32_t* lpc, const int32_t* ldst, int* lnext, int nq,
                                             TU* part, int C, int c0, bool cvec) {
  constexpr int GPW = 64 / S::LPR;  // pieces per wave
  const int lane = threadIdx.x & 63, g = lane / S::LPR;
  const int cl = (lane % S::LPR) * S::VW, cg = c0 + cl;
  int q0 = (int)(threadIdx.x >> 6) * GPW;
  while (q0 < nq) {
    int nx = 0;
    if (lane == 0) nx = atomicAdd(lnext, GPW);
    const int q = q0 + g < nq ? q0 + g : nq - 1;
    const uint32_t pc = lpc[q];
    const int dq = ldst[q];
    const int e0 = piece_start(pc), len = q0 + g < nq ? piece_len(pc) : 0;
    // the wave's first piece is its longest
    const int passes = (__builtin_amdgcn_readfirstlane(len) + 3) / 4;
    int lp[4];
    float wv[4];
    auto entries = [&](int p) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = 4 * p + u;
        const int e = e0 + (i < len ? i : 0);
        const int l = (int)llp[e];
        const float w = lw[e];
        lp[u] = i < len ? l : zrow;
        wv[u] = i < len ? w : 0.f;
      }
    };
    TU acc[S::VW];
#pragma unroll
    for (int i = 0; i < S::VW; ++i) acc[i] = 0;
    entries(0);
    for (int p = 0; p < passes; ++p) {
      TU x[4][S::VW], w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        read_row<TU, S::VW>(lv + lp[u] * S::RS + cl, x[u]);
        w[u] = (TU)wv[u];
      }
      if (p + 1 < passes) entries(p + 1);  // while the rows arrive
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < S::VW; ++i) acc[i] = fma_t(w[u], x[u][i], acc[i]);
    }
    if (len > 0) {
      TU* o = part + (int64_t)dq * C + cg;
      if (cvec && cg + S::VW <= C) {
        write_row<TU, S::VW>(o, acc);
      } else {
#pragma unroll
        for (int i = 0; i < S::VW; ++i)
          if (cg + i < C) o[i] = acc[i];
      }
    }
    q0 = __builtin_amdgcn_readfirstlane(nx);
  }
}

// Sum of squares of column c over rows 16 blk .. 16 blk + 15 (those below
// np), in row order, of a tile's staged fp64 values.
template <int RS, typename TU>
__device__ __forceinline__ double block_sumsq(const TU* lv, int blk, int c, int np) {
  double v = 0.0;
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
