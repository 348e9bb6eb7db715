// The lattice MVM  out = outputscale * W_X K_UU W_X^T V  (Section 4, eq. ski_to_bf).
//
// Everything runs in the lattice's internal order: points sorted by their
// remainder-0 lattice point, lattice points numbered by first touch in that
// order, sorted points cut into tiles of at most 256 points, and each tile
// carrying the ascending list of lattice points it touches (its runs).
//   k_splat_tile    W^T restricted to one tile: the tile's values are staged
//                   in LDS and every run sums its entries from there
//                   (Section 3.2, Splat), giving one partial row per run
//   k_splat_gather  U[j] = sum of the partial rows of lattice point j over
//                   the tiles that touch it
//   k_blur          one step of the blur along one lattice direction per
//                   chain: U'[j] = sum_t stencil[t] U[nbr(j, k, t)], missing
//                   neighbours contributing zero (Section 3.2, Blur). In
//                   SYMMETRIC order one thread advances the forward chain
//                   (direction step) and the reverse chain (direction d-step)
//                   of its row, and the last step stores their sum.
//   k_slice_tile    out = scale * W U: the tile's lattice rows are staged in
//                   LDS, every point combines its d+1 rows from there
//                   (Section 3.2, Slice); the CG variant adds noise * p and
//                   emits per-tile partial sums of p . out per column.
// Every sum runs in a fixed order: no atomics, results independent of
// scheduling. Values in the caller's point order are reached through the
// permutation (rows of V gathered when staged, rows of out scattered); the
// CG solver keeps its vectors in internal order and skips it.
//
// Channels are processed in chunks of G (a power of two <= 16) chosen so
// that the staged rows fit the LDS budget; chunks are the grid's y axis.
// Row ranges of consecutive blocks go to the same XCD (blocks are dealt
// round-robin over the 8 XCDs), so tiles that share lattice points share
// an L2.
#include <algorithm>
#include <mutex>
#include <type_traits>
#include <vector>

#include "cg_step.h"
#include "cg_tile.h"
#include "lattice_col.h"
#include "sgp_internal.h"
#include "tile.h"

namespace sgp {
namespace {

// Scalars of k_splat_tile; its arrays are separate non-aliasing kernel
// arguments, so uniform loads (tile offsets) go through the scalar cache
// and never wait behind the tile's vector loads.
template <typename TU>
struct SplatArgs {
  int64_t n;
  int64_t items;  // tiles x channel chunks
  int P, D, C, chunks;
  int vec_v;  // V rows of a tile are one contiguous run of 16-byte vectors
  int vec_perm;  // V rows, reached through perm, are whole 16-byte vectors (C == G)
  int cvec;   // rows of C channels start 16-byte aligned
  double pp_scale;  // CG: factor of each tile's p . p (the noise variance)
  int estride;  // entries between tiles' lists
  SplatLists lds;  // after the values [P+1][G] (TU; row P stays zero)
};

// W^T restricted to one tile (Section 3.2, Splat). The block stages the
// tile's values, entries and pieces in LDS from registers that were loaded
// while the previous tile was being reduced, and splat_pieces sums every
// piece into its partial row (run_dst).
//
// Inside CG (up.p set, fp64) the values are the direction p in internal
// order, and the block applies the previous iteration's direction update to
// each tile as it stages it (CgDirUpdate): every (point, column) of p is
// read once here anyway, so x and p move without a pass of their own. Each
// element is read and written by the one thread that stages it; the new p
// is what the tile splats.
// DIR: the fused variant; it is launched only where a tile's values are
// all C == G columns of the direction in internal order (and whole 16-byte
// vectors, vec_v, where the shape stages vectors).
// pp (CG, else null): row t receives pp_scale * p.p of tile t per column,
// from the staged values.
template <typename TU, int G, bool DIR>
__global__ __launch_bounds__(kSplatBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_splat_tile(
    const int32_t* __restrict__ tile_off, const int32_t* __restrict__ tile_ent,
    const uint32_t* __restrict__ slice,
    const int32_t* __restrict__ run_dst, const uint8_t* __restrict__ ent_lp,
    const float* __restrict__ ent_w, const TU* __restrict__ V, const uint32_t* __restrict__ perm,
    TU* __restrict__ part, double* __restrict__ pp, SplatArgs<TU> a, CgDirUpdate up) {
  using S = TileShape<TU, G, kSplatBlock>;
  extern __shared__ __align__(16) unsigned char smem[];
  // CG: alpha, beta and the active flags of the columns, for the update
  __shared__ double s_alpha[DIR ? kMaxCgCols : 1], s_beta[DIR ? kMaxCgCols : 1];
  __shared__ int s_active[DIR ? kMaxCgCols : 1];
  constexpr bool upd = DIR && sizeof(TU) == 8 && S::VEC;
  TU* lv = (TU*)smem;
  const int tid = threadIdx.x;
  constexpr int N = Vec16<TU>::N;

  TU v[S::VPT];
  SplatFetch<kSplatBlock> lists;
  int nq = 0, ne = 0, np = 0, q0 = 0;
  // Every load below is unconditional (indices clamped into the tile), so
  // the whole tile is in flight at once. The values are read once per MVM:
  // non-temporal, as the lists (SplatFetch).
  auto fetch = [&](int64_t item) {
    const int64_t t = item / a.chunks;
    const int ch = (int)(item - t * a.chunks);
    const int64_t p0 = t * a.P;
    np = (int)(a.n - p0 < a.P ? a.n - p0 : a.P);
    ne = tile_ent[t];
    q0 = tile_off[t];
    nq = tile_off[t + 1] - q0;
    if (S::VEC && (DIR || a.vec_v)) {
      const typename Vec16<TU>::T* src = (const typename Vec16<TU>::T*)(V + p0 * a.C);
      const int nvec = np * G / N;
#pragma unroll
      for (int u = 0; u < S::VPT / N; ++u) {
        const int vi = tid + u * kSplatBlock;
        const typename Vec16<TU>::T x = __builtin_nontemporal_load(src + (vi < nvec ? vi : nvec - 1));
#pragma unroll
        for (int j = 0; j < N; ++j) v[u * N + j] = x[j];
      }
    } else if (S::VEC && a.vec_perm) {
      // rows in the caller's order: 16-byte vectors of one row each
      const int nvec = np * G / N;
#pragma unroll
      for (int u = 0; u < S::VPT / N; ++u) {
        const int vi = tid + u * kSplatBlock;
        const int f = (vi < nvec ? vi : nvec - 1) * N;
        const int64_t src = (int64_t)perm[p0 + f / G];
        const typename Vec16<TU>::T x =
            __builtin_nontemporal_load((const typename Vec16<TU>::T*)(V + src * a.C + f % G));
#pragma unroll
        for (int j = 0; j < N; ++j) v[u * N + j] = x[j];
      }
    } else {
#pragma unroll
      for (int u = 0; u < S::VPT; ++u) {
        const int f = tid + u * kSplatBlock;
        const int p = f / G < np ? f / G : np - 1;
        const int c = ch * G + f % G;
        const int64_t pt = p0 + p;
        const int64_t src = perm ? (int64_t)perm[pt] : pt;
        v[u] = V[src * a.C + (c < a.C ? c : a.C - 1)];
      }
    }
    lists.load(ent_w + t * a.estride, ent_lp + t * a.estride, run_dst + q0, slice + tile_slice0(q0, t), ne, nq);
  };

  __shared__ double sh_pp[sizeof(TU) == 8 ? 16 * G : 1];
  int64_t pp_item = -1;  // the item whose block sums sh_pp holds
  auto finish_pp = [&]() {
    if (pp_item < 0 || tid >= G) return;
    const int c = (int)(pp_item % a.chunks) * G + tid;
    double tot = 0.0;
#pragma unroll
    for (int b = 0; b < 16; ++b) tot += sh_pp[b * G + tid];
    if (c < a.C) pp[pp_item / a.chunks * a.C + c] = a.pp_scale * tot;
  };
  int64_t item, end, step;
  xcd_items(a.items, &item, &end, &step);
  for (int i = tid; i < S::RS; i += kSplatBlock) lv[a.P * S::RS + i] = (TU)0;  // the zero row
  if constexpr (upd) {
    for (int c = tid; c < a.C && c < kMaxCgCols; c += kSplatBlock) {
      s_alpha[c] = up.st->alpha[c];
      s_beta[c] = up.st->beta[c];
      s_active[c] = up.st->active[c];
    }
  }
  if (item < end) fetch(item);
  for (; item < end; item += step) {
    const int cur_nq = nq, cur_ne = ne, cur_np = np, cur_q0 = q0;
    __syncthreads();  // the previous tile's pieces are done with the LDS
    if constexpr (sizeof(TU) == 8) {
      if (pp) finish_pp();
    }
    if (S::VEC && (DIR || a.vec_v || a.vec_perm)) {
      const int64_t p0 = (item / a.chunks) * a.P;
#pragma unroll
      for (int u = 0; u < S::VPT / N; ++u) {
        const int vi = tid + u * kSplatBlock;
        if (vi * N < cur_np * G) {
          typename Vec16<TU>::T x;
          const int f = vi * N;  // N consecutive elements of one row
          if constexpr (upd) {
            // C == G here: element f of the tile is column f % G of row f / G
            typedef float fvN __attribute__((ext_vector_type(N)));
            const int64_t e = p0 * a.C + f;
            // r and x are read once here and p, x next read by other
            // kernels: streamed past the caches (non-temporal), which keeps
            // the partial rows that the gather reads next in them
            const typename Vec16<TU>::T r2 =
                __builtin_nontemporal_load((const typename Vec16<TU>::T*)((const TU*)up.r + e));
            const fvN x2 = __builtin_nontemporal_load((const fvN*)(up.x + e));
            typename Vec16<TU>::T pn;
            fvN xn;
#pragma unroll
            for (int j = 0; j < N; ++j) {
              const int c = (f + j) % G;
              const TU pold = v[u * N + j];
              xn[j] = (float)__builtin_fma(s_alpha[c], (double)pold, (double)x2[j]);
              pn[j] = s_active[c] ? (TU)__builtin_fma(s_beta[c], (double)pold, (double)r2[j]) : pold;
            }
            __builtin_nontemporal_store(pn, (typename Vec16<TU>::T*)((TU*)up.p + e));
            __builtin_nontemporal_store(xn, (fvN*)(up.x + e));
            x = pn;
          } else {
#pragma unroll
            for (int j = 0; j < N; ++j) x[j] = v[u * N + j];
          }
          *(typename Vec16<TU>::T*)(lv + (f / G) * S::RS + f % G) = x;
        }
      }
    } else {
      const int64_t p0 = (item / a.chunks) * a.P;
#pragma unroll
      for (int u = 0; u < S::VPT; ++u) {
        const int f = tid + u * kSplatBlock;
        if (f < cur_np * G) {
          TU x = v[u];
          if constexpr (DIR && sizeof(TU) == 8 && !S::VEC) {
            // the direction update element by element (C == G here)
            const int c = f % G;
            const int64_t e = p0 * a.C + f;
            const TU pold = x;
            const double rv = __builtin_nontemporal_load((const TU*)up.r + e);
            const float xv = __builtin_nontemporal_load(up.x + e);
            x = up.st->active[c] ? (TU)__builtin_fma(up.st->beta[c], (double)pold, rv) : pold;
            __builtin_nontemporal_store(x, (TU*)up.p + e);
            __builtin_nontemporal_store((float)__builtin_fma(up.st->alpha[c], (double)pold, (double)xv), up.x + e);
          }
          lv[(f / G) * S::RS + f % G] = x;
        }
      }
    }
    {
      const int64_t t = item / a.chunks;
      lists.stage(smem, a.lds, ent_w + t * a.estride, ent_lp + t * a.estride, run_dst + cur_q0,
                  slice + tile_slice0(cur_q0, t), cur_ne, cur_nq, S::RS * (int)sizeof(TU), a.P);
    }
    __syncthreads();
    if (item + step < end) fetch(item + step);  // in flight while this tile is reduced

    if constexpr (sizeof(TU) == 8) {
      if (pp) {
        // CG: the tile's p . p per column from the staged values, its points
        // in 16 blocks of 16 added in index order, so that the sum does not
        // depend on the channel chunk. Consecutive lanes take consecutive
        // columns of one block (a column's blocks are 16 padded rows apart,
        // the same LDS bank); finish_pp adds the blocks after the next barrier.
        if (tid < 16 * G) sh_pp[tid] = block_sumsq<S::RS>(lv, tid / G, tid % G, cur_np);
        pp_item = item;
      }
    }

    splat_pieces<TU, G, kSplatBlock>(smem, smem, a.lds, cur_nq, part, a.C, (int)(item % a.chunks) * G,
                                     a.cvec != 0);
  }
  if constexpr (sizeof(TU) == 8) {
    __syncthreads();
    if (pp) finish_pp();
  }
}

// U[j] = sum of lattice point j's partial rows occ_ptr[j] .. occ_ptr[j+1]-1
// (one per piece of a run touching it, contiguous; row_vert names each row's
// lattice point). The rows are cut into ranges of R rows (gather_rows); a
// group of G lanes adds its range's rows in order, eight rows loaded at a
// time.
// A lattice point whose rows lie in one range is written directly; the part
// of a longer one that a range holds becomes a fragment (slot 0: it starts
// the range; slot 1: it ends the range), summed in range order by
// k_gather_fix. The work per group is fixed, whatever the list lengths.
// VW channels per lane (16-byte loads when the rows allow), G / VW lanes per
// group; every channel's rows are added in the same order for any VW.
// AHEAD: a batch's lattice points are requested with the batch before it.
// BETA (lattice CG, AHEAD): U = sum + beta U per column; a batch's old U rows are
// then requested with its partial rows, so that no load waits for another:
// m = 141,000, 16 fp64 columns 76 -> 67 us (2.2M rows, 4.1 TB/s), m = 80,000,
// 8 columns 32 -> 26 us.
template <typename TU, int G, int VW, bool AHEAD, bool BETA>
__global__ __launch_bounds__(kBlock) void k_splat_gather(const int32_t* __restrict__ row_vert,
                                                         const TU* __restrict__ part,
                                                         TU* U, TU* __restrict__ frag,
                                                         int64_t nrows, int C, int64_t ngroups, int R,
                                                         const double* __restrict__ beta) {
  static_assert(AHEAD || !BETA, "the old rows are found by the points requested ahead");
  constexpr int LG = G / VW;       // lanes per group
  constexpr int GPB = kBlock / LG;  // groups per block
  constexpr int B = 8;              // rows loaded together
  const int lane = threadIdx.x % LG;
  const int64_t gi = xcd_block(blockIdx.x, gridDim.x) * GPB + threadIdx.x / LG;
  if (gi >= ngroups) return;
  const int64_t o0 = gi * R;
  const int64_t o1 = o0 + R < nrows ? o0 + R : nrows;
  // a segment is a whole lattice point unless it touches a range edge that
  // its lattice point continues across
  const int32_t before = o0 > 0 ? row_vert[o0 - 1] : -1;
  const int32_t after = o1 < nrows ? row_vert[o1] : -1;
  if constexpr (!AHEAD) {
    for (int c = lane * VW; c < C; c += G) {
      int32_t cur = row_vert[o0];
      int64_t seg = o0;
      TU acc[VW];
#pragma unroll
      for (int i = 0; i < VW; ++i) acc[i] = 0;
      auto flush = [&](int64_t end) {
        const bool whole = (seg > o0 || before != cur) && (end < o1 || after != cur);
        TU* dst = whole ? U + (int64_t)cur * C + c : frag + (gi * 2 + (seg == o0 ? 0 : 1)) * C + c;
        write_row<TU, VW>(dst, acc);
      };
      for (int64_t k0 = o0; k0 < o1; k0 += B) {
        TU v[B][VW];
        int32_t rv[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
          const int64_t k = k0 + u < o1 ? k0 + u : o1 - 1;
          // partial rows are read once: non-temporal, which keeps the
          // lattice values the blur reads next in the caches
          read_row_nt<TU, VW>(part + k * C + c, v[u]);
          rv[u] = row_vert[k];
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
          if (k0 + u < o1) {
            if (rv[u] != cur) {
              flush(k0 + u);
              cur = rv[u];
              seg = k0 + u;
#pragma unroll
              for (int i = 0; i < VW; ++i) acc[i] = 0;
            }
#pragma unroll
            for (int i = 0; i < VW; ++i) acc[i] += v[u][i];
          }
        }
      }
      flush(o1);
    }
  } else {
    for (int c = lane * VW; c < C; c += G) {
      int64_t seg = o0;
      TU acc[VW], bt[VW];
#pragma unroll
      for (int i = 0; i < VW; ++i) {
        acc[i] = 0;
        bt[i] = BETA ? (TU)beta[c + i] : (TU)0;
      }
      int32_t rv[B + 1];  // a batch's lattice points, and the next row's
#pragma unroll
      for (int u = 0; u < B; ++u) rv[u] = row_vert[o0 + u < o1 ? o0 + u : o1 - 1];
      for (int64_t k0 = o0; k0 < o1; k0 += B) {
        TU v[B][VW], old[BETA ? B : 1][VW];
        int32_t rn[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
          const int64_t k = k0 + u < o1 ? k0 + u : o1 - 1;
          // partial rows are read once: non-temporal, which keeps the
          // lattice values the blur reads next in the caches
          read_row_nt<TU, VW>(part + k * C + c, v[u]);
        }
        if constexpr (BETA) {
#pragma unroll
          for (int u = 0; u < B; ++u) read_row<TU, VW>(U + (int64_t)rv[u] * C + c, old[u]);
        }
#pragma unroll
        for (int u = 0; u < B; ++u) rn[u] = row_vert[k0 + B + u < o1 ? k0 + B + u : o1 - 1];
        rv[B] = rn[0];
#pragma unroll
        for (int u = 0; u < B; ++u) {
          const int64_t k = k0 + u;
          if (k < o1) {
#pragma unroll
            for (int i = 0; i < VW; ++i) acc[i] += v[u][i];
          }
          if (k >= o1 || (k + 1 < o1 && rv[u + 1] == rv[u])) continue;
          const bool whole = (seg > o0 || before != rv[u]) && (k + 1 < o1 || after != rv[u]);
          TU* dst = whole ? U + (int64_t)rv[u] * C + c : frag + (gi * 2 + (seg == o0 ? 0 : 1)) * C + c;
          if (BETA && whole) {
#pragma unroll
            for (int i = 0; i < VW; ++i) acc[i] = fma_t(bt[i], old[BETA ? u : 0][i], acc[i]);
          }
          write_row<TU, VW>(dst, acc);
          seg = k + 1;
#pragma unroll
          for (int i = 0; i < VW; ++i) acc[i] = 0;
        }
#pragma unroll
        for (int u = 0; u < B; ++u) rv[u] = rn[u];
      }
    }
  }
}

// Lattice points whose rows span several ranges: each is summed from its
// fragments in range order by the range its rows end in (one thread per
// (range, channel); a range's first row belongs to the lattice point that
// may continue into it).
__global__ __launch_bounds__(kBlock) void k_gather_fix(const int32_t* __restrict__ row_vert,
                                                       const int32_t* __restrict__ occ_ptr,
                                                       const void* __restrict__ frag_v,
                                                       void* __restrict__ U_v, int64_t ngroups, int C,
                                                       int elem, int R, const double* __restrict__ beta) {
  const int64_t total = ngroups * C;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < total; q += stride) {
    const int64_t g1 = q / C;
    const int c = (int)(q - g1 * C);
    if (g1 == 0) continue;
    const int64_t j = row_vert[g1 * R];
    const int64_t js = occ_ptr[j], je = occ_ptr[j + 1];
    const int64_t g0 = js / R;
    if (g0 == g1 || (je - 1) / R != g1) continue;  // starts here, or ends further on
    const int64_t first = (g0 * 2 + (js == g0 * R ? 0 : 1)) * C + c;
    if (elem == 8) {
      const double acc = frag_sum((const double*)frag_v, first, g0, g1, C, c);
      double* dst = (double*)U_v + j * C + c;
      *dst = beta ? fma_t(beta[c], *dst, acc) : acc;
    } else {
      ((float*)U_v)[j * C + c] = frag_sum((const float*)frag_v, first, g0, g1, C, c);
    }
  }
}

template <typename TU>
struct BlurArgs {
  const TU* in[2];
  TU* out[2];
  const int32_t* nbr[2];  // this step's direction per chain: [point][offset], 2r per point
  int64_t m;
  int C;
  int r;
  int chains;
  int sum_out;  // last SYMMETRIC step: out[0] = forward + reverse
  int vec;      // rows of C channels start 16-byte aligned
  int nt;       // lattice values exceed the Infinity Cache: stream the outputs past it
  int64_t rows_per_block;
  TU st[2 * kMaxOrder + 1];
};

// One chain's blur of VW channels of row j: sum over t = -r..r of
// stencil[t] * U[neighbour(j, t)], in t order; a missing neighbour adds 0.
template <typename TU, int VW>
__device__ __forceinline__ void load_vw(const TU* __restrict__ in, int64_t row, int64_t valid, int C, int c,
                                        bool vec, TU (&v)[VW]);

template <typename TU, int VW>
__device__ __forceinline__ void blur_rows(const TU* __restrict__ in, const int32_t* __restrict__ nb,
                                          int64_t j, int C, int c, int r, const TU* st, bool vec,
                                          TU (&acc)[VW]) {
#pragma unroll
  for (int i = 0; i < VW; ++i) acc[i] = 0;
  if (r == 1) {
    // the three-tap stencil: both neighbour indices (one 8-byte load), then
    // the three rows, in flight together
    const int2 lh = *(const int2*)(nb + 2 * j);
    const int64_t lo = lh.x, hi = lh.y;
    TU v[3][VW];
    load_vw<TU, VW>(in, lo, j, C, c, vec, v[0]);
    load_vw<TU, VW>(in, j, j, C, c, vec, v[1]);
    load_vw<TU, VW>(in, hi, j, C, c, vec, v[2]);
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int i = 0; i < VW; ++i) acc[i] = fma_t(st[t], v[t][i], acc[i]);
    return;
  }
  // neighbour rows first (2r independent loads), then the values
  int32_t nbv[2 * kMaxOrder];
  for (int ti = 0; ti < 2 * r; ++ti) nbv[ti] = nb[j * (2 * r) + ti];
  int ti = 0;
  for (int t = -r; t <= r; ++t) {
    const int64_t row = t == 0 ? j : (int64_t)nbv[ti++];
    TU v[VW];
    load_vw<TU, VW>(in, row, j, C, c, vec, v);
#pragma unroll
    for (int i = 0; i < VW; ++i) acc[i] = fma_t(st[t + r], v[i], acc[i]);
  }
}

template <int G>
__host__ __device__ constexpr int blur_vw() { return G < 4 ? G : 4; }

// One thread per (row, VW channels).
template <typename TU, int G>
__global__ __launch_bounds__(kBlock) void k_blur(BlurArgs<TU> a) {
  constexpr int VW = blur_vw<G>();
  constexpr int LPR = G / VW;
  constexpr int R = kBlock / LPR;
  const int sub = threadIdx.x % LPR;
  const int64_t j0 = xcd_block(blockIdx.x, gridDim.x) * a.rows_per_block;
  const int64_t j1 = j0 + a.rows_per_block < a.m ? j0 + a.rows_per_block : a.m;
  for (int64_t j = j0 + threadIdx.x / LPR; j < j1; j += R) {
    for (int c = sub * VW; c < a.C; c += G) {
      const bool vec = a.vec && c + VW <= a.C;
      TU f[VW];
      blur_rows<TU, VW>(a.in[0], a.nbr[0], j, a.C, c, a.r, a.st, vec, f);
      if (a.chains == 2) {
        TU b[VW];
        blur_rows<TU, VW>(a.in[1], a.nbr[1], j, a.C, c, a.r, a.st, vec, b);
        if (a.sum_out) {
#pragma unroll
          for (int i = 0; i < VW; ++i) f[i] = f[i] + b[i];
        } else {
          TU* o1 = a.out[1] + j * a.C + c;
          if (vec) {
            if (a.nt)
              write_row_nt<TU, VW>(o1, b);
            else
              write_row<TU, VW>(o1, b);
          } else {
#pragma unroll
            for (int i = 0; i < VW; ++i)
              if (c + i < a.C) o1[i] = b[i];
          }
        }
      }
      TU* o0 = a.out[0] + j * a.C + c;
      if (vec) {
        if (a.nt)
          write_row_nt<TU, VW>(o0, f);
        else
          write_row<TU, VW>(o0, f);
      } else {
#pragma unroll
        for (int i = 0; i < VW; ++i)
          if (c + i < a.C) o0[i] = f[i];
      }
    }
  }
}

// Two consecutive blur steps in one launch, for a 3-tap stencil (r = 1):
// out(j) = sum over t2 of st[t2] * B(neighbour2(j, t2)), where B(x) = sum
// over t1 of st[t1] * in(neighbour1(x, t1)) is the first step's value at x,
// formed here in the same order as a launch of its own would form it (a
// missing lattice point contributes 0). Nine rows per output row instead of
// two launches of three; the rows mostly come from L2 and MALL.
template <typename TU>
struct Blur2Args {
  const TU* in[2];
  TU* out[2];
  const int32_t* nbr1[2];  // first step's direction, per chain ([point][offset])
  const int32_t* nbr2[2];  // second step's direction
  int64_t m;
  int C;
  int chains;
  int sum_out;
  int split;  // two chains with outputs of their own: the grid's halves take one each
  int chain0; // k_blur2_split: the first half's chain
  int halves; // k_blur2_split: 2 (both chains) or 1 (chain0 alone)
  int vec;
  int nt;     // as in BlurArgs
  int64_t rows_per_block;
  TU st[3];
};

// VW values of a lattice row, or zeros where row < 0 (a missing neighbour).
// The load is issued unconditionally (from row `valid` when row < 0) and the
// zeros selected afterwards, so a thread's loads never wait on one another
// through a branch.
template <typename TU, int VW>
__device__ __forceinline__ void load_vw(const TU* __restrict__ in, int64_t row, int64_t valid, int C, int c,
                                        bool vec, TU (&v)[VW]) {
  const TU* src = in + (row >= 0 ? row : valid) * C + c;
  if (vec) {
    read_row<TU, VW>(src, v);
  } else {
#pragma unroll
    for (int i = 0; i < VW; ++i) {
      const TU x = src[c + i < C ? i : 0];
      v[i] = c + i < C ? x : (TU)0;
    }
  }
#pragma unroll
  for (int i = 0; i < VW; ++i) v[i] = row >= 0 ? v[i] : (TU)0;
}

template <typename TU, int VW>
__device__ __forceinline__ void blur2_rows(const TU* __restrict__ in, const int32_t* __restrict__ nb1,
                                           const int32_t* __restrict__ nb2, int64_t j, int C, int c,
                                           const TU* st, bool vec, TU (&acc)[VW]) {
  // second-direction neighbours of j (t2 = -1, 0, +1), then their
  // first-direction neighbours, then the nine rows
  int64_t x[3];
  const int2 lh2 = *(const int2*)(nb2 + 2 * j);
  x[0] = lh2.x;
  x[1] = j;
  x[2] = lh2.y;
  // (all six index loads and all nine row loads issue without waiting on
  // one another: indices of a missing x are read at j and discarded)
  int64_t y[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int64_t xa = x[a] >= 0 ? x[a] : j;
    const int2 lh1 = *(const int2*)(nb1 + 2 * xa);
    y[a][0] = x[a] >= 0 ? (int64_t)lh1.x : -1;
    y[a][1] = x[a];
    y[a][2] = x[a] >= 0 ? (int64_t)lh1.y : -1;
  }
  TU v[3][3][VW];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) load_vw<TU, VW>(in, y[a][b], j, C, c, vec, v[a][b]);
#pragma unroll
  for (int i = 0; i < VW; ++i) acc[i] = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    TU bx[VW];
#pragma unroll
    for (int i = 0; i < VW; ++i) bx[i] = 0;
    if (x[a] >= 0) {
#pragma unroll
      for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int i = 0; i < VW; ++i) bx[i] = fma_t(st[b], v[a][b][i], bx[i]);
    }
#pragma unroll
    for (int i = 0; i < VW; ++i) acc[i] = fma_t(st[a], bx[i], acc[i]);
  }
}

template <typename TU, int G>
__global__ __launch_bounds__(kBlock) void k_blur2(Blur2Args<TU> a) {
  constexpr int VW = blur_vw<G>();
  constexpr int LPR = G / VW;
  constexpr int R = kBlock / LPR;
  const int sub = threadIdx.x % LPR;
  const int64_t j0 = xcd_block(blockIdx.x, gridDim.x) * a.rows_per_block;
  const int64_t j1 = j0 + a.rows_per_block < a.m ? j0 + a.rows_per_block : a.m;
  for (int64_t j = j0 + threadIdx.x / LPR; j < j1; j += R) {
    for (int c = sub * VW; c < a.C; c += G) {
      const bool vec = a.vec && c + VW <= a.C;
      TU f[VW];
      blur2_rows<TU, VW>(a.in[0], a.nbr1[0], a.nbr2[0], j, a.C, c, a.st, vec, f);
      if (a.chains == 2) {
        TU b[VW];
        blur2_rows<TU, VW>(a.in[1], a.nbr1[1], a.nbr2[1], j, a.C, c, a.st, vec, b);
        if (a.sum_out) {
#pragma unroll
          for (int i = 0; i < VW; ++i) f[i] = f[i] + b[i];
        } else {
          TU* o1 = a.out[1] + j * a.C + c;
          if (vec) {
            if (a.nt)
              write_row_nt<TU, VW>(o1, b);
            else
              write_row<TU, VW>(o1, b);
          } else {
#pragma unroll
            for (int i = 0; i < VW; ++i)
              if (c + i < a.C) o1[i] = b[i];
          }
        }
      }
      TU* o0 = a.out[0] + j * a.C + c;
      if (vec) {
        if (a.nt)
          write_row_nt<TU, VW>(o0, f);
        else
          write_row<TU, VW>(o0, f);
      } else {
#pragma unroll
        for (int i = 0; i < VW; ++i)
          if (c + i < a.C) o0[i] = f[i];
      }
    }
  }
}

// k_blur2 for two chains that write outputs of their own: the grid's first
// half takes chain 0 and its second half chain 1, the same rows each, so a
// thread waits on half as many dependent loads.
template <typename TU, int G>
__global__ __launch_bounds__(kBlock) void k_blur2_split(Blur2Args<TU> a) {
  constexpr int VW = blur_vw<G>();
  constexpr int LPR = G / VW;
  constexpr int R = kBlock / LPR;
  const int sub = threadIdx.x % LPR;
  const unsigned nb = gridDim.x / a.halves;
  const int half = blockIdx.x >= nb ? 1 : 0;
  const int chain = a.chain0 + half;
  const unsigned bid = blockIdx.x - half * nb;
  const int64_t j0 = xcd_block(bid, nb) * a.rows_per_block;
  const int64_t j1 = j0 + a.rows_per_block < a.m ? j0 + a.rows_per_block : a.m;
  for (int64_t j = j0 + threadIdx.x / LPR; j < j1; j += R) {
    for (int c = sub * VW; c < a.C; c += G) {
      const bool vec = a.vec && c + VW <= a.C;
      TU f[VW];
      blur2_rows<TU, VW>(a.in[chain], a.nbr1[chain], a.nbr2[chain], j, a.C, c, a.st, vec, f);
      TU* o = a.out[chain] + j * a.C + c;
      if (vec) {
        if (a.nt)
          write_row_nt<TU, VW>(o, f);
        else
          write_row<TU, VW>(o, f);
      } else {
#pragma unroll
        for (int i = 0; i < VW; ++i)
          if (c + i < a.C) o[i] = f[i];
      }
    }
  }
}

// A group of blur directions in one pass over its tiles (groups.h): a block
// reads a tile's rows into registers and LDS, forms each direction's step as
// k_blur would (a missing neighbour adds 0) with the neighbours from LDS, and
// writes the rows back. In place but for a chain's first group, which reads
// U0, and the reverse chain's last one, which adds the forward chain. Against
// the fused pair of steps, which reads nine rows and five index pairs per row
// of two steps, a row is read and written once per three or four. Bound by
// the memory rate on rows in no order: m = 4.2M, 16 fp32 channels 162 us a
// group (3.3 TB/s on rows of 64 bytes), m = 874,000, 16 fp64 columns 49 us
// (4.6 TB/s on rows of 128); from the caches by issue and LDS reads:
// m = 141,000, 16 fp64 columns, both chains 17 us. Blur of one MVM, groups
// against pairs (in-place steps of one direction): adjoint of m = 4.2M, d = 16
// 55 against 141 (95) ms, CG iteration on m = 874,000, d = 11 1.35 against
// 2.07 (1.71) ms. 512 threads where a row takes eight lanes: 49 against 59 us
// with 256 (133 registers). Order 2 (five taps, R = 2) with groups against a
// launch per direction: MVM of n = 200,003, d = 9, 5 columns 81 against 138 us,
// 8 CG iterations at n = 1M, d = 11, 11 columns 3.8 against 6.3 ms.
template <typename TU>
struct GroupArgs {
  const TU* in[2];          // per chain
  TU* out[2];
  const TU* add;            // added to the result (a forward chain's), or null
  int64_t tile0[2];         // the group's first tile and tiles
  int32_t tiles[2];
  int dirs[2], rev[2];      // directions, from the last one down if rev
  int C, chunk0, chunks;    // channel chunks of this launch
  unsigned blocks;          // of one chain
  int vec;
  TU st[5];
};
template <int G, typename TU>
constexpr int group_vw() { return G < 16 / (int)sizeof(TU) ? G : 16 / (int)sizeof(TU); }
// Threads of a block: at most 4 rows each, so that registers allow as many
// waves as LDS does.
template <int G, typename TU>
constexpr int group_threads() { return G / group_vw<G, TU>() > 4 ? kGroupRows * 2 : kGroupRows; }

// A row's neighbour bytes in the order of a downward pass over nd directions:
// 16-bit (R = 1) or 32-bit fields 0 .. nd-1 reversed.
template <int R>
__device__ __forceinline__ void group_reverse(uint32_t (&s)[2 * R], int nd) {
  if constexpr (R == 1) {
    uint32_t x = s[1] >> 16 | s[1] << 16, y = s[0] >> 16 | s[0] << 16;  // fields 3 2 1 0
    for (int i = nd; i < kGroupDirs; ++i) {
      x = x >> 16 | y << 16;
      y >>= 16;
    }
    s[0] = x;
    s[1] = y;
  } else {
    const uint32_t t[4] = {s[0], s[1], s[2], s[3]};
    s[0] = nd == 4 ? t[3] : nd == 3 ? t[2] : nd == 2 ? t[1] : t[0];
    s[1] = nd == 4 ? t[2] : nd == 3 ? t[1] : t[0];
    s[2] = nd == 4 ? t[1] : t[0];
    s[3] = t[0];
  }
}

template <typename TU, int G, int R>
__global__ __launch_bounds__((group_threads<G, TU>())) void k_blur_group(
    const GroupRow<R>* __restrict__ rows, GroupArgs<TU> a) {
  constexpr int VW = group_vw<G, TU>();
  constexpr int LPR = G / VW;
  constexpr int RP = group_threads<G, TU>() / LPR;  // rows at a time
  constexpr int NI = kGroupRows / RP;
  __shared__ __align__(16) TU A[kGroupRows * G];
  const int ch = blockIdx.x >= a.blocks ? 1 : 0;
  const int b = (int)xcd_block(blockIdx.x - ch * a.blocks, a.blocks);
  const int tile = b / a.chunks;
  if (tile >= a.tiles[ch]) return;  // the other chain's group has more
  const int r0 = (int)threadIdx.x / LPR, cl = (int)(threadIdx.x % LPR) * VW;
  const int c = (a.chunk0 + b - tile * a.chunks) * G + cl;
  const bool vec = a.vec && c + VW <= a.C;
  const int64_t p0 = (a.tile0[ch] + tile) * kGroupRows + r0;
  const int nd = a.dirs[ch];
  int32_t row[NI];
  uint32_t nb[NI][2 * R];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const GroupRow<R> q = rows[p0 + i * RP];
    row[i] = q.point;
#pragma unroll
    for (int w = 0; w < 2 * R; ++w) nb[i][w] = q.slots[w];
  }
  TU v[NI][VW];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const TU* src = a.in[ch] + (int64_t)row[i] * a.C + c;
    if (row[i] >= 0 && vec) {
      read_row<TU, VW>(src, v[i]);
    } else {
#pragma unroll
      for (int x = 0; x < VW; ++x) v[i][x] = row[i] >= 0 && c + x < a.C ? src[x] : (TU)0;
    }
  }
  if (a.rev[ch]) {
#pragma unroll
    for (int i = 0; i < NI; ++i) group_reverse<R>(nb[i], nd);
  }
  const TU* Ac = A + cl;
#pragma unroll
  for (int t = 0; t < kGroupDirs; ++t) {
    if (t >= nd) break;
    if (t) __syncthreads();  // the last direction's rows have been read
#pragma unroll
    for (int i = 0; i < NI; ++i) write_row<TU, VW>(A + (r0 + i * RP) * G + cl, v[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      TU x[2 * R][VW];
#pragma unroll
      for (int e = 0; e < 2 * R; ++e) {
        const int at = 2 * R * t + e;
        read_row<TU, VW>(Ac + (nb[i][at / 4] >> (8 * (at % 4)) & 255) * G, x[e]);
      }
#pragma unroll
      for (int q = 0; q < VW; ++q) {
        TU o = 0;
#pragma unroll
        for (int e = 0; e < 2 * R + 1; ++e) o = fma_t(a.st[e], e < R ? x[e][q] : e == R ? v[i][q] : x[e - 1][q], o);
        v[i][q] = o;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    if (row[i] < 0) continue;
    const int64_t at = (int64_t)row[i] * a.C + c;
    TU* dst = a.out[ch] + at;
    if (vec) {
      if (a.add) {
        TU f[VW];
        read_row<TU, VW>(a.add + at, f);
#pragma unroll
        for (int x = 0; x < VW; ++x) v[i][x] = f[x] + v[i][x];
      }
      write_row<TU, VW>(dst, v[i]);
    } else {
#pragma unroll
      for (int x = 0; x < VW; ++x)
        if (c + x < a.C) dst[x] = a.add ? a.add[at + x] + v[i][x] : v[i][x];
    }
  }
}

// LDS layout of k_slice_tile: lattice rows [RC][G] (TU; also the CG
// reduction area) | weights [P*D] (fp32) | slots [P*D] (uint16).
struct SliceLds {
  size_t w, sl, total;
  int zrow;  // an all-zero lattice row past the staged rows and the reduction area
};
template <typename TU, int G, int NT = 1024>
__host__ __device__ inline SliceLds slice_lds(int P, int D) {
  using S = TileShape<TU, G, NT>;
  SliceLds o;
  const size_t row = sizeof(TU) * (size_t)S::RS;
  size_t b = row * (size_t)S::RC;
  const size_t red = sizeof(double) * (256 * 16 + 16 * 16);  // CG tile reduction
  if (b < red) b = red;
  o.zrow = (int)((b + row - 1) / row);
  b = row * (size_t)(o.zrow + 1);
  o.w = b;
  b += sizeof(float) * (size_t)P * D;
  o.sl = b;
  b += sizeof(uint16_t) * (size_t)(P * D + 1);
  o.total = (b + 15) & ~(size_t)15;
  return o;
}

// Scalars of k_slice_tile (its arrays are separate non-aliasing kernel
// arguments, as in k_splat_tile).
template <typename TU>
struct SliceArgs {
  int64_t n;
  int64_t items;
  int P, D, C, chunks;
  int cvec;
  TU scale;
  TU noise;
  int64_t mrows;        // CG: rows whose caller index is >= mrows are not solved for
  SliceLds lds;
};

// out = scale * W U restricted to one tile (Section 3.2, Slice). The tile's
// (slot, weight) entries and its first RC lattice rows arrive in registers
// while the previous tile is computed; a tile with more runs stages the rest
// RC rows at a time. Each point is combined by LPR lanes of VW channels from
// the staged rows. The CG variant forms q = out + noise * p, moves the
// residual (out is r: r -= alpha q, alpha already known) and emits the
// tile's new r . r per column, reduced in a fixed order.
template <typename TU, int G, bool CG, int NT>
// perm: caller row of each sorted point, or null. CG only: p is the
// direction and out the residual (sorted order), hook.partials receive each
// tile's r . r per column, mperm maps sorted points to caller rows for the
// mrows mask.
__global__ __launch_bounds__(NT) void k_slice_tile(
    const int32_t* __restrict__ tile_off, const int32_t* __restrict__ tile_verts,
    const uint16_t* __restrict__ loc, const float* __restrict__ ws, const TU* __restrict__ U,
    TU* __restrict__ out, const uint32_t* __restrict__ perm, const TU* __restrict__ p,
    CgHook hook, const uint32_t* __restrict__ mperm, SliceArgs<TU> a) {
  using S = TileShape<TU, G, NT>;
  static_assert(S::RC % kSliceOrderRows == 0, "staged chunks hold whole order blocks");
  extern __shared__ __align__(16) unsigned char smem[];
  TU* lu = (TU*)smem;
  float* lw = (float*)(smem + a.lds.w);
  uint16_t* lsl = (uint16_t*)(smem + a.lds.sl);
  const int tid = threadIdx.x;
  constexpr int RC = S::RC;

  float w[S::EPT];
  uint32_t sl2[S::EPT / 2];  // two 16-bit slots per register
  TU ur[S::UPT];
  int nq = 0, np = 0, q0 = 0;
  // rows [r0, r0 + nr) (nr >= 1) of a tile's run list, whose lattice points
  // are verts[r0 ..]. Indices past the end are clamped to valid ones, so all
  // index loads issue before the row loads that depend on them.
  int32_t vj[S::UPT];
  auto load_index = [&](int r0, int nr, const int32_t* verts) {
#pragma unroll
    for (int u = 0; u < S::UPT; ++u) {
      const int r = (tid + u * S::NT) / G;
      vj[u] = verts[r0 + (r < nr ? r : nr - 1)];
    }
  };
  auto load_rows = [&](int ch) {
#pragma unroll
    for (int u = 0; u < S::UPT; ++u) {
      const int c = ch * G + (tid + u * S::NT) % G;
      ur[u] = U[(int64_t)vj[u] * a.C + (c < a.C ? c : a.C - 1)];
    }
  };
  // A tile's first-chunk row indices are requested early (fetch_index) and
  // its entries and rows later (fetch), so the rows never wait for them.
  auto fetch_index = [&](int64_t item) {
    const int64_t t = item / a.chunks;
    const int64_t p0 = t * a.P;
    np = (int)(a.n - p0 < a.P ? a.n - p0 : a.P);
    q0 = tile_off[t];
    nq = tile_off[t + 1] - q0;
    load_index(0, nq < RC ? nq : RC, tile_verts + q0);
  };
  auto fetch = [&](int64_t item) {
    const int64_t t = item / a.chunks;
    const int ch = (int)(item - t * a.chunks);
    const int64_t p0 = t * a.P;
    const int ne = np * a.D;
    const float* gw = ws + p0 * a.D;
    const uint16_t* gsl = loc + p0 * a.D;
#pragma unroll
    for (int u = 0; u < S::EPT; ++u) {
      const int e = tid + u * S::NT;
      w[u] = gw[e < ne ? e : ne - 1];
    }
    // slots in pairs (the tile starts 4-byte aligned; the array has a
    // spare slot past its end)
    const uint32_t* gsl2 = (const uint32_t*)gsl;
    const int npair = (ne + 1) / 2;
#pragma unroll
    for (int u = 0; u < S::EPT / 2; ++u) {
      const int pi = tid + u * S::NT;
      sl2[u] = gsl2[pi < npair ? pi : npair - 1];
    }
    load_rows(ch);
  };
  auto stage_rows = [&](int nr) {
#pragma unroll
    for (int u = 0; u < S::UPT; ++u) {
      const int f = tid + u * S::NT;
      if (f < nr * G) lu[(f / G) * S::RS + f % G] = ur[u];
    }
  };

  // CG: alpha of every column (known before this kernel)
  __shared__ TU s_alpha[CG ? kMaxCgCols : 1];
  if constexpr (CG) {
    for (int c = tid; c < a.C && c < kMaxCgCols; c += S::NT) s_alpha[c] = (TU)hook.st->alpha[c];
  }
  int64_t item, end, step;
  xcd_items(a.items, &item, &end, &step);
  for (int i = tid; i < S::RS; i += S::NT) lu[a.lds.zrow * S::RS + i] = (TU)0;  // the zero row
  if (item < end) {
    fetch_index(item);
    fetch(item);
  }
  for (; item < end; item += step) {
    const int64_t t = item / a.chunks;
    const int ch = (int)(item - t * a.chunks);
    const int cur_nq = nq, cur_np = np, cur_ne = np * a.D, cur_q0 = q0;
    __syncthreads();  // the previous tile is done with the LDS
#pragma unroll
    for (int u = 0; u < S::EPT; ++u) {
      const int e = tid + u * S::NT;
      if (e < cur_ne) lw[e] = w[u];
    }
#pragma unroll
    for (int u = 0; u < S::EPT / 2; ++u) {
      const int pi = tid + u * S::NT;
      if (2 * pi < cur_ne) ((uint32_t*)lsl)[pi] = sl2[u];
    }
    stage_rows(cur_nq < RC ? cur_nq : RC);

    const int grp = tid / S::LPR;
    const int cl = (tid % S::LPR) * S::VW;  // channel offset within the chunk
    const int cg = ch * G + cl;
    const bool live = cg < a.C;
    const bool full = cg + S::VW <= a.C;
    // CG: this thread's p and r values, requested before the next tile's
    // loads so that using them never waits for those
    TU pv[S::PPG][S::VW], rv[S::PPG][S::VW];
#pragma unroll
    for (int k = 0; k < S::PPG; ++k) {
      const int lp = grp + k * S::NG;
#pragma unroll
      for (int i = 0; i < S::VW; ++i) {
        pv[k][i] = 0;
        rv[k][i] = 0;
      }
      if (CG && lp < cur_np && live) {
        const int64_t pt = t * a.P + lp;
        const TU* src = p + pt * a.C + cg;
        const TU* rsrc = out + pt * a.C + cg;
        if (full && a.cvec) {
          read_row<TU, S::VW>(src, pv[k]);
          read_row<TU, S::VW>(rsrc, rv[k]);
        } else {
#pragma unroll
          for (int i = 0; i < S::VW; ++i)
            if (cg + i < a.C) {
              pv[k][i] = src[i];
              rv[k][i] = rsrc[i];
            }
        }
      }
    }

    const bool next = item + step < end;
    if (next) fetch_index(item + step);
    TU acc[S::PPG][S::VW];
#pragma unroll
    for (int k = 0; k < S::PPG; ++k)
#pragma unroll
      for (int i = 0; i < S::VW; ++i) acc[k][i] = 0;
    for (int r0 = 0; r0 < cur_nq; r0 += RC) {
      const int nr = cur_nq - r0 < RC ? cur_nq - r0 : RC;
      if (r0 > 0) {
        __syncthreads();  // previous chunk consumed
        load_index(r0, nr, tile_verts + cur_q0);
        load_rows(ch);
        stage_rows(nr);
        if (next) fetch_index(item + step);  // the indices were overwritten
      }
      __syncthreads();
      // the next tile's entries and first rows load during the last chunk
      if (r0 + RC >= cur_nq && next) fetch(item + step);
      if (live) {
#pragma unroll
        for (int k = 0; k < S::PPG; ++k) {
          const int lp = grp + k * S::NG;
          if (lp < cur_np) {
            const int eb = lp * a.D;
            // EB entries at a time: slots and weights, then their rows
            constexpr int EB = S::VW * sizeof(TU) >= 32 ? (CG ? 1 : 2) : 4;
            // A point's entries are added by block of kSliceOrderRows runs
            // of the tile's run list, then in vertex order, whatever RC is
            // (a multiple of that block): the sums do not depend on the
            // channel chunk or block shape.
            // An entry outside the block (or past the point's d+1) reads
            // the zero row with weight 0: fma(0, 0, acc) is acc exactly, as
            // acc is never -0.
            for (int s0 = 0; s0 < nr; s0 += kSliceOrderRows)
            for (int j0 = 0; j0 < a.D; j0 += EB) {
              int sv[EB];
              TU wv[EB];
#pragma unroll
              for (int u = 0; u < EB; ++u) {
                const int j = j0 + u < a.D ? j0 + u : a.D - 1;
                const int sr = (int)lsl[eb + j] - r0 - s0;
                const float wr = lw[eb + j];
                const bool in = (unsigned)sr < (unsigned)(nr - s0 < kSliceOrderRows ? nr - s0 : kSliceOrderRows) &&
                                j0 + u < a.D;
                sv[u] = in ? s0 + sr : a.lds.zrow;
                wv[u] = (TU)(in ? wr : 0.f);
              }
              TU x[EB][S::VW];
#pragma unroll
              for (int u = 0; u < EB; ++u) read_row<TU, S::VW>(lu + sv[u] * S::RS + cl, x[u]);
#pragma unroll
              for (int u = 0; u < EB; ++u)
#pragma unroll
                for (int i = 0; i < S::VW; ++i) acc[k][i] = fma_t(wv[u], x[u][i], acc[k][i]);
            }
          }
        }
      }
    }
    double prod[S::PPG][S::VW];  // CG: r . r of each (point, channel)
#pragma unroll
    for (int k = 0; k < S::PPG; ++k) {
      const int lp = grp + k * S::NG;
#pragma unroll
      for (int i = 0; i < S::VW; ++i) prod[k][i] = 0.0;
      if (lp < cur_np && live) {
        const int64_t pt = t * a.P + lp;
        TU o[S::VW];
        const bool masked = CG && a.mrows > 0 && (int64_t)mperm[pt] >= a.mrows;  // not solved for
#pragma unroll
        for (int i = 0; i < S::VW; ++i) {
          o[i] = a.scale * acc[k][i];
          if (CG) {
            const TU q = masked ? (TU)0 : fma_t(a.noise, pv[k][i], o[i]);
            o[i] = fma_t(-s_alpha[cg + i < a.C ? cg + i : 0], q, rv[k][i]);
            prod[k][i] = (double)o[i] * (double)o[i];
          }
        }
        TU* dstp = out + (perm ? (int64_t)perm[pt] : pt) * a.C + cg;
        if (full && a.cvec) {
          write_row<TU, S::VW>(dstp, o);
        } else {
#pragma unroll
          for (int i = 0; i < S::VW; ++i)
            if (cg + i < a.C) dstp[i] = o[i];
        }
      }
    }
    if (CG) {
      // the tile's r . r per column: points in 16 blocks of 16, each block
      // and then the blocks added in index order, so that the sum does not
      // depend on how channels are split over lanes; 16 channels per pass
      double* sh = (double*)smem;            // [256 points][16 channels]
      double* sh2 = sh + 256 * 16;           // [16 blocks][16 channels]
      for (int cs = 0; cs < G; cs += 16) {
        __syncthreads();  // every lane is done with the staged rows / last pass
#pragma unroll
        for (int k = 0; k < S::PPG; ++k) {
          const int lp = grp + k * S::NG;
#pragma unroll
          for (int i = 0; i < S::VW; ++i) {
            const int cc = cl + i - cs;
            if (lp < 256 && cc >= 0 && cc < 16) sh[lp * 16 + cc] = prod[k][i];
          }
        }
        __syncthreads();
        if (tid < 256) {
          // every row is read (rows past the tile hold stale values and add
          // nothing), so the reads need no branches
          const int c16 = tid % 16, blk = tid / 16;
          const double* src = sh + blk * 256 + c16;
          double x[16];
#pragma unroll
          for (int u = 0; u < 16; ++u) x[u] = src[u * 16];
          double v = 0.0;
#pragma unroll
          for (int u = 0; u < 16; ++u) v += blk * 16 + u < cur_np ? x[u] : 0.0;
          sh2[blk * 16 + c16] = v;
        }
        __syncthreads();
        if (tid < 16 && cs + tid < G && ch * G + cs + tid < a.C) {
          double v = 0.0;
          for (int blk = 0; blk < 16; ++blk) v += sh2[blk * 16 + tid];
          hook.partials[t * a.C + ch * G + cs + tid] = v;
        }
      }
    }
  }
  // CG: the tiles' r . r folded into beta, where this grid is small (kFoldBlocks)
  if constexpr (CG) cg_finish(hook, a.C, (double*)smem);
}


template <typename TU>
size_t slice_lds_g(int P, int D, int g) {
  switch (g) {
    case 1: return slice_lds<TU, 1>(P, D).total;
    case 2: return slice_lds<TU, 2>(P, D).total;
    case 4: return slice_lds<TU, 4>(P, D).total;
    case 8: return slice_lds<TU, 8>(P, D).total;
    default: return slice_lds<TU, 16>(P, D).total;
  }
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

int cu_count() {
  constexpr int kMaxDevices = 64;
  static int cus[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
  if (!cus[dev]) {
    int c = 0;
    if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c < 1) c = 256;
    cus[dev] = c;
  }
  return cus[dev];
}

// Blocks of a persistent tile kernel: as many as can be resident, at most
// one per work item. A kernel staging more than 64 KiB of LDS is first
// allowed to.
// Launch choices an autotuning run can set: the channel chunk width and the
// resident blocks per CU of the persistent splat and slice (0: as many as
// the occupancy allows; splat_bpc is k_cg_tile's in CG on the lattice). None of
// them changes a result: every sum is formed in an order that depends on
// neither the chunk width nor the grid.
struct LaunchChoice {
  int g;
  int splat_bpc;
  int slice_bpc;
};
enum TuneForm { TF_MVM = 0, TF_LAT = 1 };  // MVMs, also inside CG; CG on the lattice
struct TuneEntry {
  TuneForm form;
  int d, elem, g0, mlog;
  LaunchChoice c;
  float ms;
};
std::mutex g_tune_mu;
std::vector<TuneEntry> g_tune;                  // process-wide, keyed by lattice shape
thread_local const LaunchChoice* g_force = nullptr;  // set while candidates are timed

int mlog_of(int64_t m) {
  int b = 0;
  while (((int64_t)1 << b) < m) ++b;
  return b;
}

bool tune_find(const sgp_lattice* L, int C, int elem, TuneForm form, LaunchChoice* out) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  for (const TuneEntry& e : g_tune)
    if (e.form == form && e.d == L->d && e.elem == elem && e.g0 == lanes_for(C) && e.mlog == mlog_of(L->m)) {
      *out = e.c;
      return true;
    }
  return false;
}

unsigned persistent_grid(const void* kernel, int threads, size_t lds, int64_t items, int chosen_bpc) {
  if (lds > 65536) (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  (void)hipGetLastError();
  int bpc = tuning().blocks_per_cu;
  if (bpc <= 0) bpc = chosen_bpc;
  if (bpc <= 0) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, threads, lds) != hipSuccess || nb < 1) {
      (void)hipGetLastError();
      nb = 1;
    }
    bpc = nb;
  }
  int64_t g = (int64_t)cu_count() * bpc;
  if (g > items) g = items;
  if (g < 1) g = 1;
  return (unsigned)g;
}

// Rows per gather range: 64, halved (down to 8) while the lattice would
// have fewer than 4096 ranges, so that a small lattice's gather still
// spreads over the GPU instead of summing long ranges in few groups.
int gather_rows(const sgp_lattice* L) {
  int r = 64;
  while (r > 8 && (L->npiece + r - 1) / r < 4096) r >>= 1;
  return r;
}
int64_t gather_ranges(const sgp_lattice* L) {
  const int r = gather_rows(L);
  return (L->npiece + r - 1) / r;
}

unsigned grid_cap(int64_t work) {
  int64_t b = (work + kBlock - 1) / kBlock;
  if (b < 1) b = 1;
  if (b > 16384) b = 16384;
  return (unsigned)b;
}

// Blocks for `rows` rows at R per block, capped, and the rows each block
// takes so that the blocks cover all rows.
void split_rows(int64_t rows, int R, int64_t cap, unsigned* blocks, int64_t* rows_per_block) {
  int64_t b = (rows + R - 1) / R;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  *rows_per_block = (rows + b - 1) / b;
  *blocks = (unsigned)((rows + *rows_per_block - 1) / *rows_per_block);
}

// Whether the blur of C columns (fp64 inside CG) runs by the groups of directions
// that the lattice keeps. Of order 1 they may be as many passes as the fused
// pairs (dense lattices of few dimensions, mostly groups of two). A pair reads
// nearby rows, coalesced, a group each row once, in no order, so groups then win
// with wide rows on lattices that outgrow the L2s, and where a pair's lanes read
// their four columns element by element. Pairs | groups, MVMs (fp32) and CG
// iterations (fp64), microseconds: m = 62,000 (d = 6) C = 1 48 | 55, 4 62 | 68,
// 8 66 | 73, 16 71 | 77, 32 119 | 107, fp64 2 76 | 80, 6 110 | 100, 8 85 | 90;
// m = 245,000 (d = 6) C = 1 96 | 101, 3 152 | 144, 8 162 | 174, 11 346 | 261,
// 16 200 | 188, fp64 1 131 | 139, 8 230 | 208; m = 673,000 (d = 8) C = 1
// 205 | 220, 4 319 | 353, 8 410 | 392, 16 564 | 466, fp64 1 258 | 303, 2 339 |
// 369, 4 455 | 396. Groups of two and one that are one pass more, m = 607,000
// (d = 5): C = 1 112 | 141, 3 202 | 237, 6 312 | 268, 8 188 | 214, 12 238 | 287,
// 16 257 | 257, 32 662 | 478, fp64 4 223 | 235, 6 437 | 311, 8 306 | 286.
bool blur_by_groups(const sgp_lattice* L, int C, bool cg, bool fuse) {
  if (!L->ngroups || !fuse) return false;
  const int pairs = (L->d + 2) / 2;
  if (L->order != 1 || L->ngroups < pairs) return true;
  const int64_t row = (int64_t)C * (cg ? sizeof(double) : sizeof(float));
  const bool whole = C == 1 || C % 4 == 0 || (cg && C == 2);  // lanes read an element, or 16-byte vectors
  const bool more = L->ngroups > pairs && L->group_most <= 2;
  if (!whole) return row >= 20 || !more;
  return row >= 128 || (row >= (more ? 64 : 32) && L->m * row >= (8 << 20));
}

// m x C lattice value arrays that the blur works in beside the one it reads: its
// ping-pong between two a chain (the second chain's other one may be the input,
// where that need not outlive the blur: not inside CG), or one a chain, in place,
// by groups of directions.
int blur_arrays(const sgp_lattice* L, int C, bool cg, bool fuse) {
  return blur_by_groups(L, C, cg, fuse) ? 2 : cg ? 4 : 3;
}

// Work memory of one MVM in elements of its accumulator type: m x C lattice
// value arrays (the splat's result and the blur's), one partial row per run
// piece, two fragment rows per gather range.
size_t mvm_work_elems(const sgp_lattice* L, int C, bool cg, bool fuse) {
  return (size_t)((1 + blur_arrays(L, C, cg, fuse)) * L->m + L->npiece + 2 * gather_ranges(L)) * (size_t)C;
}

// U0 = the partial rows summed per lattice point (+ beta U0 per column when
// beta is given: device array, fp64 only). fix: points whose rows span ranges
// are finished here (else k_lattice_col does that).
template <typename TU, int G>
int gather_g(const sgp_lattice* L, const TU* part, TU* U0, TU* frag, int C, const double* beta, bool fix,
             hipStream_t s) {
  ProfScope ps(KK_SPLAT_GATHER, s);
  const int R = gather_rows(L);
  const int64_t ngroups = gather_ranges(L);
  constexpr int VWG = 16 / (int)sizeof(TU);  // channels per lane with 16-byte loads
  // Lattice points requested ahead pay where the rows outgrow the caches and the
  // waves are too few to hide their latency, first with one lane a range; below,
  // the loads past a range's end and the registers cost more. In the batch | ahead,
  // microseconds: 0.38M rows, C = 1 fp32 37 | 35, 8 31 | 33, 16 24 | 28, fp64 8
  // 23 | 28; 0.95M rows 1 42 | 39, 8 37 | 39, 16 30 | 36, fp64 8 29 | 35; 1.7M rows
  // 1 44 | 40, 3 34 | 33, 8 46 | 46, 16 58 | 59, fp64 3 45 | 42; 3.1M rows 1 52 | 45,
  // 8 92 | 85, 16 90 | 84, fp64 2 72 | 64, 16 108 | 108; 4.0M rows 8 106 | 96.
  auto launch = [&](auto vw_tag, auto beta_tag) {
    constexpr int VW = decltype(vw_tag)::value;
    constexpr bool BETA = decltype(beta_tag)::value;
    const unsigned blocks = (unsigned)((ngroups + kBlock / (G / VW) - 1) / (kBlock / (G / VW)));
    const bool ahead = BETA || L->npiece >= (G == VW ? (int64_t)1 << 18 : (int64_t)3 << 19);
    if (ahead)
      hipLaunchKernelGGL((k_splat_gather<TU, G, VW, true, BETA>), dim3(blocks), dim3(kBlock), 0, s,
                         (const int32_t*)L->row_vert.ptr, part, U0, frag, L->npiece, C, ngroups, R, beta);
    else if constexpr (!BETA)
      hipLaunchKernelGGL((k_splat_gather<TU, G, VW, false, false>), dim3(blocks), dim3(kBlock), 0, s,
                         (const int32_t*)L->row_vert.ptr, part, U0, frag, L->npiece, C, ngroups, R, beta);
  };
  auto widths = [&](auto beta_tag) {
    if (G % VWG == 0 && C % VWG == 0 && aligned16(part) && aligned16(U0) && aligned16(frag))
      launch(std::integral_constant<int, (G % VWG == 0 ? VWG : 1)>{}, beta_tag);
    else
      launch(std::integral_constant<int, 1>{}, beta_tag);
  };
  if constexpr (sizeof(TU) == 8) {
    if (beta)
      widths(std::true_type{});
    else
      widths(std::false_type{});
  } else {
    widths(std::false_type{});
  }
  SGP_LAUNCH_CHECK("k_splat_gather");
  if (!fix) return SGP_OK;
  hipLaunchKernelGGL(k_gather_fix, dim3(grid_cap(ngroups * C)), dim3(kBlock), 0, s,
                     (const int32_t*)L->row_vert.ptr, (const int32_t*)L->occ_ptr.ptr, (const void*)frag,
                     (void*)U0, ngroups, C, (int)sizeof(TU), R, beta);
  SGP_LAUNCH_CHECK("k_gather_fix");
  return SGP_OK;
}

// Whether an MVM's lattice part runs as one block per column: a three-tap
// lattice of up to 2,048 points and (inside CG) few partial sums of p.Ap. Its
// launches (the fix-up, a launch per two directions, alpha and its fold) are
// then one, which they are too short to fill. Here | separate launches, one
// MVM and ten CG iterations, C = 1 and 8: m = 851 (d = 3) 33 us, 327 us;
// 34, 342 | 39, 419; 41, 461. m = 1,460 (d = 6) 39, 404; 42, 441 | 64, 512;
// 63, 570. Beyond, one CU per column takes longer than the launches that it
// saves: with four rows a thread, m = 4,453 (d = 6) 55, 571; 63, 651 |
// 66, 503; 68, 571. As good on many columns: m = 1,460, one MVM of 256 columns
// 87 | 175 us.
bool col_path(const sgp_lattice* L, int64_t parts, bool fuse) {
  return L->order == 1 && L->m <= kColRows && parts <= kColParts && fuse;
}

template <typename TU, int MODE>
int col_launch(const sgp_lattice* L, TU* U, const TU* frag, TU* Bu, int C, double scale, const CgMvm& cgm,
               hipStream_t s) {
  ColArgs a = {};
  a.m = (int)L->m;
  a.C = C;
  a.D = L->d + 1;
  while ((1 << a.rshift) < gather_rows(L)) ++a.rshift;
  a.first = L->blur != SGP_BLUR_REVERSE ? 1 : 0;
  a.rev = L->blur != SGP_BLUR_FORWARD ? 1 : 0;
  a.lat_parts = MODE == CM_CG ? (int)cgm.lat_parts : 0;
  a.ntiles = MODE == CM_CG ? (int)cgm.ntiles : 0;
  a.scale = scale;
  for (int t = 0; t < 3; ++t) a.st[t] = L->stencil64[t];
  const size_t lds = col_lds<TU, MODE>(a);
  auto launch = [&](auto nr_tag) -> int {
    for (a.c0 = 0; a.c0 < C; a.c0 += kColGrid) {
      ProfScope ps(KK_BLUR, s);
      hipLaunchKernelGGL((k_lattice_col<TU, decltype(nr_tag)::value, MODE>),
                         dim3((unsigned)std::min(C - a.c0, kColGrid)), dim3(kColThreads), lds, s, U, frag,
                         (const int32_t*)L->occ_ptr.ptr, (const int32_t*)L->nbr.ptr, Bu, cgm.pp, cgm.alpha, a);
      SGP_LAUNCH_CHECK("k_lattice_col");
    }
    return SGP_OK;
  };
  return a.m <= kColThreads ? launch(std::integral_constant<int, 1>{}) : launch(std::integral_constant<int, 2>{});
}

// The blur of U0 (m x C): B1 .. B4 are work arrays (B4 may be U0 where it need
// not outlive the blur; of blur_arrays 2 only B1 and B2 are there); *result is the array that holds the blurred values
// (forward + reverse in SYMMETRIC order).
template <typename TU, int G>
int blur_g(const sgp_lattice* L, TU* U0, TU* B1, TU* B2, TU* B3, TU* B4, int C, bool fused, hipStream_t s,
           const TU** result) {
  const int d = L->d, T = 2 * L->order;
  const int64_t m = L->m, mC = m * C;
  const bool sym = L->blur == SGP_BLUR_SYMMETRIC;
  BlurArgs<TU> a;
  a.m = m;
  a.C = C;
  a.r = L->order;
  a.chains = sym ? 2 : 1;
  for (int t = 0; t < 2 * L->order + 1; ++t) a.st[t] = (TU)L->stencil64[t];
  unsigned bblocks;
  split_rows(m, kBlock / (G / blur_vw<G>()), 65536, &bblocks, &a.rows_per_block);
  a.vec = (C % Vec16<TU>::N == 0 && blur_vw<G>() % Vec16<TU>::N == 0 && aligned16(U0)) ? 1 : 0;
  // when the four lattice value arrays outgrow the 256 MiB Infinity Cache, the
  // blur's outputs stream past it, which keeps more of its inputs cached
  a.nt = (4.0 * (double)mC * sizeof(TU) > 256.0 * (1 << 20)) ? 1 : 0;
  const int32_t* nbr = (const int32_t*)L->nbr.ptr;
  // Chain 0 moves between B1 and B3 and never writes U0, which chain 1 reads
  // first; chain 1 moves between B2 and B4 (U0 outside CG). Steps run in
  // fused pairs when the stencil has three taps.
  const TU* cur[2] = {U0, U0};
  auto next0 = [&](const TU* c0) { return c0 == B1 ? B3 : B1; };
  auto next1 = [&](const TU* c1) { return c1 == B2 ? B4 : B2; };
  auto kdir = [&](int step, int chain) {
    return chain == 0 ? ((L->blur == SGP_BLUR_REVERSE) ? d - step : step) : d - step;
  };
  const bool fuse = L->order == 1 && fused;
  const bool groups = blur_by_groups(L, C, sizeof(TU) == 8, fused);  // (fp64 is CG's)
  // Large lattices: the chains' launches run one chain after the other (all of
  // chain 0's, then chain 1's), so that a launch's arrays sit in the Infinity
  // Cache together.
  const bool seq = (fuse || groups) && sym && blur_seq_for(4.0 * (double)mC * sizeof(TU), groups);
  std::vector<Blur2Args<TU>> later;  // chain 1's split launches, in order
  auto launch2 = [&](const Blur2Args<TU>& b, unsigned grid) -> int {
    ProfScope ps(KK_BLUR, s);
    if (b.split)
      hipLaunchKernelGGL((k_blur2_split<TU, G>), dim3(grid), dim3(kBlock), 0, s, b);
    else
      hipLaunchKernelGGL((k_blur2<TU, G>), dim3(grid), dim3(kBlock), 0, s, b);
    SGP_LAUNCH_CHECK("k_blur2");
    return SGP_OK;
  };
  auto flush_later = [&]() -> int {
    for (const auto& b : later) {
      const int rc = launch2(b, bblocks);
      if (rc) return rc;
    }
    later.clear();
    return SGP_OK;
  };
  if (groups) {
    const int ng = L->ngroups;
    GroupArgs<TU> b;
    b.C = C;
    b.vec = (C % group_vw<G, TU>() == 0 && aligned16(U0) && aligned16(B1) && aligned16(B2)) ? 1 : 0;
    for (int t = 0; t < 2 * L->order + 1; ++t) b.st[t] = a.st[t];
    // one group of chain 0 (i0 >= 0) and one of chain 1 (i1 >= 0)
    auto launch = [&](int i0, int i1, bool sum) -> int {
      unsigned n = 0;
      int64_t most = 0;
      for (int ch = 0; ch < 2; ++ch) {
        const int i = ch ? i1 : i0;
        if (i < 0) continue;
        const bool rev = ch || L->blur == SGP_BLUR_REVERSE;
        const int g = rev ? ng - 1 - i : i;
        b.in[n] = i ? (ch ? B2 : B1) : U0;
        b.out[n] = ch && !sum ? B2 : B1;
        b.tile0[n] = L->group_tile[g];
        b.tiles[n] = L->group_tiles[g];
        b.dirs[n] = L->group_dirs[g];
        b.rev[n] = rev;
        most = std::max(most, (int64_t)b.tiles[n]);
        ++n;
      }
      b.add = sum ? B1 : nullptr;
      // a launch takes all channel chunks, unless they are so many that its
      // grid would come near 2^32 threads
      const int chunks = (C + G - 1) / G;
      const int most_chunks = (int)std::max<int64_t>(1, ((int64_t)1 << 31) / (most * n * group_threads<G, TU>()));
      for (b.chunk0 = 0; b.chunk0 < chunks; b.chunk0 += b.chunks) {
        b.chunks = std::min(chunks - b.chunk0, most_chunks);
        b.blocks = (unsigned)(most * b.chunks);
        ProfScope ps(KK_BLUR, s);
        const dim3 grid(b.blocks * n), block(group_threads<G, TU>());
        if (L->order == 1)
          hipLaunchKernelGGL((k_blur_group<TU, G, 1>), grid, block, 0, s, (const GroupRow<1>*)L->group_rows.ptr, b);
        else
          hipLaunchKernelGGL((k_blur_group<TU, G, 2>), grid, block, 0, s, (const GroupRow<2>*)L->group_rows.ptr, b);
        SGP_LAUNCH_CHECK("k_blur_group");
      }
      return SGP_OK;
    };
    int rc = SGP_OK;
    *result = B1;
    if (!sym || seq) {
      for (int i = 0; !rc && i < ng; ++i) rc = launch(i, -1, false);
      for (int i = 0; !rc && sym && i < ng; ++i) rc = launch(-1, i, i == ng - 1);
    } else {
      for (int i = 0; !rc && i < ng - 1; ++i) rc = launch(i, i, false);
      if (!rc) rc = launch(ng - 1, -1, false);
      if (!rc) rc = launch(-1, ng - 1, true);
    }
    return rc;
  }
  for (int step = 0; step <= d;) {
    TU* dst0 = next0(cur[0]);
    TU* dst1 = next1(cur[1]);
    if (fuse && step + 1 <= d) {
      Blur2Args<TU> b2;
      b2.in[0] = cur[0];
      b2.in[1] = cur[1];
      b2.out[0] = dst0;
      b2.out[1] = dst1;
      for (int ch = 0; ch < 2; ++ch) {
        b2.nbr1[ch] = nbr + (int64_t)kdir(step, ch) * T * m;
        b2.nbr2[ch] = nbr + (int64_t)kdir(step + 1, ch) * T * m;
      }
      b2.m = m;
      b2.C = C;
      b2.chains = a.chains;
      b2.sum_out = (sym && step + 1 == d) ? 1 : 0;
      b2.split = (a.chains == 2 && !b2.sum_out) ? 1 : 0;
      b2.chain0 = 0;
      b2.halves = 2;
      b2.vec = a.vec;
      b2.nt = a.nt;
      b2.rows_per_block = a.rows_per_block;
      for (int t = 0; t < 3; ++t) b2.st[t] = a.st[t];
      int rc;
      if (b2.split && seq) {
        b2.halves = 1;
        if ((rc = launch2(b2, bblocks))) return rc;
        b2.chain0 = 1;
        later.push_back(b2);
      } else {
        if ((rc = flush_later())) return rc;
        if ((rc = launch2(b2, b2.split ? 2 * bblocks : bblocks))) return rc;
      }
      step += 2;
    } else {
      a.in[0] = cur[0];
      a.out[0] = dst0;
      a.nbr[0] = nbr + (int64_t)kdir(step, 0) * T * m;
      a.in[1] = cur[1];
      a.out[1] = dst1;
      a.nbr[1] = nbr + (int64_t)kdir(step, 1) * T * m;
      a.sum_out = (sym && step == d) ? 1 : 0;
      if (const int rc = flush_later()) return rc;
      {
        ProfScope ps(KK_BLUR, s);
        hipLaunchKernelGGL((k_blur<TU, G>), dim3(bblocks), dim3(kBlock), 0, s, a);
        SGP_LAUNCH_CHECK("k_blur");
      }
      step += 1;
    }
    cur[0] = dst0;
    cur[1] = dst1;
  }
  if (const int rc = flush_later()) return rc;
  *result = cur[0];
  return SGP_OK;
}

// LDS of k_splat_tile: values [P+1][G], then the entry lists.
template <typename TU>
SplatLists splat_lds(const sgp_lattice* L, int G) {
  const int rs = G * (int)sizeof(TU) >= 64 ? G + 16 / (int)sizeof(TU) : G;
  return splat_lists((int)sizeof(TU) * (L->tile_points + 1) * rs, L->max_tile_ents, L->max_tile_pieces);
}

// cgm (CG only, else null): V is the direction p, out the residual r (both
// internal order), and the MVM finishes the CG step (CgMvm).
template <typename TU, int G>
int mvm_g(const sgp_lattice* L, const TU* V, const uint32_t* perm, int C, TU* out, hipStream_t s,
          TU noise, const CgMvm* cgm, const LaunchChoice& lc, void* work, const CgDirUpdate* up, bool fuse) {
  const int D = L->d + 1;
  const int64_t m = L->m, mC = m * C;
  const TU* p = cgm ? V : nullptr;
  TU* U0 = (TU*)work;
  TU* B1 = U0 + mC;
  TU* B2 = B1 + mC;
  const int arrays = blur_arrays(L, C, cgm != nullptr, fuse);
  TU* B3 = arrays > 2 ? B2 + mC : nullptr;
  TU* B4 = arrays > 3 ? B3 + mC : U0;  // chain 1's second array (U0 itself outside CG)
  TU* part = U0 + (1 + arrays) * mC;
  TU* frag = part + L->npiece * C;  // 2 rows per gather range
  const int chunks = (C + G - 1) / G;
  const int P = L->tile_points;
  SplatArgs<TU> sa;
  sa.n = L->n;
  sa.items = L->ntiles * chunks;
  sa.P = P;
  sa.D = D;
  sa.C = C;
  sa.chunks = chunks;
  sa.vec_v = (TileShape<TU, G, kSplatBlock>::VEC && !perm && C == G && aligned16(V)) ? 1 : 0;
  sa.vec_perm = (TileShape<TU, G, kSplatBlock>::VEC && perm && C == G && aligned16(V)) ? 1 : 0;
  sa.cvec = (C % Vec16<TU>::N == 0 && aligned16(part)) ? 1 : 0;
  sa.estride = tile_ent_stride(P * D);
  sa.lds = splat_lds<TU>(L, G);
  sa.pp_scale = cgm ? (double)noise : 0.0;
  double* pp = cgm ? cgm->pp : nullptr;
  // the previous CG iteration's direction update: in this splat where its
  // values are whole vectors of all C columns, else as a pass of its own
  const bool dir_fused = up && sizeof(TU) == 8 && !perm && C == G &&
                         (!TileShape<TU, G, kSplatBlock>::VEC || sa.vec_v);
  if (up && !dir_fused) {
    const int rc = launch_cg_dir(*up, (int64_t)L->n * C, C, s);
    if (rc) return rc;
  }
  {
    ProfScope ps(KK_SPLAT, s);
    const void* kern =
        dir_fused ? (const void*)&k_splat_tile<TU, G, true> : (const void*)&k_splat_tile<TU, G, false>;
    const unsigned grid = persistent_grid(kern, kSplatBlock, (size_t)sa.lds.end, sa.items, lc.splat_bpc);
    if (dir_fused)
      hipLaunchKernelGGL((k_splat_tile<TU, G, true>), dim3(grid), dim3(kSplatBlock), (size_t)sa.lds.end, s,
                         (const int32_t*)L->stile_off.ptr, (const int32_t*)L->tile_ent.ptr, (const uint32_t*)L->slice.ptr,
                         (const int32_t*)L->run_dst.ptr, (const uint8_t*)L->ent_lp.ptr,
                         (const float*)L->ent_w.ptr, V, perm, part, pp, sa, *up);
    else
      hipLaunchKernelGGL((k_splat_tile<TU, G, false>), dim3(grid), dim3(kSplatBlock), (size_t)sa.lds.end, s,
                         (const int32_t*)L->stile_off.ptr, (const int32_t*)L->tile_ent.ptr, (const uint32_t*)L->slice.ptr,
                         (const int32_t*)L->run_dst.ptr, (const uint8_t*)L->ent_lp.ptr,
                         (const float*)L->ent_w.ptr, V, perm, part, pp, sa, CgDirUpdate{});
    SGP_LAUNCH_CHECK("k_splat_tile");
  }
  const bool col = col_path(L, cgm ? cgm->alpha.nparts : 0, fuse);
  if (const int rc = gather_g<TU, G>(L, part, U0, frag, C, nullptr, !col, s)) return rc;
  const TU* blurred = B1;
  const bool sym = L->blur == SGP_BLUR_SYMMETRIC;
  const TU scale = sym ? (TU)(0.5 * (double)L->outputscale) : (TU)L->outputscale;
  if (col) {
    int rc;
    if constexpr (sizeof(TU) == 8)
      rc = cgm ? col_launch<TU, CM_CG>(L, U0, frag, B1, C, (double)scale, *cgm, s)
               : col_launch<TU, CM_MVM>(L, U0, frag, B1, C, 0.0, CgMvm{}, s);
    else
      rc = col_launch<TU, CM_MVM>(L, U0, frag, B1, C, 0.0, CgMvm{}, s);
    if (rc) return rc;
  } else if (const int rc = blur_g<TU, G>(L, U0, B1, B2, B3, B4, C, fuse, s, &blurred)) {
    return rc;
  }
  if (cgm && !col) {
    // alpha from p.Ap = scale * u.(B u) + noise * p.p, before the slice
    const int rc = launch_cg_alpha((const double*)U0, (const double*)blurred, m, C, (double)scale, *cgm, s);
    if (rc) return rc;
  }
  CgHook bh = {};
  if (cgm) bh = cgm->beta;
  SliceArgs<TU> la;
  la.n = L->n;
  la.items = L->ntiles * chunks;
  la.P = P;
  la.D = D;
  la.C = C;
  la.chunks = chunks;
  la.cvec = (C % Vec16<TU>::N == 0 && aligned16(out) && (!p || aligned16(p))) ? 1 : 0;
  la.scale = scale;
  la.noise = noise;
  la.mrows = cgm ? L->solve_rows : 0;
  const int32_t* toff = (const int32_t*)L->tile_off.ptr;
  const int32_t* tverts = (const int32_t*)L->tile_verts.ptr;
  const uint16_t* loc = (const uint16_t*)L->loc.ptr;
  const float* ws = (const float*)L->ws.ptr;
  const uint32_t* mperm = (const uint32_t*)L->perm.ptr;
  auto launch = [&](auto nt_tag) {
    ProfScope ps(KK_SLICE, s);
    constexpr int NT = decltype(nt_tag)::value;
    la.lds = slice_lds<TU, G, NT>(P, D);
    if (cgm) {
      const unsigned grid = persistent_grid((const void*)&k_slice_tile<TU, G, true, NT>, NT, la.lds.total,
                                            la.items, lc.slice_bpc);
      bh.fold = grid <= kFoldBlocks ? 1 : 0;
      hipLaunchKernelGGL((k_slice_tile<TU, G, true, NT>), dim3(grid), dim3(NT), la.lds.total, s, toff, tverts,
                         loc, ws, blurred, out, perm, p, bh, mperm, la);
    } else {
      const unsigned grid = persistent_grid((const void*)&k_slice_tile<TU, G, false, NT>, NT, la.lds.total,
                                            la.items, lc.slice_bpc);
      hipLaunchKernelGGL((k_slice_tile<TU, G, false, NT>), dim3(grid), dim3(NT), la.lds.total, s, toff, tverts,
                         loc, ws, blurred, out, perm, (const TU*)nullptr, CgHook{}, mperm, la);
    }
  };
  constexpr int NTn = slice_threads_narrow<G>();
  // the narrow block where the mean run list takes at most 2/3 of its pass
  if (NTn < 1024 && 3 * L->nrun <= 2 * L->ntiles * (int64_t)TileShape<TU, G, NTn>::RC)
    launch(std::integral_constant<int, NTn>{});
  else
    launch(std::integral_constant<int, 1024>{});
  SGP_LAUNCH_CHECK("k_slice_tile");
  return !cgm || bh.fold ? SGP_OK : launch_cg_scalar(bh, C, s);
}

// Channel chunk: the widest power of two <= kMaxChunk covering C for which
// both tile kernels' LDS stages fit the budget. Chunks of at most 16
// channels stage whole blocks of kSliceOrderRows runs in the slice, so a
// column's results are the same bit for bit whatever the chunk; more
// columns take several chunks.
constexpr int kMaxChunk = 16;
// LDS of a CU, less the static words of the tile kernels
constexpr size_t kCgTileLds = 163840 - 2048;
int chunk_lanes(const sgp_lattice* L, int C, size_t elem) {
  int g = lanes_for(C);
  if (g > kMaxChunk) g = kMaxChunk;
  const int D = L->d + 1, P = L->tile_points;
  const size_t budget = (size_t)tuning().lds_budget;
  const size_t slice_budget = (size_t)tuning().slice_lds_budget;
  while (g > 1) {
    const size_t splat = elem == 8 ? splat_lds<double>(L, g).end : splat_lds<float>(L, g).end;
    const size_t slice = elem == 8 ? slice_lds_g<double>(P, D, g) : slice_lds_g<float>(P, D, g);
    if (splat <= budget && slice <= slice_budget) break;
    g >>= 1;
  }
  return g;
}

// work: the MVM's work memory (mvm_work_elems elements of TU), or null for the
// lattice's own buffer, grown on demand.
template <typename TU>
int mvm_dispatch(const sgp_lattice* L, const TU* V, const uint32_t* perm, int C, TU* out,
                 hipStream_t s, TU noise, const CgMvm* cgm, void* work = nullptr,
                 const CgDirUpdate* up = nullptr) {
  const bool fuse = cgm ? cgm->fuse : blur_fuse_enabled();
  if (!work) {
    int rc = dev_reserve(L, const_cast<sgp_lattice*>(L)->ubuf,
                         sizeof(TU) * mvm_work_elems(L, C, cgm != nullptr, fuse), s);
    if (rc) return rc;
    work = L->ubuf.ptr;
  }
  const int gmax = chunk_lanes(L, C, sizeof(TU));
  LaunchChoice lc{gmax, 0, 0};
  if (g_force)
    lc = *g_force;
  else
    (void)tune_find(L, C, (int)sizeof(TU), TF_MVM, &lc);
  if (lc.g < 1 || lc.g > gmax || (lc.g & (lc.g - 1))) lc.g = gmax;  // never wider than the LDS allows
  switch (lc.g) {
    case 1: return mvm_g<TU, 1>(L, V, perm, C, out, s, noise, cgm, lc, work, up, fuse);
    case 2: return mvm_g<TU, 2>(L, V, perm, C, out, s, noise, cgm, lc, work, up, fuse);
    case 4: return mvm_g<TU, 4>(L, V, perm, C, out, s, noise, cgm, lc, work, up, fuse);
    case 8: return mvm_g<TU, 8>(L, V, perm, C, out, s, noise, cgm, lc, work, up, fuse);
    default: return mvm_g<TU, 16>(L, V, perm, C, out, s, noise, cgm, lc, work, up, fuse);
  }
}


// ---------------------------------------------------------------------------
// CG with its vectors on the lattice (cg_tile.h).

struct LatWork {
  double *yr, *yp, *yx, *u, *b1, *b2, *b3, *b4, *part, *frag;
};
LatWork lat_work(const sgp_lattice* L, int C, const CgLat& cl) {
  const int64_t mC = L->m * C;
  LatWork w = {};
  double* p = cl.work;
  for (double** a : {&w.yr, &w.yp, &w.yx, &w.u, &w.b1, &w.b2, &w.b3, &w.b4}) {
    if (a == &w.b3 && blur_arrays(L, C, true, cl.fuse) == 2) break;
    *a = p;
    p += mC;
  }
  w.part = p;
  w.frag = p + L->npiece * C;
  return w;
}

template <int G, int MODE>
int cg_tile_launch(const sgp_lattice* L, int C, const CgLat& cl, const CgHook& hook, const double* Y,
                   const LaunchChoice& lc, hipStream_t s) {
  const LatWork w = lat_work(L, C, cl);
  CgTileArgs a;
  a.n = L->n;
  a.chunks = (C + G - 1) / G;
  a.items = L->ntiles * a.chunks;
  a.P = L->tile_points;
  a.D = L->d + 1;
  a.C = C;
  a.mrows = L->solve_rows;
  a.estride = tile_ent_stride(a.P * a.D);
  a.lds = cg_tile_lds<G>(L, C);
  constexpr int NT = cg_tile_threads<G>();
  const float* b = MODE == CT_FIRST ? cl.rhs : cl.bs;
  // the library's own arrays are aligned (every one of the m x C arrays where
  // C is even); the caller's b and x may not be
  const bool cv = G == 1 || (C % (G < 4 ? G : 4) == 0 && aligned16(cl.work) && aligned16(cl.bs) &&
                             aligned16(b) && (MODE != CT_OUT || aligned16(cl.x)));
  CgHook h = hook;
  auto launch = [&](auto cv_tag) {
    ProfScope ps(KK_SPLAT, s);
    constexpr bool CV = decltype(cv_tag)::value;
    const unsigned grid =
        persistent_grid((const void*)&k_cg_tile<G, MODE, CV>, NT, a.lds.total, a.items, lc.splat_bpc);
    h.fold = grid <= kFoldBlocks ? 1 : 0;
    hipLaunchKernelGGL((k_cg_tile<G, MODE, CV>), dim3(grid), dim3(NT), a.lds.total, s,
                       (const int32_t*)L->tile_off.ptr, (const int32_t*)L->tile_verts.ptr,
                       (const uint16_t*)L->loc.ptr, (const float*)L->ws.ptr, (const int32_t*)L->stile_off.ptr,
                       (const int32_t*)L->tile_ent.ptr, (const uint32_t*)L->slice.ptr,
                       (const int32_t*)L->run_dst.ptr, (const uint8_t*)L->ent_lp.ptr,
                       (const float*)L->ent_w.ptr, Y, b, (const uint32_t*)L->perm.ptr, cl.bs, w.part, cl.x,
                       h, a);
  };
  if (cv)
    launch(std::true_type{});
  else if constexpr (G > 1)
    launch(std::false_type{});
  SGP_LAUNCH_CHECK("k_cg_tile");
  return MODE == CT_OUT || h.fold ? SGP_OK : launch_cg_scalar(h, C, s);
}

enum LatStep { LS_START, LS_FIRST, LS_ITER, LS_OUT };

template <int G>
int lat_cg_g(const sgp_lattice* L, int C, const CgLat& cl, LatStep step, const LaunchChoice& lc, hipStream_t s) {
  const LatWork w = lat_work(L, C, cl);
  const double* beta = cl.beta.st->beta;
  int rc;
  if (step == LS_OUT) return cg_tile_launch<G, CT_OUT>(L, C, cl, cl.beta, w.yx, lc, s);
  if (step == LS_START) {
    if ((rc = cg_tile_launch<G, CT_FIRST>(L, C, cl, cl.start, nullptr, lc, s))) return rc;
    return gather_g<double, G>(L, w.part, w.u, w.frag, C, nullptr, true, s);
  }
  const double* bu = nullptr;
  if ((rc = blur_g<double, G>(L, w.u, w.b1, w.b2, w.b3, w.b4, C, cl.fuse, s, &bu))) return rc;
  const double scale = (L->blur == SGP_BLUR_SYMMETRIC ? 0.5 : 1.0) * (double)L->outputscale;
  CgMvm am = {};
  am.alpha = cl.alpha;
  am.lat_parts = cl.lat_parts;
  if ((rc = launch_cg_alpha(w.u, bu, L->m, C, scale, am, s))) return rc;
  {
    ProfScope ps(KK_CG_DIR, s);
    const int64_t total = L->m * C;
    const int first = step == LS_FIRST ? 1 : 0;
    const CgState* st = cl.alpha.st;
    if (C % 2 == 0 && aligned16(cl.work))
      hipLaunchKernelGGL((k_cg_lattice<2>), dim3(grid_cap(total / 2)), dim3(kBlock), 0, s, bu, w.yr, w.yp,
                         w.yx, total, C, scale, cl.noise, first, st);
    else
      hipLaunchKernelGGL((k_cg_lattice<1>), dim3(grid_cap(total)), dim3(kBlock), 0, s, bu, w.yr, w.yp, w.yx,
                         total, C, scale, cl.noise, first, st);
    SGP_LAUNCH_CHECK("k_cg_lattice");
  }
  if ((rc = cg_tile_launch<G, CT_ITER>(L, C, cl, cl.beta, w.yr, lc, s))) return rc;
  return gather_g<double, G>(L, w.part, w.u, w.frag, C, beta, true, s);
}

size_t cg_tile_lds_g(const sgp_lattice* L, int C, int g) {
  switch (g) {
    case 1: return cg_tile_lds<1>(L, C).total;
    case 2: return cg_tile_lds<2>(L, C).total;
    case 4: return cg_tile_lds<4>(L, C).total;
    case 8: return cg_tile_lds<8>(L, C).total;
    default: return cg_tile_lds<16>(L, C).total;
  }
}

// The widest channel chunk of k_cg_tile.
int lat_lanes(const sgp_lattice* L, int C) {
  int g = lanes_for(C);
  if (g > kMaxChunk) g = kMaxChunk;
  while (g > 1 && cg_tile_lds_g(L, C, g) > kCgTileLds) g >>= 1;
  return g;
}

int lat_cg(const sgp_lattice* L, int C, const CgLat& cl, LatStep step, hipStream_t s) {
  const int g = lat_lanes(L, C);
  LaunchChoice lc{g, 0, 0};
  if (g_force)
    lc = *g_force;
  else
    (void)tune_find(L, C, (int)sizeof(double), TF_LAT, &lc);
  if (lc.g < 1 || lc.g > g || (lc.g & (lc.g - 1))) lc.g = g;
  switch (lc.g) {
    case 1: return lat_cg_g<1>(L, C, cl, step, lc, s);
    case 2: return lat_cg_g<2>(L, C, cl, step, lc, s);
    case 4: return lat_cg_g<4>(L, C, cl, step, lc, s);
    case 8: return lat_cg_g<8>(L, C, cl, step, lc, s);
    default: return lat_cg_g<16>(L, C, cl, step, lc, s);
  }
}

}  // namespace

// Whether a lattice's solves keep their vectors on the lattice. They pay
// while the m lattice rows are few against the n points: an iteration then
// moves 80 m C bytes of lattice vectors in place of 52 n C of point vectors,
// and no more work memory than the point form takes (24 m C against 16 n C
// bytes, hence 2/3). Measured, point form against lattice form: m / n = 0.07
// (n = 2M, d = 11, C = 16) 18.36 -> 14.9 ms for a build and 20 iterations;
// 0.022 (n = 500,000, d = 8, C = 1) 1.79 -> 1.31 ms for 16; 0.44 (n = 2M)
// equal.
// The bound below is for the iterates, not for speed: on smaller lattices they
// depend on the rounding after about 12 iterations (the Krylov basis loses its
// orthogonality once the largest eigenvalue has converged), so those keep the
// point form's arithmetic. In time the lattice form would lose there on few
// points, where the point form has fewer launches, and gain on many (16
// iterations, point | lattice form): n = 20,000, d = 3, m = 715, C = 8 0.58 |
// 0.70 ms; n = 30,011, d = 7, m = 3,132, C = 8 0.85 | 0.89; n = 200,000, d = 6,
// m = 1,410, C = 8 1.40 | 1.15; n = 2M, d = 6, m = 2,048, C = 16 8.08 | 5.03.
// The rule depends on the lattice alone, so a column is solved the same way in
// any batch; point sets of one shape may fall on either side of it.
constexpr int64_t kLatticeCgMin = 4096;
bool cg_on_lattice(const sgp_lattice* L) {
  return L->m >= kLatticeCgMin && 3 * L->m <= 2 * L->n && cg_tile_lds_g(L, kMaxCgCols, 1) <= kCgTileLds;
}

size_t cg_lat_work_elems(const sgp_lattice* L, int C, bool fuse) {
  return (size_t)((4 + blur_arrays(L, C, true, fuse)) * L->m + L->npiece + 2 * gather_ranges(L)) * (size_t)C;
}

int cg_lat_start(const sgp_lattice* L, int C, const CgLat& cl, hipStream_t s) {
  return lat_cg(L, C, cl, LS_START, s);
}
int cg_lat_iter(const sgp_lattice* L, int C, const CgLat& cl, bool first, hipStream_t s) {
  return lat_cg(L, C, cl, first ? LS_FIRST : LS_ITER, s);
}
int cg_lat_out(const sgp_lattice* L, int C, const CgLat& cl, hipStream_t s) {
  return lat_cg(L, C, cl, LS_OUT, s);
}

int mvm_into(const sgp_lattice* L, const float* V, int C, float* out, hipStream_t s) {
  return mvm_dispatch<float>(L, V, (const uint32_t*)L->perm.ptr, C, out, s, 0.f, nullptr);
}

int mvm_cg(const sgp_lattice* L, double* p, int C, hipStream_t s, double noise, const CgMvm& cg,
           const CgDirUpdate* up) {
  return mvm_dispatch<double>(L, p, nullptr, C, cg.r, s, noise, &cg, nullptr, up);
}

size_t mvm_f32_work_bytes(const sgp_lattice* L, int C) {
  return sizeof(float) * mvm_work_elems(L, C, false, blur_fuse_enabled());
}

int mvm_f32(const sgp_lattice* L, const float* V, int C, float* out, hipStream_t s) {
  return mvm_dispatch<float>(L, V, nullptr, C, out, s, 0.f, nullptr);
}

// Times every candidate launch choice on this lattice and keeps the fastest
// for lattices of the same shape. What is timed is what runs: an fp32 MVM, or
// an iteration of a solve in the form that this lattice's take (whose MVM
// carries the direction update where the chunk covers all columns, or which
// has one tile kernel and no slice to choose for).
int autotune(const sgp_lattice* L, int C, bool fp64, int reps, hipStream_t s, int32_t* choice,
             float* best_ms) {
  const int elem = fp64 ? 8 : 4;
  const bool lat = fp64 && cg_on_lattice(L);
  const int gmax = lat ? lat_lanes(L, C) : chunk_lanes(L, C, elem);
  DevBuf buf;
  const size_t bytes = sizeof(float) * (size_t)L->n * (size_t)C;
  int rc = dev_alloc(buf, 2 * bytes, s);
  if (rc) return rc;
  struct Cleanup {
    DevBuf* b;
    hipStream_t s;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    ~Cleanup() {
      g_force = nullptr;
      (void)hipStreamSynchronize(s);
      if (e0) (void)hipEventDestroy(e0);
      if (e1) (void)hipEventDestroy(e1);
      dev_free(*b);
    }
  } cleanup{&buf, s};
  if ((rc = launch_fill_u32((uint32_t*)buf.ptr, bytes / 4, 0x3F800000u, s))) return rc;  // ones
  SGP_HIP(hipEventCreate(&cleanup.e0));
  SGP_HIP(hipEventCreate(&cleanup.e1));
  const float* V = (const float*)buf.ptr;
  float* out = (float*)((char*)buf.ptr + bytes);
  auto time_mvm = [&](float* ms) -> int {
    int rc_ = mvm_into(L, V, C, out, s);  // warm-up (sizes buffers, sets LDS limits)
    if (rc_) return rc_;
    SGP_HIP(hipEventRecord(cleanup.e0, s));
    for (int r = 0; r < reps; ++r)
      if ((rc_ = mvm_into(L, V, C, out, s))) return rc_;
    SGP_HIP(hipEventRecord(cleanup.e1, s));
    SGP_HIP(hipEventSynchronize(cleanup.e1));
    SGP_HIP(hipEventElapsedTime(ms, cleanup.e0, cleanup.e1));
    *ms /= (float)reps;
    return SGP_OK;
  };
  LaunchChoice best{gmax, 0, 0};
  float best_t = -1.f;
  for (int g = gmax; g >= 1 && g >= gmax / 4; g >>= 1) {
    for (int sb = 0; sb <= 1; ++sb) {
      for (int lb = 0; lb <= (lat ? 0 : 1); ++lb) {
        const LaunchChoice cand{g, sb, lb};
        float ms = 0.f;
        g_force = &cand;
        rc = fp64 ? cg_time(L, V, out, C, reps, cleanup.e0, cleanup.e1, &ms, s) : time_mvm(&ms);
        g_force = nullptr;
        if (rc) return rc;
        if (best_t < 0.f || ms < best_t) {
          best_t = ms;
          best = cand;
        }
      }
    }
  }
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    const TuneEntry e{lat ? TF_LAT : TF_MVM, L->d, elem, lanes_for(C), mlog_of(L->m), best, best_t};
    bool found = false;
    for (TuneEntry& x : g_tune)
      if (x.form == e.form && x.d == e.d && x.elem == e.elem && x.g0 == e.g0 && x.mlog == e.mlog) {
        x = e;
        found = true;
      }
    if (!found) g_tune.push_back(e);
  }
  if (choice) {
    choice[0] = best.g;
    choice[1] = best.splat_bpc;
    choice[2] = best.slice_bpc;
  }
  if (best_ms) *best_ms = best_t;
  mark_use(L, s);
  return SGP_OK;
}

void autotune_reset() {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  g_tune.clear();
}

}  // namespace sgp

using namespace sgp;

extern "C" int lattice_mvm(const sgp_lattice* L, const float* values, int32_t C, float* out,
                           void* stream) {
  if (!L || !values || !out) {
    set_error("lattice_mvm: NULL argument");
    return SGP_EINVAL;
  }
  if (C < 1) {
    set_error("lattice_mvm: C must be >= 1 (got %d)", (int)C);
    return SGP_EINVAL;
  }
  const size_t bytes = sizeof(float) * (size_t)L->n * (size_t)C;
  const char* v0 = (const char*)values;
  const char* o0 = (const char*)out;
  if (v0 < o0 + bytes && o0 < v0 + bytes) {
    set_error("lattice_mvm: out overlaps values");
    return SGP_EINVAL;
  }
  const int rc = mvm_into(L, values, C, out, (hipStream_t)stream);
  if (rc == SGP_OK) mark_use(L, (hipStream_t)stream);
  return rc;
}

// Work memory of lattice_mvm_noalloc: one array per device, part of the
// code object, held until the process ends. In host code `scratch` names a
// host-side stand-in, not device memory: kernels receive the device address
// that hipGetSymbolAddress returns for the current device, looked up once per
// device on its first call.
namespace {
constexpr size_t kScratchBytes = (size_t)SGP_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch[kScratchDevices] = {};

int scratch_address(int dev, void** out) {
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      (void)hipGetLastError();
      set_error("lattice_mvm_noalloc: no device address for the scratch array on device %d: %s", dev,
                hipGetErrorString(e));
      return SGP_EHIP;
    }
    g_scratch[dev] = ptr;
  }
  *out = g_scratch[dev];
  return SGP_OK;
}
}  // namespace

extern "C" int lattice_mvm_noalloc(const sgp_lattice* L, const float* values, int32_t C, float* out,
                                   void* stream) {
  if (!L || !values || !out) {
    set_error("lattice_mvm_noalloc: NULL argument");
    return SGP_EINVAL;
  }
  if (C < 1) {
    set_error("lattice_mvm_noalloc: C must be >= 1 (got %d)", (int)C);
    return SGP_EINVAL;
  }
  const size_t bytes = sizeof(float) * (size_t)L->n * (size_t)C;
  const char* v0 = (const char*)values;
  const char* o0 = (const char*)out;
  if (v0 < o0 + bytes && o0 < v0 + bytes) {
    set_error("lattice_mvm_noalloc: out overlaps values");
    return SGP_EINVAL;
  }
  const size_t need = sizeof(float) * mvm_work_elems(L, C, false, false);  // the same whatever the switch says
  if (need > kScratchBytes) {
    set_error("lattice_mvm_noalloc: this lattice and C = %d need %zu bytes of work memory; the "
              "no-allocation entry point has %zu (use lattice_mvm)", (int)C, need, kScratchBytes);
    return SGP_EINVAL;
  }
  int dev = 0;
  SGP_HIP(hipGetDevice(&dev));
  if (dev != L->device || dev < 0 || dev >= kScratchDevices) {
    set_error("lattice_mvm_noalloc: make the lattice's device (%d) current (current: %d)", L->device, dev);
    return SGP_EINVAL;
  }
  void* work = nullptr;
  int rc = scratch_address(dev, &work);
  if (rc) return rc;
  rc = mvm_dispatch<float>(L, values, (const uint32_t*)L->perm.ptr, C, out, (hipStream_t)stream, 0.f,
                           nullptr, work);
  if (rc == SGP_OK) mark_use(L, (hipStream_t)stream);
  return rc;
}

extern "C" int sgp_autotune(const sgp_lattice* L, int32_t C, int32_t fp64, int32_t reps, void* stream,
                            int32_t* choice, float* ms_per_mvm) {
  if (!L) {
    set_error("sgp_autotune: NULL lattice");
    return SGP_EINVAL;
  }
  if (C < 1 || (fp64 && C > kMaxCgCols) || reps < 1) {
    set_error("sgp_autotune: need C >= 1 (at most %d in fp64) and reps >= 1", kMaxCgCols);
    return SGP_EINVAL;
  }
  return autotune(L, C, fp64 != 0, reps, (hipStream_t)stream, choice, ms_per_mvm);
}

extern "C" int sgp_autotune_reset(void) {
  autotune_reset();
  build_tune_reset();
  return SGP_OK;
}
