// Kernels of the CG iteration that keeps its vectors on the lattice.
//
// A = scale W B W^T + noise I, so every vector of the recurrence started at
// b lies in span(b) + range(W):
//   r = rho b + W yr,   p = pi b + W yp,   x = xi b + W yx
// with one scalar per column and m lattice rows in place of n point rows.
// With u = W^T p one step (Section 2, Krylov methods) is
//   p.Ap = scale u.(B u) + noise p.p
//   yx += alpha yp,  xi += alpha pi
//   yr -= alpha (scale B u + noise yp),  rho -= alpha noise pi
//   r.r and u' = W^T r + beta u from one pass over the tiles (k_cg_tile)
//   yp' = yr + beta yp,  pi' = rho + beta pi,  p'.p' = r.r + beta^2 p.p
// (r is orthogonal to the previous p). The residual is formed at every point
// from b and yr, so r.r is a sum of squares as before, with no cancellation
// beyond the rounding of r itself (about 1e-16 |b|).
#ifndef SGP_CG_TILE_H
#define SGP_CG_TILE_H
#include "cg_step.h"
#include "tile.h"

namespace sgp {
namespace {

enum CgTileMode {
  CT_FIRST = 0,  // r = b (gathered from the caller's order and kept in sorted order), splat, b.b
  CT_ITER = 1,   // r = rho b + W yr, splat, r.r
  CT_OUT = 2     // x = xi b + W yx to the caller's order
};

template <int G>
constexpr int cg_tile_threads() { return slice_threads_narrow<G>(); }
// Waves per SIMD that the LDS stage leaves room for.
template <int G>
constexpr int cg_tile_waves() { return G == 4 ? 2 : 4; }
// TileShape with one order block of lattice rows staged at a time: narrow
// chunks stage no more rows than a tile mostly has, and more blocks fit a CU.
template <int G>
struct CgShape : TileShape<double, G, cg_tile_threads<G>()> {
  static constexpr int RC = kSliceOrderRows;
  static constexpr int UPT = RC * G / cg_tile_threads<G>();
};

// LDS layout of k_cg_tile: lattice rows [RC][G], later the tile's residuals
// [P][G] (the splat's zero row is row P then; row RC stays zero) | slice
// weights [P*D] (fp32) | slots [P*D] (uint16) | the splat's lists.
struct CgTileLds {
  int w, sl;
  SplatLists lists;
  size_t total;
};
template <int G>
CgTileLds cg_tile_lds(const sgp_lattice* L, int C) {
  using S = CgShape<G>;
  const int pd = L->tile_points * (L->d + 1);
  CgTileLds o;
  int b = (int)sizeof(double) * (S::RC + 1) * S::RS;
  o.w = b;
  b += 4 * pd;
  o.sl = b;
  b += 2 * (pd + 2);
  o.lists = splat_lists(b, L->max_tile_ents, L->max_tile_pieces);
  const int fold = (int)sizeof(double) * kFold * C;  // the last block's fold
  o.total = (size_t)(o.lists.end > fold ? o.lists.end : fold);
  return o;
}

struct CgTileArgs {
  int64_t n;
  int64_t items;  // tiles x channel chunks
  int P, D, C, chunks;
  int64_t mrows;  // rows whose caller index is >= mrows (> 0) are not solved for
  int estride;    // entries between tiles' splat lists
  CgTileLds lds;
};

// N entries of a point: their staged rows are read together and added in
// vertex order.
template <int N, int RS, int VW>
__device__ __forceinline__ void slice_step(const double* rows, const uint16_t* slot, const float* wt,
                                           double (&acc)[VW]) {
  double x[N][VW], w[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    w[u] = (double)wt[u];
    read_row<double, VW>(rows + (int)slot[u] * RS, x[u]);
  }
#pragma unroll
  for (int u = 0; u < N; ++u)
#pragma unroll
    for (int i = 0; i < VW; ++i) acc[i] = fma_t(w[u], x[u][i], acc[i]);
}

// One tile at a time (persistent blocks, tiles of one XCD's range): the
// slice of the tile's lattice rows gives the residual at its points, whose
// splat goes straight back to partial rows, so neither r nor p nor x is read
// or written per point; b (fp32, sorted order) is the only point array.
// Registers hold the next tile's entries, pieces, b and lattice rows while
// this one is computed, and the row indices of the tile after it, so that the
// row loads never wait for them. Point sums add entries by block of
// kSliceOrderRows runs, then in vertex order, and pieces add entries in
// order, so no result depends on the channel chunk or the grid. CV: rows of C
// channels are whole vectors of a lane's channels, 16-byte aligned.
// Bound by LDS reads and the barriers between its phases: at n = 2M, d = 11,
// C = 16 a tile takes about 9.5 us, of which its 0.83 MB of LDS row reads take
// 3.5 us at the rate of random padded rows (233 of a CU's 300 B/ns, measured).
// What the iteration keeps in flight does not fit the 128 registers of four
// waves a SIMD: 11 of a lane's spill at G = 16 (48 bytes), 19 to 21 at G = 8 and
// 2, 3 at G = 1, and 70 to 80 scalar ones into vector lanes; a spilled value that
// is read back waits behind the tile's loads. G = 4, at two waves, has none.
// 299 us an iteration, where the splat with the direction update (244 us) and
// the slice with the residual update (260 us) moved the same vectors per point.
template <int G, int MODE, bool CV>
__global__ __launch_bounds__(cg_tile_threads<G>()) __attribute__((amdgpu_waves_per_eu(cg_tile_waves<G>()))) void k_cg_tile(
    const int32_t* __restrict__ tile_off, const int32_t* __restrict__ tile_verts,
    const uint16_t* __restrict__ loc, const float* __restrict__ ws,
    const int32_t* __restrict__ stile_off, const int32_t* __restrict__ tile_ent,
    const uint32_t* __restrict__ slice, const int32_t* __restrict__ run_dst, const uint8_t* __restrict__ ent_lp,
    const float* __restrict__ ent_w, const double* __restrict__ Y, const float* __restrict__ b,
    const uint32_t* __restrict__ perm, float* __restrict__ bs, double* __restrict__ part,
    float* __restrict__ x, CgHook hook, CgTileArgs a) {
  constexpr int NT = cg_tile_threads<G>();
  using S = CgShape<G>;
  static_assert(S::RC > S::kPts, "a tile's residuals and a zero row fit the staged rows");
  constexpr int RC = S::RC;
  constexpr bool kSlice = MODE != CT_FIRST, kSplat = MODE != CT_OUT;
  constexpr int VL = G >= 2 ? 2 : 1;  // elements per staged load
  constexpr int LV = S::UPT / VL;     // staged loads per thread
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double s_coef[kMaxCgCols];
  double* lu = (double*)smem;
  float* lw = (float*)(smem + a.lds.w);
  uint16_t* lsl = (uint16_t*)(smem + a.lds.sl);
  const int tid = threadIdx.x;
  const int grp = tid / S::LPR;
  const int cl = (tid % S::LPR) * S::VW;  // this lane's channel offset within a chunk
  // points reached through the permutation, or checked against mrows
  const bool use_perm = MODE != CT_ITER || a.mrows > 0;

  float w[S::EPT], bn[S::PPG][S::VW];
  uint32_t sl2[S::EPT / 2];
  int32_t vj[LV], pr[S::PPG];
  SplatFetch<NT> lists;
  double ur[S::UPT];
  struct Meta {
    int t, ch, np, nq, nqp, q0, qp0, ents;
  };
  auto load_index = [&](int r0, int nr, const int32_t* verts) {
#pragma unroll
    for (int u = 0; u < LV; ++u) {
      const int r = (tid + u * NT) * VL / G;
      vj[u] = verts[r0 + (r < nr ? r : nr - 1)];
    }
  };
  auto load_rows = [&](int ch) {
#pragma unroll
    for (int u = 0; u < LV; ++u) {
      const int c = ch * G + (tid + u * NT) * VL % G;
      const double* src = Y + (int64_t)vj[u] * a.C;
      if constexpr (VL == 2 && CV) {
        const dvec2 v = *(const dvec2*)(src + (c < a.C ? c : 0));
        ur[u * VL] = v[0];
        ur[u * VL + VL - 1] = v[1];
      } else {
#pragma unroll
        for (int i = 0; i < VL; ++i) ur[u * VL + i] = src[c + i < a.C ? c + i : a.C - 1];
      }
    }
  };
  auto stage_rows = [&](int nr) {
#pragma unroll
    for (int u = 0; u < LV; ++u) {
      const int f = (tid + u * NT) * VL;
      if (f < nr * G) {
        double* d = lu + (f / G) * S::RS + f % G;
        if constexpr (VL == 2) {
          dvec2 v;
          v[0] = ur[u * 2];
          v[1] = ur[u * 2 + 1];
          *(dvec2*)d = v;
        } else {
          *d = ur[u];
        }
      }
    }
  };
  // Every load is unconditional (indices clamped into the tile). Entries are
  // read once per iteration: non-temporal, which keeps the lattice rows and
  // the partial rows in the caches.
  auto fetch_index = [&](int item, Meta& mt) {
    const int t = a.chunks == 1 ? item : (int)((unsigned)item / (unsigned)a.chunks);
    const int64_t p0 = (int64_t)t * a.P;
    mt.t = t;
    mt.ch = item - t * a.chunks;
    mt.np = (int)(a.n - p0 < a.P ? a.n - p0 : a.P);
    if constexpr (kSlice) {
      mt.q0 = tile_off[t];
      mt.nq = tile_off[t + 1] - mt.q0;
      load_index(0, mt.nq < RC ? mt.nq : RC, tile_verts + mt.q0);
    }
    if constexpr (kSplat) {
      mt.qp0 = stile_off[t];
      mt.nqp = stile_off[t + 1] - mt.qp0;
      mt.ents = tile_ent[t];
    }
    if (use_perm) {
#pragma unroll
      for (int k = 0; k < S::PPG; ++k) {
        const int lp = grp + k * S::NG;
        pr[k] = (int32_t)perm[p0 + (lp < mt.np ? lp : mt.np - 1)];
      }
    }
  };
  int32_t prc[S::PPG];  // caller rows of the tile whose loads were issued last
  auto fetch = [&](const Meta& mt) {
    const int64_t p0 = (int64_t)mt.t * a.P, e0 = p0 * a.D;
    const int ne = mt.np * a.D;
    if constexpr (kSlice) load_rows(mt.ch);
#pragma unroll
    for (int k = 0; k < S::PPG; ++k) {
      const int lp = grp + k * S::NG;
      prc[k] = use_perm ? pr[k] : 0;
      const int64_t row = MODE == CT_FIRST ? (int64_t)pr[k] : p0 + (lp < mt.np ? lp : mt.np - 1);
      const int cg = mt.ch * G + cl;
      const float* src = b + row * a.C;
      if constexpr (CV) {
        read_row_nt<float, S::VW>(src + (cg < a.C ? cg : 0), bn[k]);
      } else {
#pragma unroll
        for (int i = 0; i < S::VW; ++i) bn[k][i] = src[cg + i < a.C ? cg + i : a.C - 1];
      }
    }
    if constexpr (kSlice) {
#pragma unroll
      for (int u = 0; u < S::EPT; ++u) {
        const int e = tid + u * NT;
        w[u] = __builtin_nontemporal_load(ws + e0 + (e < ne ? e : ne - 1));
      }
      // slots in pairs (the tile starts 4-byte aligned; the array has a
      // spare slot past its end)
      const uint32_t* gsl2 = (const uint32_t*)(loc + e0);
      const int npair = (ne + 1) / 2;
#pragma unroll
      for (int u = 0; u < S::EPT / 2; ++u) {
        const int pi = tid + u * NT;
        sl2[u] = __builtin_nontemporal_load(gsl2 + (pi < npair ? pi : npair - 1));
      }
    }
  };

  if constexpr (kSlice) {
    for (int c = tid; c < a.C && c < kMaxCgCols; c += NT)
      s_coef[c] = MODE == CT_OUT ? hook.st->xi[c] : hook.st->rho[c];
  }
  int64_t item0, end0, step0;
  xcd_items(a.items, &item0, &end0, &step0);
  int item = (int)item0;
  const int end = (int)end0, step = (int)step0;
  for (int i = tid; i < S::RS; i += NT) lu[RC * S::RS + i] = 0.0;  // the slice's zero row
  Meta cur = {}, nxt = {};
  if (item < end) {
    fetch_index(item, cur);
    fetch(cur);
    if (item + step < end) fetch_index(item + step, nxt);
  }
  for (; item < end; item += step) {
    const int64_t p0 = (int64_t)cur.t * a.P;
    const int ne = cur.np * a.D;
    const int cg = cur.ch * G + cl;
    const bool live = cg < a.C;
    __syncthreads();  // the previous tile is done with the LDS
    if constexpr (kSlice) {
#pragma unroll
      for (int u = 0; u < S::EPT; ++u) {
        const int e = tid + u * NT;
        if (e < ne) lw[e] = w[u];
      }
#pragma unroll
      for (int u = 0; u < S::EPT / 2; ++u) {
        const int pi = tid + u * NT;
        if (2 * pi < ne) ((uint32_t*)lsl)[pi] = sl2[u];
      }
      stage_rows(cur.nq < RC ? cur.nq : RC);
    }
    // the splat's lists of this tile: in flight during its slice
    const float* ew = ent_w + (int64_t)cur.t * a.estride;
    const uint8_t* elp = ent_lp + (int64_t)cur.t * a.estride;
    const uint32_t* esl = slice + tile_slice0(cur.qp0, cur.t);
    if constexpr (kSplat) lists.load(ew, elp, run_dst + cur.qp0, esl, cur.ents, cur.nqp);
    float bv[S::PPG][S::VW];
    int32_t prow[S::PPG];
#pragma unroll
    for (int k = 0; k < S::PPG; ++k) {
      prow[k] = prc[k];
#pragma unroll
      for (int i = 0; i < S::VW; ++i) bv[k][i] = bn[k][i];
    }
    __syncthreads();
    // the next tile's loads (its row indices are here), then the indices of
    // the one after; a tile with more runs than a chunk needs the registers
    // for its own rows first
    const bool next = item + step < end, next2 = item + 2 * step < end;
    Meta nx2 = {};
    auto advance = [&]() {
      if (next) fetch(nxt);
      if (next2) fetch_index(item + 2 * step, nx2);
    };
    const bool one_pass = !kSlice || cur.nq <= RC;
    if (one_pass) advance();
    double acc[S::PPG][S::VW];
#pragma unroll
    for (int k = 0; k < S::PPG; ++k)
#pragma unroll
      for (int i = 0; i < S::VW; ++i) acc[k][i] = 0.0;
    if constexpr (kSlice) {
      for (int r0 = 0; r0 < cur.nq; r0 += RC) {
        const int nr = cur.nq - r0 < RC ? cur.nq - r0 : RC;
        if (r0 > 0) {
          __syncthreads();  // previous chunk consumed
          load_index(r0, nr, tile_verts + cur.q0);
          load_rows(cur.ch);
          stage_rows(nr);
          __syncthreads();
          if (r0 + RC >= cur.nq) {
            if (next) fetch_index(item + step, nxt);  // its indices were overwritten
            advance();
          }
        }
        if (live) {
#pragma unroll
          for (int k = 0; k < S::PPG; ++k) {
            const int lp = grp + k * S::NG;
            if (lp >= cur.np) continue;
            const uint16_t* es = lsl + lp * a.D;
            const float* ew1 = lw + lp * a.D;
            constexpr int EB = S::VW >= 4 ? 2 : 4;  // entries at a time
            if (one_pass) {
              // every entry's row is staged
              int j = 0;
              for (; j + EB <= a.D; j += EB) slice_step<EB, S::RS>(lu + cl, es + j, ew1 + j, acc[k]);
              for (; j < a.D; ++j) slice_step<1, S::RS>(lu + cl, es + j, ew1 + j, acc[k]);
            } else {
              // (an entry outside the chunk reads the zero row with weight 0,
              // which leaves acc as it is)
              for (int j = 0; j < a.D; ++j) {
                const int sr = (int)es[j] - r0;
                const bool in = (unsigned)sr < (unsigned)nr;
                double xr[S::VW];
                read_row<double, S::VW>(lu + (in ? sr : RC) * S::RS + cl, xr);
                const double wv = (double)(in ? ew1[j] : 0.f);
#pragma unroll
                for (int i = 0; i < S::VW; ++i) acc[k][i] = fma_t(wv, xr[i], acc[k][i]);
              }
            }
          }
        }
      }
    }
    // r (or x) at this thread's points
#pragma unroll
    for (int k = 0; k < S::PPG; ++k) {
      const int lp = grp + k * S::NG;
      const bool masked = a.mrows > 0 && (int64_t)prow[k] >= a.mrows;  // not solved for
#pragma unroll
      for (int i = 0; i < S::VW; ++i) {
        double v = (double)bv[k][i];
        if constexpr (kSlice) v = fma_t(s_coef[cg + i < a.C ? cg + i : 0], v, acc[k][i]);
        acc[k][i] = masked || (CV ? cg : cg + i) >= a.C ? 0.0 : v;
      }
      if (lp < cur.np && live) {
        if constexpr (MODE == CT_FIRST) {
          float* d = bs + (p0 + lp) * a.C + cg;
          if constexpr (CV) {
            write_row<float, S::VW>(d, bv[k]);
          } else {
#pragma unroll
            for (int i = 0; i < S::VW; ++i)
              if (cg + i < a.C) d[i] = bv[k][i];
          }
        }
        if constexpr (MODE == CT_OUT) {
          float o[S::VW];
#pragma unroll
          for (int i = 0; i < S::VW; ++i) o[i] = (float)acc[k][i];
          float* d = x + (int64_t)prow[k] * a.C + cg;
          if constexpr (CV) {
            write_row<float, S::VW>(d, o);
          } else {
#pragma unroll
            for (int i = 0; i < S::VW; ++i)
              if (cg + i < a.C) d[i] = o[i];
          }
        }
      }
    }
    if constexpr (kSplat) {
      lists.stage(smem, a.lds.lists, ew, elp, run_dst + cur.qp0, esl, cur.ents, cur.nqp,
                  S::RS * (int)sizeof(double), a.P);
      if constexpr (kSlice) __syncthreads();  // every lane is done with the staged rows
#pragma unroll
      for (int k = 0; k < S::PPG; ++k) {
        const int lp = grp + k * S::NG;
        if (lp < cur.np) write_row<double, S::VW>(lu + lp * S::RS + cl, acc[k]);
      }
      if (tid < S::RS) lu[a.P * S::RS + tid] = 0.0;  // the splat's zero row
      __syncthreads();
      // the tile's r.r per column
      if (tid < 16 * G) {
        const int cc = tid / 16;
        const double rr = tile_sumsq<S::RS>(lu, tid % 16, cc, cur.np);
        if (tid % 16 == 0 && cur.ch * G + cc < a.C) hook.partials[(int64_t)cur.t * a.C + cur.ch * G + cc] = rr;
      }
      splat_pieces_split<double, G, NT>(smem, smem, a.lds.lists, cur.nqp, part, a.C, cur.ch * G, CV);
    }
    cur = nxt;
    nxt = nx2;
  }
  if constexpr (kSplat) {
    cg_finish(hook, a.C, (double*)smem);
  }
}

// The step's lattice vectors, element by element (alpha and beta known):
// yp = yr + beta yp for columns still active (the direction of this
// iteration, beta of the previous one), yx += alpha yp,
// yr -= alpha (scale B u + noise yp). first: yp = yx = yr = 0 before.
// Seven streams of m x C fp64: bound by the cache that holds them (m = 141,000,
// 16 columns 23 us, 5.5 TB/s).
template <int VL>
__global__ __launch_bounds__(kBlock) void k_cg_lattice(const double* __restrict__ bu, double* __restrict__ yr,
                                                       double* __restrict__ yp, double* __restrict__ yx,
                                                       int64_t total, int C, double scale, double noise,
                                                       int first, const CgState* __restrict__ st) {
  typedef double dv __attribute__((ext_vector_type(VL)));
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; h < total / VL; h += stride) {
    const int c = (int)((h * VL) % C);
    const dv b = *(const dv*)(bu + h * VL);
    dv r, p, q;
    if (first) {
#pragma unroll
      for (int i = 0; i < VL; ++i) r[i] = p[i] = q[i] = 0.0;
    } else {
      r = *(const dv*)(yr + h * VL);
      p = *(const dv*)(yp + h * VL);
      q = *(const dv*)(yx + h * VL);
    }
#pragma unroll
    for (int i = 0; i < VL; ++i) {
      const double al = st->alpha[c + i];
      if (st->active[c + i]) p[i] = __builtin_fma(st->beta[c + i], p[i], r[i]);
      q[i] = __builtin_fma(al, p[i], q[i]);
      r[i] = __builtin_fma(-al, __builtin_fma(noise, p[i], scale * b[i]), r[i]);
    }
    *(dv*)(yr + h * VL) = r;
    *(dv*)(yp + h * VL) = p;
    *(dv*)(yx + h * VL) = q;
  }
}

}  // namespace
}  // namespace sgp
#endif  // SGP_CG_TILE_H
