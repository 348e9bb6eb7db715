// The lattice part of an MVM, one block per column, for lattices whose column
// fits a CU's LDS: what is left of the splat's gather (lattice points whose
// partial rows span gather ranges), the whole blur, and inside CG p.Ap and
// alpha.
#ifndef SGP_LATTICE_COL_H
#define SGP_LATTICE_COL_H
#include "cg_step.h"
#include "tile.h"

namespace sgp {
namespace {

constexpr int kColThreads = 1024;
constexpr int kColRows = 2 * kColThreads;  // most lattice points
constexpr int kColParts = 1024;            // most partial sums of p.Ap

enum ColMode {
  CM_MVM = 0,  // blur
  CM_CG = 1    // and alpha of the CG iteration (CgMvm)
};

// Columns of one launch: 2^30 threads (a grid has less than 2^32).
constexpr int kColGrid = 1 << 20;

struct ColArgs {
  int m, C, D;
  int c0;          // first column
  int rshift;      // log2 of the rows per gather range
  int first, rev;  // chains to run: directions 0 .. d, and d .. 0
  int lat_parts, ntiles;
  double scale;
  double st[3];
};

// Padded place of row j, so that a thread reading eight consecutive rows does
// not share its LDS bank with its neighbours.
__host__ __device__ __forceinline__ int col_at(int j) { return j + (j >> 3); }

template <typename TU, int MODE>
size_t col_lds(const ColArgs& a) {
  if (MODE == CM_MVM) return sizeof(TU) * (size_t)a.m;
  return sizeof(double) * (size_t)(2 * (col_at(a.m) + 1) + a.m / 8 + 1 + a.lat_parts + (a.ntiles + 15) / 16 + kFold);
}

// A block filters a column. Thread t holds rows t + i * 1024 in registers; a
// blur step reads the neighbours' rows from LDS, and the next step's neighbour
// indices are in flight meanwhile. Every sum is formed as by the kernels that
// larger lattices use (k_gather_fix, the blur, k_cg_alpha, the fold), in the
// same order, so that results are the same bit for bit. Bound by the latency
// of its steps (two barriers and the LDS reads, some 0.4 us): m = 430, d = 3,
// one column 4.0 us for an MVM's part and 7.7 us inside CG, where the
// launches that it stands for took 12 and 22 us.
template <typename TU, int NR, int MODE>
__global__ __launch_bounds__(kColThreads) void k_lattice_col(TU* __restrict__ U, const TU* __restrict__ frag,
                                                             const int32_t* __restrict__ occ_ptr,
                                                             const int32_t* __restrict__ nbr, TU* __restrict__ Bu,
                                                             const double* __restrict__ pp, CgHook h, ColArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  TU* A = (TU*)smem;
  const int rows = col_at(a.m) + 1;
  TU* us = A + rows;                       // CG: the column before the blur
  double* gs = (double*)(us + rows);       // CG: sums of 8 rows, then partial sums and their fold
  double* parts = gs + a.m / 8 + 1;
  double* fold = parts + (a.lat_parts + (a.ntiles + 15) / 16);
  const int tid = threadIdx.x, c = a.c0 + (int)blockIdx.x;
  const int m = a.m;
  TU st[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) st[t] = (TU)a.st[t];
  TU u[NR], f[NR], v[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int j = tid + i * kColThreads;
    u[i] = 0;
    f[i] = 0;
    v[i] = 0;
    if (j < m) {
      const int js = occ_ptr[j], je = occ_ptr[j + 1];
      const int g0 = js >> a.rshift, g1 = (je - 1) >> a.rshift;
      const int64_t at = (int64_t)j * a.C + c;
      TU x = U[at];
      if (g0 != g1) {  // rows in several ranges: their fragments in range order
        x = frag_sum(frag, ((int64_t)g0 * 2 + (js == g0 << a.rshift ? 0 : 1)) * a.C + c, g0, g1, a.C, c);
        U[at] = x;
      }
      u[i] = x;
      if (MODE == CM_CG) us[col_at(j)] = x;
    }
  }
  auto chain = [&](bool reverse, TU (&o)[NR]) {
    int2 nb[NR];
    auto indices = [&](int s) {
      const int2* src = (const int2*)nbr + (int64_t)(reverse ? a.D - 1 - s : s) * m;
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const int j = tid + i * kColThreads;
        nb[i] = src[j < m ? j : m - 1];
      }
    };
    indices(0);
    __syncthreads();  // the LDS column is free
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int j = tid + i * kColThreads;
      o[i] = u[i];
      if (j < m) A[j] = o[i];
    }
    __syncthreads();
    for (int s = 0; s < a.D; ++s) {
      TU lo[NR], hi[NR];
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        lo[i] = A[nb[i].x >= 0 ? nb[i].x : 0];
        hi[i] = A[nb[i].y >= 0 ? nb[i].y : 0];
        lo[i] = nb[i].x >= 0 ? lo[i] : (TU)0;
        hi[i] = nb[i].y >= 0 ? hi[i] : (TU)0;
      }
      if (s + 1 < a.D) indices(s + 1);
      __syncthreads();  // every neighbour has been read
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const int j = tid + i * kColThreads;
        o[i] = fma_t(st[2], hi[i], fma_t(st[1], o[i], fma_t(st[0], lo[i], (TU)0)));
        if (j < m && s + 1 < a.D) A[j] = o[i];
      }
      __syncthreads();
    }
  };
  if (a.first) chain(false, f);
  if (a.rev) {
    chain(true, v);
#pragma unroll
    for (int i = 0; i < NR; ++i) f[i] = a.first ? f[i] + v[i] : v[i];
  }
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int j = tid + i * kColThreads;
    if (j < m) Bu[(int64_t)j * a.C + c] = f[i];
  }
  if constexpr (MODE == CM_CG) {
    // p.Ap = scale * u.(B u) (+ noise * p.p): sums of 8 rows, of 16 of those,
    // and of two chunks, then the tiles' p.p by 16
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int j = tid + i * kColThreads;
      if (j < m) A[col_at(j)] = f[i];
    }
    __syncthreads();
    const int groups = (m + 7) / 8;
    for (int g = tid; g < groups; g += kColThreads) {
      double dot = 0.0;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int j = 8 * g + k;
        const double x = j < m ? (double)us[col_at(j)] : 0.0, y = j < m ? (double)A[col_at(j)] : 0.0;
        if (j < m) dot = __builtin_fma(x, y, dot);
      }
      gs[g] = a.scale * dot;
    }
    __syncthreads();
    for (int s = tid; s < a.lat_parts; s += kColThreads) {
      double acc = 0.0;
      for (int ck = 2 * s; ck < 2 * s + 2 && ck * 16 < groups; ++ck) {
        double w = 0.0;
        for (int g = 16 * ck; g < 16 * ck + 16 && g < groups; ++g) w += gs[g];
        acc += w;
      }
      parts[s] = acc;
    }
    const int pg = (a.ntiles + 15) / 16, nparts = a.lat_parts + pg;
    for (int g = tid; g < pg; g += kColThreads) {
      double w = 0.0;
      for (int t = 16 * g; t < 16 * g + 16 && t < a.ntiles; ++t) w += pp[(int64_t)t * a.C + c];
      parts[a.lat_parts + g] = w;
    }
    __syncthreads();
    if (tid < kFold) {
      double s = 0.0;
      for (int b = tid; b < nparts; b += kFold) s += parts[b];
      fold[tid] = s;
    }
    __syncthreads();
    if (tid == 0) {
      double w = 0.0;
      for (int g = 0; g < kFold && g < nparts; ++g) w += fold[g];
      cg_scalar_column(h.st, c, h.mode, h.tol, h.noise, w);
    }
  }
}

}  // namespace
}  // namespace sgp
#endif  // SGP_LATTICE_COL_H
