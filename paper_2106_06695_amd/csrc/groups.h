// Groups of blur directions: for up to kGroupDirs consecutive directions, the
// lattice points that are connected through neighbours along them (a part;
// neighbours are R = 1 or 2 points to either side, the stencil's order) are brought together in tiles of kGroupRows
// rows, so that the blur takes the whole group of directions in one pass
// (k_blur_group). A point set of bounded extent has few points per part: four
// directions join at most 132 of them at m = 141,000 (d = 11), 189 at
// m = 874,000 (d = 11), 166 at m = 4.2M (d = 16). To find and place them takes
// 0.1 ms of a build at m = 141,000 (d = 11), 0.4 ms at 681,000 (d = 20), 3.0 ms
// at 4.2M (d = 16), random accesses to the roots; a blur there gains 0.1, 0.3
// and 2 ms. On dense lattices of few dimensions the first cut does not fit and is
// divided. Builds without any search, with every cut joined and counted, and
// with those left out that a sampled part tells not to fit (k_group_init), which
// adds some 8 us where the first cut fits: m = 62,000 (d = 6) 0.56, 0.94, 0.73 ms;
// 245,000 (d = 6) 1.06, 1.98, 1.32; 673,000 (d = 8) 2.25, 3.12, 2.55; 1.13M
// (d = 5, no groups in the end) 3.05, 4.70, 2.95 (its neighbour look-ups are
// faster now, too). Groups that are no fewer passes than the fused pairs only
// pay there with wide rows (blur_by_groups).
#ifndef SGP_GROUPS_H
#define SGP_GROUPS_H
#include <hip/hip_runtime.h>

#include "sgp_internal.h"

namespace sgp {
namespace {

// Parts are kept by size class, so that tiles fill without a search: sizes
// 1 .. 15 have a class each, larger ones share the class of as many parts a
// tile (15 .. 1). A tile's last row stays empty.
__host__ __device__ constexpr int group_class(int size) { return size <= 15 ? size - 1 : 30 - kGroupPart / size; }
__host__ __device__ constexpr int group_per_tile(int c) { return c < 15 ? kGroupPart / (c + 1) : 30 - c; }
__host__ __device__ constexpr int group_stride(int c) { return c < 15 ? c + 1 : kGroupPart / (30 - c); }

struct GroupSpec {
  int first[kMaxGroups], dirs[kMaxGroups];
  int skip[kMaxGroups];       // parts known already
  int64_t tile0[kMaxGroups];  // first tile
};

// The root of x: every entry points to a smaller index or, at a root, to
// itself. Other threads join roots meanwhile; a value read too early is still
// one of x's ancestors. HALVE shortens the path on the way.
template <bool HALVE>
__device__ __forceinline__ int32_t group_find(int32_t* parent, int32_t x) {
  int32_t p = parent[x];
  while (p != x) {
    const int32_t g = parent[p];
    if (HALVE && g != p) parent[x] = g;
    x = p;
    p = g;
  }
  return x;
}

// A point's neighbours along direction k: -R .. -1, 1 .. R.
template <int R>
__device__ __forceinline__ void group_nbrs(const int32_t* nbr, int64_t k, int64_t m, int64_t j, int32_t (&o)[2 * R]) {
  if constexpr (R == 1) {
    const int2 v = ((const int2*)nbr)[k * m + j];
    o[0] = v.x;
    o[1] = v.y;
  } else {
    const int4 v = ((const int4*)nbr)[k * m + j];
    o[0] = v.x;
    o[1] = v.y;
    o[2] = v.z;
    o[3] = v.w;
  }
}

// Whether the part of `start` has more than kGroupPart points: its points are
// visited breadth first by one block, a thread per neighbour, for at most
// kGroupSteps steps. False may also mean that they did not suffice. A step adds
// at most a point a thread to the 255 there are, so the table is never full.
constexpr int kGroupSteps = 16;
template <int R>
__device__ inline bool group_outgrows(const int32_t* __restrict__ nbr, int64_t m, int first, int dirs,
                                      int32_t start) {
  constexpr int E = 2 * R * kGroupDirs, T = 1024;
  __shared__ int32_t list[kGroupRows], table[T];
  __shared__ int count;
  const int tid = threadIdx.x;
  auto slot_of = [](int32_t x) { return (int)((uint32_t)x * 0x9E3779B1u >> 22); };
  for (int i = tid; i < T; i += 256) table[i] = -1;
  __syncthreads();
  if (tid == 0) {
    list[0] = start;
    table[slot_of(start)] = start;
    count = 1;
  }
  __syncthreads();
  int done = 0, known = 1;  // points visited, and found
  for (int step = 0; step < kGroupSteps && done < known && known <= kGroupPart; ++step) {
    const int i = done + tid / E, e = tid % E;
    if (i < known && e / (2 * R) < dirs) {
      const int32_t x = nbr[((first + e / (2 * R)) * m + list[i]) * (2 * R) + e % (2 * R)];
      for (int s = x >= 0 ? slot_of(x) : -1; s >= 0; s = (s + 1) % T) {
        const int32_t old = (int32_t)atomicCAS((uint32_t*)table + s, ~0u, (uint32_t)x);
        if (old == x) break;
        if (old < 0) {
          const int at = atomicAdd(&count, 1);
          if (at < kGroupRows) list[at] = x;
          break;
        }
      }
    }
    __syncthreads();
    done = done + 256 / E < known ? done + 256 / E : known;
    known = count;
    __syncthreads();
  }
  return known > kGroupPart;
}

// Whether a group's parts are known already, or one of its samples outgrows a
// tile (k_group_init): every thread of a block gets the same answer.
__device__ __forceinline__ bool group_over(const uint8_t* __restrict__ over, int g) {
  static_assert(kGroupSamples == 4 * 64, "four answers a lane");
  return __ballot(((const uint32_t*)(over + g * kGroupSamples))[threadIdx.x & 63] != 0) != 0;
}

// parent = the smallest of a point and its neighbours along the group; also
// clears the sizes and the class counts. The first kGroupSamples blocks look at
// the part of a point each: a group whose parts outgrow a tile mostly has many
// points in such parts (17 to 95% on dense lattices of d = 5 to 7, 1% at d = 8),
// and to join and count them takes many steps to few roots (m = 245,000, d = 6,
// groups of four and three directions: 530 us), so it is then left out.
template <int R>
__global__ __launch_bounds__(256) void k_group_init(const int32_t* __restrict__ nbr, int64_t m, GroupSpec sp,
                                                    int32_t* __restrict__ parent, int32_t* __restrict__ info,
                                                    uint32_t* __restrict__ cnt, uint8_t* __restrict__ over) {
  const int g = (int)blockIdx.y;
  if (sp.skip[g]) return;
  if (blockIdx.x < kGroupSamples) {
    const int64_t at = (2 * (int64_t)blockIdx.x + 1) * m / (2 * kGroupSamples);
    const bool big = group_outgrows<R>(nbr, m, sp.first[g], sp.dirs[g], (int32_t)at);
    if (threadIdx.x == 0) over[g * kGroupSamples + blockIdx.x] = big ? 1 : 0;
    return;
  }
  const int64_t block = (int64_t)blockIdx.x - kGroupSamples;
  if (block == 0 && threadIdx.x < kGroupWords) cnt[g * kGroupWords + threadIdx.x] = 0;
  const int64_t stride = (int64_t)(gridDim.x - kGroupSamples) * blockDim.x;
  for (int64_t j = block * blockDim.x + threadIdx.x; j < m; j += stride) {
    int32_t p = (int32_t)j;
#pragma unroll
    for (int t = 0; t < kGroupDirs; ++t)
      if (t < sp.dirs[g]) {
        int32_t nb[2 * R];
        group_nbrs<R>(nbr, sp.first[g] + t, m, j, nb);
#pragma unroll
        for (int i = 0; i < 2 * R; ++i)
          if (nb[i] >= 0 && nb[i] < p) p = nb[i];
      }
    parent[g * m + j] = p;
    info[g * m + j] = 0;
  }
}

// Join the two ends of every neighbour pair. A root is only ever linked to a
// smaller index, by compare-and-swap, so every loop here goes strictly down
// and ends.
template <int R>
__global__ __launch_bounds__(256) void k_group_join(const int32_t* __restrict__ nbr, int64_t m, GroupSpec sp,
                                                    int32_t* __restrict__ parents,
                                                    const uint8_t* __restrict__ over) {
  const int g = (int)blockIdx.y;
  if (sp.skip[g] || group_over(over, g)) return;
  int32_t* parent = parents + g * m;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < m; j += stride) {
    int32_t hi[R * kGroupDirs];  // each pair from its lower end
#pragma unroll
    for (int t = 0; t < R * kGroupDirs; ++t)
      hi[t] = t / R < sp.dirs[g] ? nbr[2 * R * ((int64_t)(sp.first[g] + t / R) * m + j) + R + t % R] : -1;
    int32_t a = (int32_t)j;
#pragma unroll
    for (int t = 0; t < R * kGroupDirs; ++t) {
      if (hi[t] < 0) continue;
      a = group_find<true>(parent, a);
      int32_t b = group_find<true>(parent, hi[t]);
      while (a != b) {
        if (a < b) {
          const int32_t x = a;
          a = b;
          b = x;
        }
        const int32_t old = (int32_t)atomicCAS((uint32_t*)parent + a, (uint32_t)a, (uint32_t)b);
        if (old == a) break;
        a = group_find<true>(parent, old);
      }
      a = a < b ? a : b;
    }
  }
}

// Every point's root, its place among the part's points, and the part's size
// (in info, at the root). Points of a wave with its first lane's root are
// counted together: a part of a lattice without gaps may hold every point.
__global__ __launch_bounds__(256) void k_group_count(int64_t m, GroupSpec sp, int32_t* __restrict__ parents,
                                                     int32_t* __restrict__ infos, int32_t* __restrict__ place,
                                                     const uint8_t* __restrict__ over) {
  if (sp.skip[blockIdx.y] || group_over(over, (int)blockIdx.y)) return;
  const int64_t at = blockIdx.y * m;
  int32_t* parent = parents + at;
  int32_t* info = infos + at;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int lane = threadIdx.x & 63;
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < m; j += stride) {
    const int32_t r = group_find<false>(parent, (int32_t)j);
    parent[j] = r;  // the only store here: a late one of an ancestor would undo it
    const int32_t r0 = __builtin_amdgcn_readfirstlane(r);
    const unsigned long long same = __ballot(r == r0);
    const int lead = (int)__ffsll(same) - 1;
    int before = 0;
    if (r == r0)
      before = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(same >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)same, 0));
    int base = 0;
    if (r != r0 || lane == lead) base = atomicAdd(info + r, r == r0 ? (int)__popcll(same) : 1);
    const int base0 = __shfl(base, lead);
    place[at + j] = (r == r0 ? base0 : base) + before;
  }
}

// Number the parts within their size classes: at a root, info becomes
// (number << 5) | class. cnt: a group's parts by class, then the largest (of a
// group that was left out, a size past a tile's).
constexpr int kGroupSpan = 8;
__global__ __launch_bounds__(256) void k_group_class(int64_t m, GroupSpec sp, const int32_t* __restrict__ parents,
                                                     int32_t* __restrict__ infos, uint32_t* __restrict__ cnts,
                                                     const uint8_t* __restrict__ over) {
  __shared__ uint32_t hist[kGroupClasses], first[kGroupClasses];
  __shared__ int largest;
  if (sp.skip[blockIdx.y]) return;
  const int64_t at = blockIdx.y * m;
  uint32_t* cnt = cnts + blockIdx.y * kGroupWords;
  const int tid = threadIdx.x;
  if (group_over(over, (int)blockIdx.y)) {
    if (blockIdx.x == 0 && tid == 0) cnt[kGroupClasses] = kGroupRows;
    return;
  }
  if (tid < kGroupClasses) hist[tid] = 0;
  if (tid == 0) largest = 0;
  __syncthreads();
  int cls[kGroupSpan];
  uint32_t num[kGroupSpan];
#pragma unroll
  for (int i = 0; i < kGroupSpan; ++i) {
    const int64_t j = ((int64_t)blockIdx.x * kGroupSpan + i) * 256 + tid;
    cls[i] = -1;
    num[i] = 0;
    if (j < m && parents[at + j] == (int32_t)j) {
      const int size = infos[at + j];
      cls[i] = group_class(size < kGroupPart ? size : kGroupPart);
      if (size > kGroupRows / 2) atomicMax(&largest, size);
      num[i] = atomicAdd(&hist[cls[i]], 1u);
    }
  }
  __syncthreads();
  if (tid < kGroupClasses) first[tid] = hist[tid] ? atomicAdd(cnt + tid, hist[tid]) : 0u;
  if (tid == 0 && largest) atomicMax(cnt + kGroupClasses, (uint32_t)largest);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kGroupSpan; ++i)
    if (cls[i] >= 0) {
      const int64_t j = ((int64_t)blockIdx.x * kGroupSpan + i) * 256 + tid;
      infos[at + j] = (int32_t)(((first[cls[i]] + num[i]) << 5) | (uint32_t)cls[i]);
    }
}

// Tiles of a group's classes before class c.
__host__ __device__ inline int64_t group_tiles(const uint32_t* cnt, int c) {
  int64_t t = 0;
  for (int i = 0; i < c; ++i) {
    const uint32_t q = (uint32_t)group_per_tile(i);
    t += (cnt[i] + q - 1) / q;
  }
  return t;
}

// Each point's row in the group's tiles (no part has more than kGroupPart
// points); also sets all bits of the rows' records, `words` words.
__global__ __launch_bounds__(256) void k_group_place(int64_t m, const int32_t* __restrict__ parents,
                                                     const int32_t* __restrict__ infos,
                                                     const uint32_t* __restrict__ cnts, int32_t* __restrict__ place,
                                                     uint32_t* __restrict__ rows, int64_t words) {
  __shared__ uint32_t cnt[kGroupClasses];
  __shared__ int32_t tile[kGroupClasses];
  const int g = (int)blockIdx.y;
  const int64_t at = g * m;
  for (int64_t i = ((int64_t)g * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x; i < words;
       i += (int64_t)gridDim.x * gridDim.y * blockDim.x)
    rows[i] = ~0u;
  if (threadIdx.x < kGroupClasses) cnt[threadIdx.x] = cnts[g * kGroupWords + threadIdx.x];
  __syncthreads();
  if (threadIdx.x < kGroupClasses) tile[threadIdx.x] = (int32_t)group_tiles(cnt, threadIdx.x);
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < m; j += stride) {
    const uint32_t inf = (uint32_t)infos[at + parents[at + j]];
    const int c = (int)(inf & 31);
    const uint32_t i = inf >> 5, q = (uint32_t)group_per_tile(c);
    place[at + j] +=
        (tile[c] + (int32_t)(i / q)) * kGroupRows + (int32_t)(i % q) * group_stride(c);
  }
}

// The rows' records: the lattice point, and its neighbours within the tile, a
// byte each (-R .. -1, 1 .. R per direction), the tile's empty row where there
// is none. Rows without a point keep all bits set.
template <int R>
__global__ __launch_bounds__(256) void k_group_rows(const int32_t* __restrict__ nbr, int64_t m, GroupSpec sp,
                                                    const int32_t* __restrict__ places,
                                                    GroupRow<R>* __restrict__ rows) {
  const int g = (int)blockIdx.y;
  const int32_t* place = places + g * m;
  GroupRow<R>* out = rows + sp.tile0[g] * kGroupRows;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < m; j += stride) {
    int32_t nb[kGroupDirs][2 * R];
#pragma unroll
    for (int t = 0; t < kGroupDirs; ++t) {
      if (t < sp.dirs[g]) {
        group_nbrs<R>(nbr, sp.first[g] + t, m, j, nb[t]);
      } else {
#pragma unroll
        for (int i = 0; i < 2 * R; ++i) nb[t][i] = -1;
      }
    }
    GroupRow<R> q;
    q.point = (int32_t)j;
#pragma unroll
    for (int w = 0; w < 2 * R; ++w) {
      uint32_t s = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = 4 * w + i;  // byte e is neighbour e % 2R of direction e / 2R
        const int32_t x = nb[e / (2 * R)][e % (2 * R)];
        s |= (x >= 0 ? (uint32_t)place[x] % kGroupRows : (uint32_t)(kGroupRows - 1)) << (8 * i);
      }
      q.slots[w] = s;
    }
    out[place[j]] = q;
  }
}

}  // namespace
}  // namespace sgp
#endif  // SGP_GROUPS_H
