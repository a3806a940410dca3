// The tile kernels of the single-vector products and their launches: one
// wavefront per workload slice, every row written through a writer that knows
// what becomes of a row's sum (the product, or an update fused into it).
#pragma once

#include <algorithm>

#include "tc_host.h"

namespace tc {

namespace {

// What a kernel is given to make a writer from: the product itself, ...
struct PlainSpec {
  static constexpr bool kMapped = false;  // x is in internal ids
  using Rest = TileRest;                  // a one-tile product: the launch writes its rest too
  const float* x;
  using X = GlobalX;
  __device__ X make() const { return X{x}; }
};
// ... one tile of several: its chunks' sums are added by a launch after the last
// tile, so they are stored plainly, without the tickets' code and arguments (a
// product of 9 launches over 600K entries: 34.0 -> 32.8 us), ...
struct TileSpec : PlainSpec {
  using Rest = NoRest;
};
// ... the PageRank update (the dangling mass of x in nd <= 64 partial sums), ...
struct PrSpec {
  static constexpr bool kMapped = false;
  using Rest = TileRest;
  const float* x;
  double c;
  const double* dparts;
  int32_t nd;
  int64_t n;
  using X = PrX;
  __device__ X make() const { return X{x, c, wave_parts(dparts, nd) / (double)n, (1.0 - c) / (double)n}; }
};
// ... or the restart of a one-query RWR (seed: an internal id on the device).
struct RwrSpec {
  static constexpr bool kMapped = false;
  using Rest = TileRest;
  const float* x;
  double c;
  const int32_t* seed;
  using X = RwrX;
  __device__ X make() const { return X{x, c, *seed}; }
};

// ... and the product in the caller's ids: row r goes to y[rowinv[r]]; x in
// internal ids, or (MAP) in the caller's, through cperm.
template <bool MAP>
struct UserSpec {
  static constexpr bool kMapped = MAP;
  using Rest = TileRest;
  const float* x;
  const int32_t* cperm;
  const int32_t* rowinv;
  struct X {
    const float* __restrict__ x;
    const int32_t* __restrict__ cperm;
    const int32_t* __restrict__ rowinv;
    __device__ float operator()(int32_t i) const { return MAP ? x[cperm[i]] : x[i]; }
    __device__ void addy(float* y, int32_t rid, double s) const { y[rowinv[rid & ~kAddFlag]] = (float)s; }
  };
  __device__ X make() const { return X{x, cperm, rowinv}; }
};

// S wavefronts per workload of the tile (row slices): wl_blocks blocks of
// them, then blocks for the rows without entries.
constexpr int kEmptyPer = 4;  // rows without entries per thread
template <int S, class Spec>
__global__ void __launch_bounds__(kB) k_tile(const Wl* __restrict__ wl, int64_t n_wl, uint32_t wl_blocks,
                                             const int32_t* __restrict__ idx, const float* __restrict__ val,
                                             const int32_t* __restrict__ rowid, Spec spec, float* __restrict__ y,
                                             double* __restrict__ partial, typename Spec::Rest rest) {
  const int lane = lane_id();
  if constexpr (Spec::Rest::kWhole)
    if (blockIdx.x >= wl_blocks) {
      write_empty(rest, spec.make(), y, (int64_t)(blockIdx.x - wl_blocks) * kB + threadIdx.x,
                  (int64_t)(gridDim.x - wl_blocks) * kB);
      return;
    }
  const int64_t w = (int64_t)blockIdx.x * kWpb + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (w >= n_wl * S) return;
  const Wl d = wl[w / S];
  tile_item<S, false>(d, lane, idx, val, rowid, spec.make(), y, partial, (int32_t)(w % S), rest);
}

// x with its first `hot` columns from cb on in LDS and the others gathered
// through the caches.  Both reads run on every lane without a branch: a lane
// whose column is staged gives its buffer load an offset past the buffer,
// which returns 0 and makes no request, and the others read LDS word 0.
// ALL: every column of the tile is staged.
template <class X, bool ALL>
struct HotX {
  X b;
  const float* xs;
  int32_t cb, hot;
  __amdgpu_buffer_rsrc_t r;  // x, limited to its 4 n_cols bytes
  __device__ float operator()(int32_t i) const {
    const uint32_t k = (uint32_t)(i - cb);
    if constexpr (ALL) return xs[k];
    const bool in = k < (uint32_t)hot;
    const float l = xs[in ? k : 0];
    const float g = __builtin_bit_cast(
        float, __builtin_amdgcn_raw_buffer_load_b32(r, in ? (int32_t)0x80000000 : i * 4, 0, 0));
    return in ? l : g;
  }
  __device__ void addy(float* y, int32_t rid, double s) const { b.addy(y, rid, s); }
};

// Tile pass with the tile's hottest columns staged in LDS.  Columns are sorted
// by length, so the first `hot` of a tile carry a large share of its entries
// (the first 40K of a 2^20-node R-MAT graph: 73%), and a gather that LDS
// serves is no L2 request; the requests bound k_tile (205 G/s on that graph,
// the rate of the random-gather measurement within one L2).  One workgroup of
// 16 wavefronts per compute unit, since the staging takes its LDS.  Its items
// (workload slices, slice-major: equal slices of every workload) are
// blockIdx.x + k gridDim.x, handed to the wavefronts by an LDS counter.
// Measured, k_tile -> this, us per product: R-MAT 2^20 symmetrised (31.4M
// entries) 155 -> 101, its PageRank matrix (16.1M) 96 -> 65, its HITS matrix
// (32.2M) 171 -> 116; 2^18 symmetrised (7.6M) 40 -> 27.5; Chung-Lu 2^22 (59M)
// 408 -> 370; uniform 2^20 x 16 117 -> 113.  What is left on the first: 10.6M
// L2 read requests (23.5M before) at 130 G/s, and a tenth between the XCDs.
constexpr int kHotB = 1024;
template <int S, bool ALL, class Spec>
__global__ void __launch_bounds__(kHotB) k_tile_hot(const Wl* __restrict__ wl, uint32_t n_wl,
                                                    const int32_t* __restrict__ idx, const float* __restrict__ val,
                                                    const int32_t* __restrict__ rowid, Spec spec, int32_t n_cols,
                                                    int32_t cb, int32_t hot, float* __restrict__ y,
                                                    double* __restrict__ partial, typename Spec::Rest rest) {
  extern __shared__ float xs[];  // the staged columns, then the item counter
  uint32_t* ctr = (uint32_t*)(xs + hot);
  if (threadIdx.x == 0) *ctr = 0;
  stage_x<kHotB>(xs, spec.x + cb, hot);
  __syncthreads();
  const int lane = lane_id();
  const HotX<typename Spec::X, ALL> xg{
      spec.make(), xs, cb, hot,
      __builtin_amdgcn_make_buffer_rsrc((void*)spec.x, (short)0, n_cols * 4, 0x00020000)};
  if constexpr (Spec::Rest::kWhole)
    write_empty(rest, xg, y, (int64_t)blockIdx.x * kHotB + threadIdx.x, (int64_t)gridDim.x * kHotB);
  const uint32_t items = n_wl * S, G = gridDim.x;
  auto take = [&]() -> uint32_t {
    uint32_t k = 0;
    if (lane == 0) k = atomicAdd(ctr, 1u);
    return blockIdx.x + (uint32_t)__builtin_amdgcn_readfirstlane(k) * G;
  };
  uint32_t w = take();
  if (w >= items) return;
  Wl d = wl[w % n_wl];
  for (;;) {  // the next item and its descriptor are read while the current one runs
    const uint32_t wn = take();
    const Wl dn = wl[(wn < items ? wn : w) % n_wl];
    tile_item<S, true>(d, lane, idx, val, rowid, xg, y, partial, (int32_t)(w / n_wl), rest);
    if (wn >= items) break;
    d = dn;
    w = wn;
  }
}

// The split rows of a one-tile product whose tile launch draws no tickets, one
// wavefront a row: the chunk sums added left to right (the bits of the tickets').
template <class Spec>
__global__ void __launch_bounds__(kB) k_tile_splits(const SplitRow* __restrict__ split, int64_t n,
                                                    const double* __restrict__ partial, Spec spec,
                                                    float* __restrict__ y) {
  const int lane = lane_id();
  const int64_t i = (int64_t)blockIdx.x * kWpb + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (i >= n) return;
  __shared__ double buf[kWpb][4 * kWave];
  const SplitRow s = split[i];
  const auto x = spec.make();
  const double acc = sum_slots_wave(partial + s.slot_begin, s.n_slots, lane, buf[threadIdx.x / kWave]);
  if (lane == 0) x.addy(y, s.row, acc);
}

// Columns of tile t that k_tile_hot stages, or 0 for k_tile.  Measured k_tile /
// k_tile_hot, R-MAT (r), Chung-Lu (c), uniform (u) and mildly skewed columns
// (share of the entries in the 40896 columns: r .99-.56, c .90-.50, u .57-.02):
//  - Below 3M entries the staging (up to 160 KB into every compute unit, 3.4 us)
//    does not pay: 0.68-1.15 at 1-2M; 1.00-1.54 at 3.1-9M on r and c, u below.
//  - What LDS serves has to make up for gathers of the other columns by half as
//    many wavefronts, and the more floats x has, the farther away they are.  With
//    at least half as many entries in the staged columns as the tile has columns
//    0.98-1.67, most of it 1.05 and more; with fewer 0.87-0.99 (u, 2^22 columns,
//    4-16M entries: 0.90-0.92; 2.3M columns, 4-16M: 0.92-0.97; 2^20, 4M: 0.97)
//    and 1.02-1.04 at most (u, 1.6M columns, 16M entries).
//  - A row that one wavefront sums alone takes 7.5 ns an entry here and 4.2 in
//    k_tile: past a 2048th of the entries (the automatic split length is an
//    8192th) it lasts as long as the whole pass, and unsplit hubs set the time
//    (c 2^20, 14.7M entries, split_len 0: 533 us with k_tile, 966 here).
//  - A tile that fits is staged whole also with 8 entries per float staged in
//    every compute unit.
// The build option lds_stage = 1 stages every tile that fits, and the others by
// the same rule; -1 none.  x must fit the buffer load's 32-bit offsets.
constexpr int64_t kHotMinReuse = 8;
inline int64_t hot_width(const tc_handle* h, int t, int64_t items) {
  if (!h->lds_tiles || h->n_cols >= kBufMaxFloats || items >= ((int64_t)1 << 31)) return 0;
  const int64_t width = h->tile_col_end[t] - h->tile_col_begin[t], nnz = h->tile_nnz[t];
  const bool fits = width <= h->lds_floats;
  const int64_t stage = std::max<int64_t>(0, std::min(h->hot_room(), width));
  if (fits && (h->lds_tiles == 2 || nnz >= kHotMinReuse * width * h->n_cu)) return stage;
  if (nnz < kHotMinNnz || kRowShare * h->tile_long[t] > nnz || 2 * h->tile_hot_nnz[t] < width) return 0;
  return stage;
}

inline bool one_tile(const tc_handle* h) { return h->n_tiles == 1 && h->n_panels == 0 && h->kernel == 0; }
// The rest of a one-tile product (empty: its rows without entries too).
inline TileRest tile_rest(const tc_handle* h, bool empty) {
  return TileRest{h->d_empty, empty ? h->n_empty : 0, h->d_split, h->d_slot_split, h->tickets ? h->d_ticket : nullptr};
}

// The launch of tile t's kernel.
template <class Spec>
void launch_rows(tc_handle* h, int t, int64_t b, int64_t n, const Spec& sp, float* y, hipStream_t st,
                 const typename Spec::Rest& rest) {
  const int32_t S = tile_slices(h, t, n);
  if constexpr (!Spec::kMapped) {  // staging takes x in internal ids
    const int64_t hot = n > 0 ? hot_width(h, t, n * S) : 0;
    if (hot > 0) {
      auto kern = hot == h->tile_col_end[t] - h->tile_col_begin[t]
                      ? pick_slices(S, k_tile_hot<1, true, Spec>, k_tile_hot<2, true, Spec>, k_tile_hot<4, true, Spec>,
                                    k_tile_hot<8, true, Spec>)
                      : pick_slices(S, k_tile_hot<1, false, Spec>, k_tile_hot<2, false, Spec>,
                                    k_tile_hot<4, false, Spec>, k_tile_hot<8, false, Spec>);
      const uint32_t lds = (uint32_t)(4 * (hot + 1));
      if (lds > 65536) HIPC(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
      // one item per compute unit before a second one on any (7.3M entries in 891
      // workloads of 8192: 37 us; 67 where 56 workgroups take sixteen each, 41 in k_tile)
      const unsigned grid = (unsigned)std::min<int64_t>(h->n_cu, n * S);
      launch_tile(h, kern, dim3(grid), dim3(kHotB), lds, st, (const Wl*)(h->d_wl + b), (uint32_t)n,
                  (const int32_t*)h->d_idx, (const float*)h->d_val, (const int32_t*)h->d_rowid, sp, (int32_t)h->n_cols,
                  (int32_t)h->tile_col_begin[t], (int32_t)hot, y, h->d_partial, rest);
      return;
    }
  }
  const unsigned wb = nblk(n * S, kWpb), eb = nblk(rest.n_empty, kB * kEmptyPer);
  launch_tile(h, pick_slices(S, k_tile<1, Spec>, k_tile<2, Spec>, k_tile<4, Spec>, k_tile<8, Spec>), dim3(wb + eb),
              dim3(kB), 0, st, (const Wl*)(h->d_wl + b), n, wb, (const int32_t*)h->d_idx, (const float*)h->d_val,
              (const int32_t*)h->d_rowid, sp, y, h->d_partial, rest);
}

// y's rows of tile t, and the rest, through the writer of `sp`.
template <class Spec>
void run_tile(tc_handle* h, int t, const Spec& sp, float* y, hipStream_t st, const typename Spec::Rest& rest) {
  const int64_t b = h->tile_wl_begin[t], n = h->tile_wl_begin[t + 1] - b;
  if (n == 0 && rest.n_empty == 0) return;
  launch_rows(h, t, b, n, sp, y, st, rest);
  if constexpr (Spec::Rest::kWhole)
    if (!rest.ticket && h->n_split_rows > 0) {
      hipLaunchKernelGGL(k_tile_splits<Spec>, dim3(nblk(h->n_split_rows, kWpb)), dim3(kB), 0, st,
                         (const SplitRow*)h->d_split, h->n_split_rows, (const double*)h->d_partial, sp, y);
      HIPC(hipGetLastError());
    }
}

}  // namespace
}  // namespace tc
