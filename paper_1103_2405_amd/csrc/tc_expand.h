// The row of every entry of a CSR, for the builder and the gradient.
#pragma once

#include "tc_internal.h"

namespace tc {

namespace {

// Block b writes the rows of entries [b kExpand, (b + 1) kExpand): the row that
// holds the first one by a 64-way search of rp, the rows that start inside
// marked at their first entry in LDS (empty rows share it with the next row:
// the largest id wins), then a running maximum over the block's entries.  Work
// is split by entries, so a hub row costs no more than its entries: 7.6M
// entries of R-MAT 2^18 in 20 us, where one wavefront per 64 rows took 99.
// A block that meets more than kExpandWalk rows to a thread (long runs of empty
// rows) searches the row of each entry instead: one gap of 2^26 empty rows
// walked by its block took the transpose of 2M entries 119 ms, so it takes 0.43.
constexpr int kExpandB = 256, kExpandPer = 8, kExpand = kExpandB * kExpandPer, kExpandWalk = 32;
__global__ void __launch_bounds__(kExpandB) k_rows_of(const int64_t* __restrict__ rp, int64_t n_rows, int64_t nnz,
                                                      int32_t* __restrict__ row_of) {
  __shared__ int32_t mark[kExpand];
  __shared__ int32_t wtop[kExpandB / kWave];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  const int64_t base = (int64_t)blockIdx.x * kExpand, end = base + kExpand < nnz ? base + kExpand : nnz;
#pragma unroll
  for (int u = 0; u < kExpandPer; ++u) mark[u * kExpandB + tid] = 0;
  // last row in [lo, hi) that starts at or before base (rp[0] = 0 <= base)
  int64_t lo = 0, hi = n_rows;
  while (hi - lo > 1) {
    const int64_t step = (hi - lo + kWave - 1) / kWave, q = lo + (int64_t)lane * step;
    const uint64_t m = __ballot(q < hi && rp[q < hi ? q : lo] <= base);
    const int64_t at = lo + (int64_t)(63 - __builtin_clzll(m)) * step;  // lane 0's bit is set
    hi = at + step < hi ? at + step : hi;
    lo = at;
  }
  __syncthreads();
  bool open = true;
  int64_t r = lo + 1 + tid;
  for (int i = 0; i < kExpandWalk && open; ++i, r += kExpandB) {
    const int64_t s = r < n_rows ? rp[r] : end;
    open = s < end;
    if (open) atomicMax(&mark[s - base], (int32_t)r);
  }
  const int64_t e0 = base + (int64_t)tid * kExpandPer;
  int32_t v[kExpandPer];
  if (!__syncthreads_or(open)) {
    int32_t top = (int32_t)lo;
#pragma unroll
    for (int u = 0; u < kExpandPer; ++u) {
      top = max(top, mark[tid * kExpandPer + u]);
      v[u] = top;
    }
    int32_t run = top;  // maximum of this thread's entries and every earlier one of its wavefront
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int32_t t = __shfl_up(run, d, kWave);
      if (lane >= d) run = max(run, t);
    }
    if (lane == kWave - 1) wtop[wv] = run;
    __syncthreads();
    int32_t before = __shfl_up(run, 1, kWave);
    if (lane == 0) before = (int32_t)lo;
    for (int w = 0; w < wv; ++w) before = max(before, wtop[w]);
#pragma unroll
    for (int u = 0; u < kExpandPer; ++u) v[u] = max(v[u], before);
  } else {
    // the last row that starts at or before the entry, of [lo, n_rows)
#pragma unroll
    for (int u = 0; u < kExpandPer; ++u) v[u] = (int32_t)lo;
    for (int64_t len = n_rows - lo; len > 1; len -= len / 2)
#pragma unroll
      for (int u = 0; u < kExpandPer; ++u)
        if (rp[v[u] + len / 2] <= e0 + u) v[u] += (int32_t)(len / 2);
  }
  if (e0 + kExpandPer <= end) {
    *(int4*)(row_of + e0) = make_int4(v[0], v[1], v[2], v[3]);
    *(int4*)(row_of + e0 + 4) = make_int4(v[4], v[5], v[6], v[7]);
  } else {
#pragma unroll
    for (int u = 0; u < kExpandPer; ++u)
      if (e0 + u < end) row_of[e0 + u] = v[u];
  }
}

// row_of (16-byte aligned, like every pool block) for nnz > 0 entries
inline void rows_of(const int64_t* rp, int64_t n_rows, int64_t nnz, int32_t* row_of, hipStream_t st) {
  hipLaunchKernelGGL(k_rows_of, dim3((unsigned)((nnz + kExpand - 1) / kExpand)), dim3(kExpandB), 0, st, rp, n_rows,
                     nnz, row_of);
}

}  // namespace
}  // namespace tc
