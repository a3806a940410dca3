// Device-side building blocks shared by the library's product kernels: the
// tile pass over one workload (Section 3.1, Solution 3), wavefront sums, the
// sum of a split row's partial slots and a few small vector kernels.
//
// Tile pass: one wavefront per workload (or per row slice of a workload).
//   row-major:    the wavefront walks one row at a time, lanes striding the
//                 padded row, then a cross-lane sum; the last lane updates y.
//   column-major: lane r owns row r of the rectangle and walks its columns;
//                 consecutive lanes read consecutive addresses.
//   chunk:        one piece of a split heavy row; its sum goes to a partial
//                 slot that is added to y after the last tile.
// Products are exact in FP64 and each row's per-tile sum is accumulated in
// FP64, then added to the FP32 y once per tile.
#pragma once

#include "tc_internal.h"

namespace tc {

// RWR restart fused into the product (one tile: each row's value is final
// where it is written): R'[row][q] = fl32(c fl32(y) + (1 - c) [row == seed_q]),
// the same rounding as the separate update after a stored y.
struct RwrEpi {
  double c;
  const int32_t* seeds;  // internal ids, one per right-hand side
};

// PageRank update fused into the row-panel pass (Eq. 6): every row is
// written as p' = fl32(c (fl32(y) + d/n) + (1 - c)/n), the separate update's
// rounding; a split row's sum over its unsplit segments also goes to yraw (in
// the order of the split-row list), for the pass that adds its chunks.
struct PanelPr {
  double c;
  const double* dparts;   // partial sums of the dangling mass of the iterate the product reads
  int32_t nd;             // (at most 64)
  int64_t n;
  const int64_t* psb;     // [panels + 1] split rows of each panel
  const SplitRow* split;  // split rows, increasing row
  float* yraw;
};

__device__ inline float rwr_restart(double c, float y, bool is_seed) {
  return (float)(c * (double)y + (is_seed ? 1.0 - c : 0.0));
}

namespace {

constexpr int kB = 256;
constexpr int kWpb = kB / kWave;  // workloads per block

inline unsigned nblk(int64_t n, int64_t per) { return (unsigned)((n + per - 1) / per); }

__device__ inline int lane_id() { return (int)__lane_id(); }

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, kWave);
  return v;
}

__device__ inline void add_to_y(float* y, int32_t row, double s) { y[row] = (float)((double)y[row] + s); }

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
// the same where only the elements are aligned (row ids; the hardware needs 4 bytes)
typedef int v4iu __attribute__((ext_vector_type(4), aligned(4)));
typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));
typedef int v2iu __attribute__((ext_vector_type(2), aligned(4)));

// Streams of the matrix are read once per product: non-temporal loads keep
// them from evicting x and y from the caches.
__device__ inline int32_t ld_nt(const int32_t* p) { return __builtin_nontemporal_load(p); }
__device__ inline float ld_nt(const float* p) { return __builtin_nontemporal_load(p); }
__device__ inline v4i ld_nt4(const int32_t* p) { return __builtin_nontemporal_load((const v4i*)p); }
__device__ inline v4f ld_nt4(const float* p) { return __builtin_nontemporal_load((const v4f*)p); }

// x[i] by a raw buffer load: a 32-bit byte offset from one scalar base, so a
// gather needs no 64-bit address per lane (about 1% faster on the panel
// pass).  Same value and cache policy as x[i]; x must hold at most
// kBufMaxFloats floats, so that 4 i fits the signed offset.  The descriptor
// covers the whole 32-bit range (no record limit); its word 3 is the CDNA
// raw-dword format.
constexpr int64_t kBufMaxFloats = (int64_t)1 << 29;
__device__ inline float ld_buf(const float* x, int32_t i) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)x, (short)0, -1, 0x00020000);
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, i * 4, 0, 0));
}

// Cross-lane moves of a double through DPP (two 32-bit halves).  Lanes whose
// source is outside the row read 0 (bound_ctrl), rows outside ROWMASK add 0.
template <int CTRL, int ROWMASK = 0xf>
__device__ inline double dpp_f64(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  const int l2 = __builtin_amdgcn_update_dpp(0, lo, CTRL, ROWMASK, 0xf, true);
  const int h2 = __builtin_amdgcn_update_dpp(0, hi, CTRL, ROWMASK, 0xf, true);
  return __hiloint2double(h2, l2);
}

// Sum over each 8-lane half of a DPP row; the totals land in lanes 7 and 15
// of the row (the first three steps of the row's running sum).
__device__ inline double row8_sum(double v) {
  v += dpp_f64<0x111>(v);  // row_shr:1
  v += dpp_f64<0x112>(v);  // row_shr:2
  v += dpp_f64<0x114>(v);  // row_shr:4
  return v;
}
// Sum over each DPP row of 16 lanes; the total lands in the row's lane 15.
__device__ inline double row16_sum(double v) {
  v = row8_sum(v);
  v += dpp_f64<0x118>(v);  // row_shr:8
  return v;
}
// ... over 32 lanes (total in lanes 31 and 63)
__device__ inline double row32_sum(double v) {
  v = row16_sum(v);
  return v + dpp_f64<0x142, 0xa>(v);
}
// ... over the wavefront (total in lane 63)
__device__ inline double wave_total(double v) {
  v = row16_sum(v);
  v += dpp_f64<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp_f64<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}

// Copies n floats of x into LDS by the B threads of a workgroup, eight 16-byte
// loads in flight per thread, then two (a plain loop would wait for each load
// before the next).  xs is 16-byte aligned; past n nothing is read.
template <int B>
__device__ inline void stage_x(float* xs, const float* __restrict__ x, int32_t n) {
  const int32_t n4 = ((uintptr_t)x & 15) == 0 ? n & ~3 : 0, t4 = 4 * (int32_t)threadIdx.x;
  int32_t k = 0;
  for (; k + 32 * B <= n4; k += 32 * B) {
    v4f t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = *(const v4f*)(x + k + 4 * B * u + t4);
#pragma unroll
    for (int u = 0; u < 8; ++u) *(v4f*)(xs + k + 4 * B * u + t4) = t[u];
  }
  for (; k < n4; k += 8 * B) {
    const int32_t a = k + t4, b = a + 4 * B;
    const v4f ta = *(const v4f*)(x + (a < n4 ? a : 0)), tb = *(const v4f*)(x + (b < n4 ? b : 0));
    if (a < n4) *(v4f*)(xs + a) = ta;
    if (b < n4) *(v4f*)(xs + b) = tb;
  }
  for (int32_t q = n4 + (int32_t)threadIdx.x; q < n; q += B) xs[q] = x[q];
}

template <class G>
__device__ inline double dot4(v4i i, v4f v, const G& xg) {
  const float x0 = xg(i.x), x1 = xg(i.y), x2 = xg(i.z), x3 = xg(i.w);
  double s = (double)v.x * (double)x0;
  s = fma((double)v.y, (double)x1, s);
  s = fma((double)v.z, (double)x2, s);
  return fma((double)v.w, (double)x3, s);
}

// A chunk's sum into its partial slot; SAME: read in the same kernel, possibly
// on another XCD (finish_chunk), so written through to where that reads it.
template <bool SAME>
__device__ inline void put_partial(double* partial, int32_t slot, double v) {
  if constexpr (SAME)
    __hip_atomic_store(partial + slot, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    partial[slot] = v;
}

// Row-major rectangle with 64-element-aligned rows (S a multiple of 64), or
// rows padded to 32: every lane reads 4 consecutive entries (16 bytes) per
// 256-entry chunk.
//   w_pad = 32:  a chunk holds 8 rows, 8 lanes each -> sums per half DPP row
//   w_pad = 64:  a chunk holds 4 rows, 16 lanes each -> sums per DPP row
//   w_pad = 128: a chunk holds 2 rows, 32 lanes each
//   otherwise:   one row at a time, chunks of 256 (last one masked)
// Two chunks are in flight per iteration (8 gathers per lane).
template <int S, bool SAME, class G>
__device__ inline void rm_wide(const Wl& d, int lane, const int32_t* __restrict__ idx,
                               const float* __restrict__ val, const int32_t* __restrict__ rowid,
                               const G& x, float* __restrict__ y, double* __restrict__ partial,
                               bool chunk, int32_t sl) {
  const int64_t off = d.data_off;
  const int32_t wp = d.w_pad, nr = d.n_rows;
  if (wp == 32 || wp == 64 || wp == 128) {
    const int lpr = wp >> 2;             // lanes per row
    const int rpc = kWave / lpr;         // rows per chunk
    const int my = lane / lpr;           // my row inside the chunk
    const int nchunk = (nr + rpc - 1) / rpc;
    for (int q = 2 * sl; q < nchunk; q += 2 * S) {
      const int ra = q * rpc + my, rb = (q + 1) * rpc + my;
      const bool oka = ra < nr, okb = rb < nr;
      // row ids read with the matrix loads (clamped to a valid entry; chunks have none to write)
      const int32_t ida = chunk ? 0 : ld_nt(rowid + d.rowid_off + (oka ? ra : 0));
      const int32_t idb = chunk ? 0 : ld_nt(rowid + d.rowid_off + (okb ? rb : 0));
      double sa = 0.0, sb = 0.0;
      v4i ia, ib;
      v4f va, vb;
      if (oka) {
        ia = ld_nt4(idx + off + (int64_t)q * 256 + 4 * lane);
        va = ld_nt4(val + off + (int64_t)q * 256 + 4 * lane);
      }
      if (okb) {
        ib = ld_nt4(idx + off + (int64_t)(q + 1) * 256 + 4 * lane);
        vb = ld_nt4(val + off + (int64_t)(q + 1) * 256 + 4 * lane);
      }
      if (oka) sa = dot4(ia, va, x);
      if (okb) sb = dot4(ib, vb, x);
      if (wp == 32) {
        sa = row8_sum(sa);
        sb = row8_sum(sb);
      } else if (wp == 64) {
        sa = row16_sum(sa);
        sb = row16_sum(sb);
      } else {
        sa = row32_sum(sa);
        sb = row32_sum(sb);
      }
      if ((lane % lpr) == lpr - 1) {
        if (chunk) {
          if (oka) put_partial<SAME>(partial, d.info >> 2, sa);
        } else {
          if (oka) x.addy(y, ida, sa);
          if (okb) x.addy(y, idb, sb);
        }
      }
    }
    return;
  }
  for (int32_t r = sl; r < nr; r += S) {
    const int64_t base = off + (int64_t)r * wp;
    const int32_t idr = chunk ? 0 : ld_nt(rowid + d.rowid_off + r);
    double acc = 0.0;
    int32_t c = 4 * lane;
    for (; c + 256 < wp; c += 512) {
      const v4i ia = ld_nt4(idx + base + c), ib = ld_nt4(idx + base + c + 256);
      const v4f va = ld_nt4(val + base + c), vb = ld_nt4(val + base + c + 256);
      acc += dot4(ia, va, x) + dot4(ib, vb, x);
    }
    if (c < wp) acc += dot4(ld_nt4(idx + base + c), ld_nt4(val + base + c), x);
    acc = wave_total(acc);
    if (lane == kWave - 1) {
      if (chunk)
        put_partial<SAME>(partial, d.info >> 2, acc);
      else
        x.addy(y, idr, acc);
    }
  }
}

// Column-major rectangle: lane owns rows r = 64 u + lane; U row blocks and C
// columns are in flight together (U * C independent gathers per lane).  Every
// load runs on every lane: a lane past the last row reads the workload's first
// entry and takes index 0 and value 0 instead (its sum is never stored).  A
// load under a per-lane branch would end its branch with a wait for it, so
// the loads would go out one at a time.
template <int U, int C, int S, class G>
__device__ inline void cm_rows(const Wl& d, int lane, const int32_t* __restrict__ idx,
                               const float* __restrict__ val, const int32_t* __restrict__ rowid,
                               const G& x, float* __restrict__ y, int32_t sl) {
  const int64_t off = d.data_off, hp = d.h_pad;
  const int32_t w = d.w_pad, nr = d.n_rows;
  // slice sl of S takes the 64-row blocks sl, sl + S, ..., U of them at a time
  for (int32_t r0 = sl * kWave; r0 < nr; r0 += U * S * kWave) {
    double acc[U];
    bool ok[U];
    int32_t rid[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc[u] = 0.0;
      ok[u] = r0 + u * S * kWave + lane < nr;
    }
    // the rows' ids go out with the first matrix loads (a lane past the last
    // row reads the workload's first id and never uses it)
#pragma unroll
    for (int u = 0; u < U; ++u) rid[u] = ld_nt(rowid + d.rowid_off + (ok[u] ? r0 + u * S * kWave + lane : 0));
    int32_t c = 0;
    for (; c + C <= w; c += C) {
      int32_t ii[U][C];
      float vv[U][C], xv[U][C];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < C; ++k) {
          const int64_t e = ok[u] ? off + (int64_t)(c + k) * hp + r0 + u * S * kWave + lane : off;
          const int32_t ti = ld_nt(idx + e);
          const float tv = ld_nt(val + e);
          ii[u][k] = ok[u] ? ti : 0;
          vv[u][k] = ok[u] ? tv : 0.0f;
        }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < C; ++k) xv[u][k] = x(ii[u][k]);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < C; ++k) acc[u] = fma((double)vv[u][k], (double)xv[u][k], acc[u]);
    }
    for (; c < w; ++c) {
      int32_t ii[U];
      float vv[U], xv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t e = ok[u] ? off + (int64_t)c * hp + r0 + u * S * kWave + lane : off;
        const int32_t ti = ld_nt(idx + e);
        const float tv = ld_nt(val + e);
        ii[u] = ok[u] ? ti : 0;
        vv[u] = ok[u] ? tv : 0.0f;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) xv[u] = x(ii[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) acc[u] = fma((double)vv[u], (double)xv[u], acc[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (ok[u]) x.addy(y, rid[u], acc[u]);
  }
}

// V consecutive entries of a stream, read once (16, 8 or 4 bytes).
template <int V>
struct Pack {
  int32_t i[V];
  float v[V];
};
template <int V>
__device__ inline Pack<V> ld_pack(const int32_t* __restrict__ idx, const float* __restrict__ val, uint32_t e) {
  Pack<V> p;
  if constexpr (V == 4) {
    const v4i a = ld_nt4(idx + e);
    const v4f b = ld_nt4(val + e);
    p.i[0] = a.x, p.i[1] = a.y, p.i[2] = a.z, p.i[3] = a.w;
    p.v[0] = b.x, p.v[1] = b.y, p.v[2] = b.z, p.v[3] = b.w;
  } else if constexpr (V == 2) {
    const v2i a = __builtin_nontemporal_load((const v2i*)(idx + e));
    const v2f b = __builtin_nontemporal_load((const v2f*)(val + e));
    p.i[0] = a.x, p.i[1] = a.y;
    p.v[0] = b.x, p.v[1] = b.y;
  } else {
    p.i[0] = ld_nt(idx + e);
    p.v[0] = ld_nt(val + e);
  }
  return p;
}

// Column-major rectangle by wide loads: a lane owns V consecutive rows of each
// group of 64 V rows, so one load per stream serves V entries where cm_rows
// issues one per entry; U groups and C columns are in flight together (U V C
// independent gathers per lane).  Each row is summed by one lane in column
// order, so the bits are cm_rows'.  For the staged tile kernel, which runs 16
// wavefronts per compute unit: 104 us against 117 on a 31M-entry power-law
// matrix.  With 32 of them (k_tile) it measured slower, 421 against 408 us on
// 59M entries, and so did the panel pass's small workloads (a whole product on
// 118M entries 736 against 730 us).
// As in cm_rows, every load runs on every lane: a lane past the stored rows
// reads the workload's first entry, and pad rows hold zeros; neither is stored.
template <int V, int U, int C, int S, class G>
__device__ inline void cm_vec(const Wl& d, int lane, const int32_t* __restrict__ idx0,
                               const float* __restrict__ val0, const int32_t* __restrict__ rowid0,
                               const G& x, float* __restrict__ y, int32_t sl) {
  const int32_t* idx = idx0 + d.data_off;
  const float* val = val0 + d.data_off;
  const int32_t* rowid = rowid0 + d.rowid_off;
  const uint32_t hp = (uint32_t)d.h_pad;
  const int32_t w = d.w_pad, nr = d.n_rows;
  // slice sl of S takes the groups sl, sl + S, ..., U of them at a time
  for (int32_t r0 = sl * (kWave * V); r0 < nr; r0 += U * S * (kWave * V)) {
    double acc[U][V];
    uint32_t e[U], es[U];
    int32_t rid[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t r = (uint32_t)(r0 + u * S * (kWave * V) + lane * V);
      const bool in = r < hp;
      e[u] = in ? r : 0;
      es[u] = in ? hp : 0;
      // the rows' ids go out with the first matrix loads
      if constexpr (V == 4) {
        const v4iu t = __builtin_nontemporal_load((const v4iu*)(rowid + e[u]));
        rid[u][0] = t.x, rid[u][1] = t.y, rid[u][2] = t.z, rid[u][3] = t.w;
      } else if constexpr (V == 2) {
        const v2iu t = __builtin_nontemporal_load((const v2iu*)(rowid + e[u]));
        rid[u][0] = t.x, rid[u][1] = t.y;
      } else {
        rid[u][0] = ld_nt(rowid + e[u]);
      }
#pragma unroll
      for (int v = 0; v < V; ++v) acc[u][v] = 0.0;
    }
    int32_t c = 0;
    for (; c + C <= w; c += C) {
      Pack<V> m[U][C];
      float xv[U][C][V];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < C; ++k) {
          m[u][k] = ld_pack<V>(idx, val, e[u]);
          e[u] += es[u];
        }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < C; ++k)
#pragma unroll
          for (int v = 0; v < V; ++v) xv[u][k][v] = x(m[u][k].i[v]);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < C; ++k)
#pragma unroll
          for (int v = 0; v < V; ++v) acc[u][v] = fma((double)m[u][k].v[v], (double)xv[u][k][v], acc[u][v]);
    }
    if constexpr (C > 1) {
      for (; c < w; ++c) {
        Pack<V> m[U];
        float xv[U][V];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          m[u] = ld_pack<V>(idx, val, e[u]);
          e[u] += es[u];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int v = 0; v < V; ++v) xv[u][v] = x(m[u].i[v]);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int v = 0; v < V; ++v) acc[u][v] = fma((double)m[u].v[v], (double)xv[u][v], acc[u][v]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int v = 0; v < V; ++v)
        if (r0 + u * S * (kWave * V) + lane * V + v < nr) x.addy(y, rid[u][v], acc[u][v]);
  }
}

// Any layout, any padding (used when the rectangle is not 64-aligned).
template <int S, bool SAME, class G>
__device__ inline void generic_wl(const Wl& d, int lane, int layout, const int32_t* __restrict__ idx,
                                  const float* __restrict__ val, const int32_t* __restrict__ rowid,
                                  const G& x, float* __restrict__ y, double* __restrict__ partial,
                                  int32_t sl) {
  if (layout == kCM) {
    const int64_t hp = d.h_pad;
    for (int32_t r = sl * kWave + lane; r < d.n_rows; r += kWave * S) {
      double acc = 0.0;
      for (int32_t c = 0; c < d.w_pad; ++c) {
        const int64_t e = d.data_off + (int64_t)c * hp + r;
        acc = fma((double)val[e], (double)x(idx[e]), acc);
      }
      x.addy(y, rowid[d.rowid_off + r], acc);
    }
    return;
  }
  const int64_t wp = d.w_pad;
  for (int32_t r = sl; r < d.n_rows; r += S) {
    const int64_t base = d.data_off + r * wp;
    double acc = 0.0;
    for (int64_t c = lane; c < wp; c += kWave) acc = fma((double)val[base + c], (double)x(idx[base + c]), acc);
    acc = wave_total(acc);
    if (lane == kWave - 1) {
      if (layout == kChunk)
        put_partial<SAME>(partial, d.info >> 2, acc);
      else
        x.addy(y, rowid[d.rowid_off + r], acc);
    }
  }
}

// y update of one row by a tile: the row's first writer stores fl32(s); a
// later tile (kAddFlag in the row id) stores fl32(y + s).
__device__ inline void addy_first_touch(float* y, int32_t rid, double s) {
  if (rid & kAddFlag) {
    const int32_t row = rid & ~kAddFlag;
    y[row] = (float)((double)y[row] + s);
  } else {
    y[rid] = (float)s;
  }
}

// x as read by a tile: straight from global memory (through L1/L2) ...
struct GlobalX {
  const float* __restrict__ x;
  __device__ float operator()(int32_t i) const { return x[i]; }
  __device__ void addy(float* y, int32_t row, double s) const { addy_first_touch(y, row, s); }
};

// ... or with the PageRank update fused into the row writes (one tile: each
// row's value is final where it is written):
//   p'[row] = fl32(c (fl32(s) + d/n) + (1 - c)/n),
// the rounding of the separate update after a stored y.
struct PrX {
  const float* __restrict__ x;
  double c, dn, tele;
  __device__ float operator()(int32_t i) const { return x[i]; }
  __device__ void addy(float* y, int32_t rid, double s) const {
    y[rid & ~kAddFlag] = (float)(c * ((double)(float)s + dn) + tele);
  }
};

// ... or with the RWR restart of one query fused in (one tile):
//   r'[row] = fl32(c fl32(s) + (1 - c) [row == seed]),
// the rounding of the separate update after a stored y.
struct RwrX {
  const float* __restrict__ x;
  double c;
  int32_t seed;
  __device__ float operator()(int32_t i) const { return x[i]; }
  __device__ void addy(float* y, int32_t rid, double s) const {
    const int32_t row = rid & ~kAddFlag;
    y[row] = (float)(c * (double)(float)s + (row == seed ? 1.0 - c : 0.0));
  }
};

// ... or writing a private copy of y: every row of a tile is written once,
// so the copy is stored whatever the first-writer flag says.
struct PrivX {
  const float* __restrict__ x;
  __device__ float operator()(int32_t i) const { return x[i]; }
  __device__ void addy(float* y, int32_t rid, double s) const { y[rid & ~kAddFlag] = (float)s; }
};

// VEC: column-major rectangles by wide loads (cm_vec), whose 32-bit offsets
// need an area below kVecMaxArea; larger or unaligned ones go the other way.
constexpr int64_t kVecMaxArea = (int64_t)1 << 29;
template <int S = 1, bool VEC = false, bool SAME = false, class G>
__device__ __attribute__((always_inline)) inline void run_workload(const Wl& d, int lane, const int32_t* __restrict__ idx,
                                    const float* __restrict__ val, const int32_t* __restrict__ rowid, const G& x,
                                    float* __restrict__ y, double* __restrict__ partial, int32_t sl = 0) {
  const int layout = d.info & 3;
  const bool aligned = (d.data_off & 3) == 0;
  if (VEC && layout == kCM && (d.h_pad & 63) == 0 && aligned && (int64_t)d.w_pad * d.h_pad < kVecMaxArea) {
    // 64-row blocks per slice (every slice of a workload has to choose alike)
    const int32_t blocks = (d.n_rows + kWave * S - 1) / (kWave * S);
    if (blocks > 4)
      cm_vec<4, 2, 1, S>(d, lane, idx, val, rowid, x, y, sl);
    else if (blocks > 2)
      cm_vec<4, 1, 2, S>(d, lane, idx, val, rowid, x, y, sl);
    else if (blocks > 1)
      cm_vec<2, 1, 4, S>(d, lane, idx, val, rowid, x, y, sl);
    else
      cm_vec<1, 1, 8, S>(d, lane, idx, val, rowid, x, y, sl);
  } else if (layout == kCM && (d.h_pad & 63) == 0) {
    // row blocks of this slice
    const int32_t blocks = ((d.n_rows + kWave - 1) / kWave - sl + S - 1) / S;
    if (blocks >= 8)
      cm_rows<8, 1, S>(d, lane, idx, val, rowid, x, y, sl);
    else if (blocks >= 4)
      cm_rows<4, 2, S>(d, lane, idx, val, rowid, x, y, sl);
    else if (blocks >= 2)
      cm_rows<2, 4, S>(d, lane, idx, val, rowid, x, y, sl);
    else
      cm_rows<1, 8, S>(d, lane, idx, val, rowid, x, y, sl);
  } else if (layout != kCM && aligned && ((d.w_pad & 63) == 0 || (d.w_pad == 32 && layout == kRM))) {
    rm_wide<S, SAME>(d, lane, idx, val, rowid, x, y, partial, layout == kChunk, sl);
  } else {
    generic_wl<S, SAME>(d, lane, layout, idx, val, rowid, x, y, partial, sl);
  }
}

// What a one-tile product writes besides its workloads' rows: the rows
// without entries, and the split rows' sums, each by the wavefront that
// finishes the row's last chunk (ticket[i] counts split row i's finished
// chunks modulo their number).
struct TileRest {
  static constexpr bool kWhole = true;
  const int32_t* empty;
  int64_t n_empty;
  const SplitRow* split;
  const int32_t* slot_split;  // partial slot -> split row
  uint32_t* ticket;           // null: another launch adds the chunk sums
};
// ... or nothing: one tile of several, whose chunk sums another launch adds
struct NoRest {
  static constexpr bool kWhole = false;
  static constexpr int64_t n_empty = 0;
};

// After a chunk's sum is in its slot: the wavefront of the row's last chunk
// adds the slots left to right from 0.0 (the bits of sum_slots) and writes the
// row.  The slots travel by agent-scope accesses, which pass the XCD's L2:
// the wait makes this wavefront's slot complete there before its ticket is
// drawn, so the last ticket's wavefront reads every slot.  No fence (an
// agent-scope release would write back the whole L2) and no wavefront waits
// for another.  The ticket counts modulo the row's chunks, so any whole number
// of products, also ones that overlapped on the handle against its contract,
// leaves it at 0 for the next (a reset by the last wavefront would lose what
// another product counted meanwhile, and finish the row early ever after).
// (i, sr: the chunk's split row, read before the chunk is summed.)
template <class X>
__device__ inline void finish_chunk(int32_t i, const SplitRow& sr, int lane, const X& x, float* __restrict__ y,
                                    const double* partial, const TileRest& rest) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  const uint32_t last = (uint32_t)sr.n_slots - 1;
  uint32_t t = 0;
  if (lane == 0) t = atomicInc(rest.ticket + i, last);  // relaxed, agent scope
  if (__builtin_amdgcn_readfirstlane(t) != last) return;
  asm volatile("" ::: "memory");
  double acc = 0.0;
  for (int32_t q = 0; q < sr.n_slots; q += kWave) {
    const double v = q + lane < sr.n_slots ? __hip_atomic_load(partial + sr.slot_begin + q + lane, __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT)
                                           : 0.0;
    const int m = min(kWave, sr.n_slots - q);
    for (int k = 0; k < m; ++k)
      acc += __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), k),
                              __builtin_amdgcn_readlane(__double2loint(v), k));
  }
  if (lane == 0) x.addy(y, sr.row, acc);
}

// A workload slice; the chunks of a one-tile product draw their tickets
template <int S, bool VEC, class X, class Rest>
__device__ inline void tile_item(const Wl& d, int lane, const int32_t* __restrict__ idx, const float* __restrict__ val,
                                 const int32_t* __restrict__ rowid, const X& x, float* __restrict__ y,
                                 double* __restrict__ partial, int32_t sl, const Rest& rest) {
  if constexpr (Rest::kWhole) {
    const bool chunk = (d.info & 3) == kChunk && rest.ticket && sl == 0;
    int32_t i = 0;
    SplitRow sr{0, 0, 0, 0};
    if (chunk) {
      i = rest.slot_split[d.info >> 2];
      sr = rest.split[i];
    }
    run_workload<S, VEC, true>(d, lane, idx, val, rowid, x, y, partial, sl);
    if (chunk) finish_chunk(i, sr, lane, x, y, partial, rest);
  } else {
    run_workload<S, VEC, false>(d, lane, idx, val, rowid, x, y, partial, sl);
  }
}

template <class X>
__device__ inline void write_empty(const TileRest& rest, const X& x, float* __restrict__ y, int64_t i, int64_t step) {
  for (; i < rest.n_empty; i += step) x.addy(y, rest.empty[i], 0.0);
}

// p[0] + p[s] + ... + p[(n-1) s], added in that order; 32 loads go out
// together, then 8 (a split row can have hundreds of chunks, summed by one
// thread: the loads in flight set its time)
__device__ inline double sum_slots(const double* __restrict__ p, int64_t n, int64_t s = 1) {
  double acc = 0.0;
  int64_t q = 0;
  for (; q + 32 <= n; q += 32) {
    double t[32];
#pragma unroll
    for (int u = 0; u < 32; ++u) t[u] = p[(q + u) * s];
#pragma unroll
    for (int u = 0; u < 32; ++u) acc += t[u];
  }
  for (; q + 8 <= n; q += 8) {
    double t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = p[(q + u) * s];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += t[u];
  }
  for (; q < n; ++q) acc += p[q * s];
  return acc;
}

// The same sum as sum_slots (left to right from 0.0, so the same bits) by a
// whole wavefront: each round the lanes copy 256 slots at once into the
// wavefront's LDS buffer `buf` (256 doubles), then lane 0 adds them in slot
// order from LDS.  A row of hundreds of chunks then costs a few global load
// latencies instead of one per 32 slots.  The sum is valid in lane 0.
__device__ inline double sum_slots_wave(const double* __restrict__ p, int64_t n, int lane, double* buf) {
  double acc = 0.0;
  for (int64_t q = 0; q < n; q += 4 * kWave) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = q + u * kWave + lane;
      buf[u * kWave + lane] = i < n ? p[i] : 0.0;
    }
    __builtin_amdgcn_wave_barrier();
    const int m = (int)(n - q < 4 * kWave ? n - q : 4 * kWave);
    if (lane == 0) {
      int k = 0;
      for (; k + 8 <= m; k += 8) {
        double t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = buf[k + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += t[u];
      }
      for (; k < m; ++k) acc += buf[k];
    }
    __builtin_amdgcn_wave_barrier();
  }
  return acc;
}

// ---- vector kernels
// out[k*row_stride + q] = in[perm[k]*row_stride + q]   (rows gathered)
__global__ void k_gather_rows(const float* __restrict__ in, const int32_t* __restrict__ perm, int64_t n, int32_t w,
                              float* __restrict__ out) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * w) return;
  const int64_t k = t / w;
  const int32_t q = (int32_t)(t % w);
  out[t] = in[(int64_t)perm[k] * w + q];
}

// ... of one float: four per thread, so that their gathers go out together and
// the permutation and the output move 16 bytes a lane (any alignment).  Bound by
// the gathers' requests: 2^23 floats 45.9 us (183 G/s) where a float per thread,
// with 64-bit divisions by the row width, took 49.3.
__global__ void __launch_bounds__(kB) k_gather1(const float* __restrict__ in, const int32_t* __restrict__ perm,
                                                int64_t n, float* __restrict__ out) {
  const int64_t t = 4 * ((int64_t)blockIdx.x * kB + threadIdx.x);
  if (t + 4 <= n) {
    const v4iu p = __builtin_nontemporal_load((const v4iu*)(perm + t));
    v4fu v;
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = in[p[u]];
    *(v4fu*)(out + t) = v;
  } else {
    for (int64_t k = t; k < n; ++k) out[k] = in[perm[k]];
  }
}

// ... of 4 * w4 floats (16-byte aligned rows), one 16-byte piece per thread
__global__ void __launch_bounds__(kB) k_gather_rows4(const v4f* __restrict__ in, const int32_t* __restrict__ perm,
                                                     int64_t n, uint32_t w4, v4f* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * kB + threadIdx.x;
  if (t >= n * w4) return;
  const int64_t k = (w4 & (w4 - 1)) == 0 ? t >> __builtin_ctz(w4) : t / w4;
  out[t] = in[(int64_t)perm[k] * w4 + (t - k * w4)];
}

template <int NV>
__device__ inline void block_sum_store(double (&v)[NV], double* out_base, int64_t stride) {
  __shared__ double sm[NV][kB / kWave];
  const int lane = lane_id(), wv = threadIdx.x / kWave;
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    double s = wave_sum(v[q]);
    if (lane == 0) sm[q][wv] = s;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      double s = 0.0;
      for (int w = 0; w < kB / kWave; ++w) s += sm[q][w];
      out_base[q * stride] = s;
    }
  }
}

// Sum of v over the block (the order of block_sum_store), in every thread.
__device__ inline double block_sum(double v) {
  __shared__ double sm[kB / kWave];
  const double s = wave_sum(v);
  __syncthreads();  // the previous sum's readers are done
  if (lane_id() == 0) sm[threadIdx.x / kWave] = s;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < kB / kWave; ++w) t += sm[w];
  return t;
}

// Sum of up to 64 partials by every wavefront that needs it (each lane reads
// one): a launch of its own for it costs 2-5 us.
__device__ inline double wave_parts(const double* __restrict__ parts, int np) {
  return wave_sum(lane_id() < np ? parts[lane_id()] : 0.0);
}

// A reduction's second half in the same launch: every block gives its partial
// sum (v, of thread 0), and the block that draws the last ticket may read them
// all: true in that block.  The partials travel by agent-scope accesses, each
// complete before its block draws (no fence: an agent-scope release writes
// back the L2, 18 us where 1024 blocks did it); no block waits for another.
// The last block sets the ticket back to 0.
__device__ inline bool last_block(double* parts, double v, uint32_t* ticket) {
  __shared__ uint32_t last;
  if (threadIdx.x == 0) {
    __hip_atomic_store(parts + blockIdx.x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x;
    if (last) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  return last != 0;
}

// Sum of parts[b, e) in a fixed order, in the last block of last_block.
__device__ inline double sum_parts(const double* parts, int b, int e) {
  double s = 0.0;
  for (int i = b + (int)threadIdx.x; i < e; i += kB)
    s += __hip_atomic_load(parts + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return block_sum(s);
}

constexpr int kRedBlocks = 1024;

// Sum of nparts consecutive partials for each of nv quantities, fixed order:
// one wavefront per quantity (lane-strided sums, then the wavefront's tree),
// quantities spread over the wavefronts of the grid.
__global__ void k_finish(const double* __restrict__ parts, int nparts, int nv, double* __restrict__ out) {
  const int lane = lane_id();
  for (int q = blockIdx.x * kWpb + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave); q < nv;
       q += gridDim.x * kWpb) {
    const double* pq = parts + (int64_t)q * nparts;
    double s = 0.0;
    for (int i0 = lane; i0 < nparts; i0 += 8 * kWave) {  // eight loads in flight (past the end: pq[0], not added)
      double t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = pq[i0 + u * kWave < nparts ? i0 + u * kWave : 0];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += i0 + u * kWave < nparts ? t[u] : 0.0;
    }
    s = wave_sum(s);
    if (lane == 0) out[q] = s;
  }
}

}  // namespace
}  // namespace tc
