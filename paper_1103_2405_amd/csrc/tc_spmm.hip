// Multi-right-hand-side products Y = A X on the tiled composite format (the
// batched queries of Appendix F, Eq. 9, many restart vectors at once).
#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>

#include "tc_host.h"

namespace tc {

namespace {

// ---- multiple right-hand sides.  Pad entries (value 0) are skipped.
//
// SpMM, Y := A X with X row-major n_cols x k.  Each lane owns V consecutive
// right-hand sides (one 16-byte load per gathered X row and lane for V = 4) and
// KG lanes form a group that covers a row of up to 32 of them; the 64 / KG
// groups of a wavefront take different entries, so one load instruction
// serves 64 / KG entries and every gathered X row is one coalesced access.
// When k is no multiple of V the last lane of the row starts at k - V instead:
// it computes up to V - 1 right-hand sides a second time and stores only its
// own, and no lane reads past the row.
//
// A step covers SUB entries per group, all gathers in flight together; their
// values and indices are read once per wavefront, coalesced, one step ahead,
// and handed to the groups by lane shuffles.
template <int V>
struct Vec {
  double a[V];
  __device__ void zero() {
#pragma unroll
    for (int i = 0; i < V; ++i) a[i] = 0.0;
  }
};
template <int V>
struct FVec {
  float a[V];
};

// The right-hand sides of one lane: columns [col, col + V) of X and Y, of which
// it stores those from `own` on; act: it has any.
template <int V, int KG>
struct Cols {
  int32_t col, own;
  bool act;
  __device__ Cols(int lane, int32_t c0, int32_t k) {
    const int32_t c = c0 + (lane % KG) * V;
    act = c < k;
    col = act ? min(c, k - V) : 0;
    own = c - col;
  }
};

// X by 32-bit offsets through a buffer descriptor (n_cols <= 2^24 and at most
// 2^31 bytes): an inactive lane (pad entry, or right-hand sides past k) gives
// an offset past the buffer, reads zeros and makes no request.
template <int V>
struct SmallX {
  __amdgpu_buffer_rsrc_t r;
  uint32_t k4;  // bytes of a row
  __device__ SmallX(const float* X, int64_t n_cols, int32_t k)
      : r(__builtin_amdgcn_make_buffer_rsrc((void*)X, (short)0, (int32_t)(n_cols * k * 4), 0x00020000)),
        k4((uint32_t)k * 4) {}
  __device__ FVec<V> operator()(int32_t row, int32_t col, bool on) const {
    const int32_t o = on ? (int32_t)(__umul24((uint32_t)row, k4) + (uint32_t)col * 4) : (int32_t)0x80000000;
    FVec<V> x;
    if constexpr (V == 4) {
      const auto t = __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0);
      const v4f f = __builtin_bit_cast(v4f, t);
      x.a[0] = f.x, x.a[1] = f.y, x.a[2] = f.z, x.a[3] = f.w;
    } else if constexpr (V == 2) {
      const auto t = __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0);
      const v2f f = __builtin_bit_cast(v2f, t);
      x.a[0] = f.x, x.a[1] = f.y;
    } else {
      x.a[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0));
    }
    return x;
  }
};

typedef float v2fu __attribute__((ext_vector_type(2), aligned(4)));

// ... or of any size by 64-bit addresses.  Branch-free: an inactive lane reads
// X[0 .. V) and takes zeros (a load under a branch would end its branch with
// a wait for that load, so a step's gathers would go out one at a time).
template <int V>
struct LargeX {
  const float* X;
  int64_t k;
  __device__ LargeX(const float* x, int64_t, int32_t k_) : X(x), k(k_) {}
  __device__ FVec<V> operator()(int32_t row, int32_t col, bool on) const {
    const float* p = X + (on ? row * k + col : 0);
    FVec<V> x;
    if constexpr (V == 4) {
      const v4fu t = *(const v4fu*)p;
      x.a[0] = t.x, x.a[1] = t.y, x.a[2] = t.z, x.a[3] = t.w;
    } else if constexpr (V == 2) {
      const v2fu t = *(const v2fu*)p;
      x.a[0] = t.x, x.a[1] = t.y;
    } else {
      x.a[0] = *p;
    }
#pragma unroll
    for (int i = 0; i < V; ++i) x.a[i] = on ? x.a[i] : 0.0f;
    return x;
  }
};

template <int V>
__device__ inline void fma_vec(Vec<V>& acc, float v, const FVec<V>& x) {
#pragma unroll
  for (int i = 0; i < V; ++i) acc.a[i] = fma((double)v, (double)x.a[i], acc.a[i]);
}

template <int V>
__device__ inline void store_row(float* p, int32_t own, const float* o) {
  if constexpr (V == 4) {
    if (own == 0) {
      *(v4fu*)p = v4fu{o[0], o[1], o[2], o[3]};
      return;
    }
  } else if constexpr (V == 2) {
    if (own == 0) {
      *(v2fu*)p = v2fu{o[0], o[1]};
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < V; ++i)
    if (i >= own) p[i] = o[i];
}

// One row of Y, the first writer's store or a later tile's add; RWR: the
// restart of every right-hand side (its seed in LDS) fused in.
template <int V, bool RWR>
__device__ inline void write_row(float* __restrict__ Y, int32_t rid, int32_t k, int32_t col, int32_t own,
                                 const Vec<V>& s, const RwrEpi& epi, const int32_t* seeds_lds) {
  const int32_t row = rid & ~kAddFlag;
  float* p = Y + (int64_t)row * k + col;
  float o[V];
  if constexpr (RWR) {
#pragma unroll
    for (int i = 0; i < V; ++i) o[i] = rwr_restart(epi.c, (float)s.a[i], row == seeds_lds[col + i]);
  } else if (rid & kAddFlag) {
#pragma unroll
    for (int i = 0; i < V; ++i) o[i] = (float)((double)p[i] + s.a[i]);
  } else {
#pragma unroll
    for (int i = 0; i < V; ++i) o[i] = (float)s.a[i];
  }
  store_row<V>(p, own, o);
}

// Cross-group sum of a row-major row: the groups took interleaved entries,
// and an xor tree over the group bits of the lane id adds their sums.  At the
// first log2 V levels each lane passes on one half of its columns and adds up the
// other; the last steps hand every lane all V sums (the additions of the whole
// tree; 10 shuffles rather than 20 for V = 4 and 32 groups: 56.3 -> 48.5 us at k = 5 of
// a uniform matrix of 2^17 rows and 2.1M entries, 56.4 -> 42.7 at k = 4).
template <int V, int KG>
__device__ inline void group_sum(Vec<V>& s, int lane) {
  static_assert(V * KG <= kWave, "a level per halving");
  // the half of (a, b) that this lane keeps, with the partner's
  auto halve = [&](double a, double b, int o) {
    const bool up = lane & o;
    return (up ? b : a) + __shfl_xor(up ? a : b, o, kWave);
  };
  double t;
  if constexpr (V == 4)
    t = halve(halve(s.a[0], s.a[2], KG), halve(s.a[1], s.a[3], KG), 2 * KG);
  else if constexpr (V == 2)
    t = halve(s.a[0], s.a[1], KG);
  else
    t = s.a[0];
#pragma unroll
  for (int o = V * KG; o < kWave; o <<= 1) t += __shfl_xor(t, o, kWave);
  const int c = lane & (KG - 1);
  if constexpr (V == 4) {
    s.a[0] = __shfl(t, c, kWave);
    s.a[1] = __shfl(t, c + 2 * KG, kWave);
    s.a[2] = __shfl(t, c + KG, kWave);
    s.a[3] = __shfl(t, c + 3 * KG, kWave);
  } else if constexpr (V == 2) {
    s.a[0] = __shfl(t, c, kWave);
    s.a[1] = __shfl(t, c + KG, kWave);
  } else {
    s.a[0] = t;
  }
}

// The slots of one step: SUB * G of them (G = 64 / KG groups), L per lane;
// slot u * G + g belongs to group g's sub-step u.
template <int KG, int SUB>
struct Slots {
  static constexpr int G = kWave / KG, N = SUB * G, L = (N + kWave - 1) / kWave;
  float v[L];
  int32_t i[L];
  // slot s at element at(s) of the stream, where in(s), else the pad (0, 0)
  // (it reads element `safe`)
  template <class In, class At>
  __device__ void load(const int32_t* __restrict__ idx, const float* __restrict__ val, int lane, int64_t safe, In in,
                       At at) {
#pragma unroll
    for (int j = 0; j < L; ++j) {
      const int s = j * kWave + lane;
      const bool ok = s < N && in(s);
      const int64_t e = ok ? at(s) : safe;
      const float tv = ld_nt(val + e);
      const int32_t ti = ld_nt(idx + e);
      v[j] = ok ? tv : 0.0f;
      i[j] = ok ? ti : 0;
    }
  }
  __device__ void get(int u, int g, float& vo, int32_t& io) const {
    if constexpr (KG == 1) {
      vo = v[u];
      io = i[u];
    } else {
      const int src = (u % KG) * G + g;
      vo = __shfl(v[u / KG], src, kWave);
      io = __shfl(i[u / KG], src, kWave);
    }
  }
};

// sum over entries [lo, hi) of the row-major row at `base`: sub-step u of each
// step of SUB * G entries gives group g the entry u * G + g, and a group adds
// its own in increasing order.  (Counted by what is left: the entry after the
// last step of a row of almost 2^31 entries has no 32-bit number.)
template <int V, int KG, int SUB, class XR>
__device__ inline Vec<V> rm_range(const int32_t* __restrict__ idx, const float* __restrict__ val, const XR& X,
                                  int64_t base, int32_t lo, int32_t hi, const Cols<V, KG>& c, int lane) {
  using Sl = Slots<KG, SUB>;
  const int g = lane / KG;
  Vec<V> acc;
  acc.zero();
  Sl nx;
  int64_t at = base + lo;
  int32_t left = hi - lo;
  auto fetch = [&](int64_t e, int32_t n) {
    nx.load(idx, val, lane, base, [&](int s) { return s < n; }, [&](int s) { return e + s; });
  };
  if (left > 0) fetch(at, left);
  for (; left > 0; left -= Sl::N, at += Sl::N) {
    const Sl cur = nx;
    float v[SUB];
    FVec<V> x[SUB];
#pragma unroll
    for (int u = 0; u < SUB; ++u) {
      int32_t i;
      cur.get(u, g, v[u], i);
      x[u] = X(i, c.col, c.act && v[u] != 0.0f);
    }
    fetch(at + Sl::N, left - Sl::N);  // past the end: the row's first entry, not used
    __builtin_amdgcn_sched_barrier(0);  // every load is out before the first sum waits
#pragma unroll
    for (int u = 0; u < SUB; ++u) fma_vec<V>(acc, v[u], x[u]);
  }
  return acc;
}

// Column-major rectangle, rows sl * U * G, + slices * U * G, ...: a step covers
// U rows and C columns per group (U C gathers in flight); each row is summed by
// its group's lanes in column order.
template <int V, int KG, int U, int C, bool FENCE, bool RWR, class XR>
__device__ inline void cm_range(const Wl& d, int32_t sl, int32_t slices, const int32_t* __restrict__ idx,
                                const float* __restrict__ val, const int32_t* __restrict__ rowid, const XR& X,
                                float* __restrict__ Y, int32_t k, const Cols<V, KG>& c, int lane, const RwrEpi& epi,
                                const int32_t* sd) {
  using Sl = Slots<KG, U * C>;
  constexpr int R = U * Sl::G;  // rows of a step
  const int g = lane / KG;
  const int32_t w = d.w_pad, nr = d.n_rows, rstep = slices * R;
  const int64_t off = d.data_off, hp = d.h_pad;
  int32_t r0 = sl * R, c0 = 0;
  if (r0 >= nr) return;
  Sl nx;
  auto fetch = [&](int32_t r, int32_t cc) {
    nx.load(
        idx, val, lane, off, [&](int s) { return cc + s / R < w && r + s % R < nr; },
        [&](int s) { return off + (int64_t)(cc + s / R) * hp + r + s % R; });
  };
  int32_t rid[U];
  Vec<V> acc[U];
  auto begin = [&](int32_t r) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t q = r + u * Sl::G + g;
      rid[u] = ld_nt(rowid + d.rowid_off + (q < nr ? q : 0));
      acc[u].zero();
    }
  };
  fetch(r0, 0);
  begin(r0);
  for (;;) {
    const Sl cur = nx;
    const bool last = c0 + C >= w;
    const int32_t rn = last ? r0 + rstep : r0, cn = last ? 0 : c0 + C;
    float v[U * C];
    FVec<V> x[U * C];
#pragma unroll
    for (int q = 0; q < U * C; ++q) {  // sub-step q: column c0 + q / U, row r0 + (q % U) G + g
      int32_t i;
      cur.get(q, g, v[q], i);
      x[q] = X(i, c.col, c.act && v[q] != 0.0f);
    }
    fetch(rn, cn);  // past the rectangle: its first entry, not used
    if constexpr (FENCE) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < U * C; ++q) fma_vec<V>(acc[q % U], v[q], x[q]);
    if (last) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c.act && r0 + u * Sl::G + g < nr) write_row<V, RWR>(Y, rid[u], k, c.col, c.own, acc[u], epi, sd);
      if (rn >= nr) break;
      begin(rn);
    }
    r0 = rn;
    c0 = cn;
  }
}

// Entries in flight per group of KG lanes: R of a row-major row or chunk; U x C
// (rows x columns) of a column-major rectangle of one column (U1 x 1), of two or
// three, of more.  Registers set the wavefronts: the deep form takes 93-181 VGPRs
// (2 to 5 wavefronts per SIMD), the others 53-80 (6 to 8).  More wavefronts win where
// X's part of a pass lies near (uniform 2^16 rows and columns, 1M entries, with the
// row sums of every column shuffled whole, k = 4: 71 -> 42 us, 32: 61 -> 46, 100: 239 ->
// 150; group_sum makes the 42 33), more in flight where it does not
// (R-MAT 2^20, k = 32: 339 deep, 356 not) and where one wavefront has to sum a
// long row (Chung-Lu 2^20 without split rows, five steps at k = 16: 2,180 / 2,890).
// One lane a row (k = 1, 2, 4) has 64 entries in flight a wavefront to begin with.
template <int V, int KG, bool DEEP>
struct Flight {  // deep; KG of 4 and 8
  static constexpr int R = DEEP ? 8 : 4, U1 = DEEP ? 8 : 4;
  static constexpr int U2 = DEEP ? 4 : 2, C2 = 2, U4 = 2, C4 = DEEP ? 4 : 2;
  static constexpr bool kFence = false;
};
template <>
struct Flight<4, 2, false> {  // k = 5-8; the fence: 42 against 46 us on the uniform matrix, k = 8
  static constexpr int R = 4, U1 = 4, U2 = 2, C2 = 2, U4 = 1, C4 = 4;
  static constexpr bool kFence = true;
};
template <>
struct Flight<2, 2, false> {  // k = 3
  static constexpr int R = 4, U1 = 2, U2 = 2, C2 = 1, U4 = 2, C4 = 1;
  static constexpr bool kFence = false;
};
template <>
struct Flight<4, 1, false> {  // k = 4
  static constexpr int R = 2, U1 = 1, U2 = 1, C2 = 1, U4 = 1, C4 = 1;
  static constexpr bool kFence = false;
};
template <>
struct Flight<2, 1, false> {  // k = 2
  static constexpr int R = 4, U1 = 1, U2 = 1, C2 = 1, U4 = 1, C4 = 1;
  static constexpr bool kFence = false;
};
template <>
struct Flight<1, 1, false> {  // k = 1
  static constexpr int R = 4, U1 = 2, U2 = 1, C2 = 2, U4 = 1, C4 = 2;
  static constexpr bool kFence = false;
};

// One wavefront's part of a workload: piece `part` of a leading chunk workload
// (a split row's pieces: kPiece entries each, sums to slot chunk slot * parts +
// part of `partial`), or row slice `part` of `parts` of any other workload.  (A
// chunk among the others is done whole, as one piece.)
constexpr int kPiece = 512;
template <int V, int KG, bool DEEP, bool RWR, class XR>
__device__ inline void spmm_item(const Wl& d, int32_t part, int32_t parts, bool lead, const int32_t* __restrict__ idx,
                                 const float* __restrict__ val, const int32_t* __restrict__ rowid, const XR& xr,
                                 float* __restrict__ Y, int32_t k, const Cols<V, KG>& c, int lane,
                                 double* __restrict__ partial, const RwrEpi& epi, const int32_t* sd) {
  constexpr int G = kWave / KG;
  using F = Flight<V, KG, DEEP>;
  const bool g0 = lane < KG;
  if (lead) {
    const int32_t lo = (int32_t)min<int64_t>((int64_t)part * kPiece, d.w_pad), hi = lo + min(kPiece, d.w_pad - lo);
    Vec<V> acc = rm_range<V, KG, F::R>(idx, val, xr, d.data_off, lo, hi, c, lane);
    group_sum<V, KG>(acc, lane);
    if (c.act && g0)
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (i >= c.own) partial[((int64_t)(d.info >> 2) * parts + part) * k + c.col + i] = acc.a[i];
    return;
  }
  const int layout = d.info & 3;
  if (layout == kCM) {
    if (d.w_pad == 1)
      cm_range<V, KG, F::U1, 1, F::kFence, RWR>(d, part, parts, idx, val, rowid, xr, Y, k, c, lane, epi, sd);
    else if (d.w_pad <= 3)
      cm_range<V, KG, F::U2, F::C2, F::kFence, RWR>(d, part, parts, idx, val, rowid, xr, Y, k, c, lane, epi, sd);
    else
      cm_range<V, KG, F::U4, F::C4, F::kFence, RWR>(d, part, parts, idx, val, rowid, xr, Y, k, c, lane, epi, sd);
    return;
  }
  for (int32_t r = part; r < d.n_rows; r += parts) {
    const int64_t base = d.data_off + (int64_t)r * d.w_pad;
    const int32_t rid = layout == kChunk ? 0 : ld_nt(rowid + d.rowid_off + r);
    Vec<V> acc = d.w_pad > 2 * G ? rm_range<V, KG, F::R>(idx, val, xr, base, 0, d.w_pad, c, lane)
                 : d.w_pad > G   ? rm_range<V, KG, 2>(idx, val, xr, base, 0, d.w_pad, c, lane)
                                 : rm_range<V, KG, 1>(idx, val, xr, base, 0, d.w_pad, c, lane);
    group_sum<V, KG>(acc, lane);
    if (!(c.act && g0)) continue;
    if (layout == kChunk) {
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (i >= c.own) partial[(int64_t)(d.info >> 2) * k + c.col + i] = acc.a[i];
    } else {
      write_row<V, RWR>(Y, rid, k, c.col, c.own, acc, epi, sd);
    }
  }
}

// The passes over a tile, pass p = blockIdx.y for the right-hand sides V KG p, ...:
// wavefronts for the pieces of the tile's leading chunk workloads, then for
// the row slices of the others.
//
// Bound at k = 32 on a 31.4M-entry power-law matrix of 1M rows (304 us of the
// kernel, 346 a product; 336 and 378 with two launches, four rows or eight
// entries in flight without the next step's entries, and a branch per entry):
// 2.0 GB of L2 misses, 6.5 TB/s, the card's streaming-read rate.  124 VGPRs,
// four wavefronts per SIMD: capping them for 5 or 6 measured 358 and 404 us (the
// kernel spills), 16 entries in flight 367, 8 row slices 455 (wavefronts
// without a row to sum), 2 362; a persistent grid with an LDS item counter 351.
// By k, us a product of the R-MAT matrix of 2^20 (16M entries) with one right-hand
// side per lane for k no multiple of 4, and now: 3 228 -> 174, 4 199 -> 165, 8 224 ->
// 190, 37 1,295 -> 719; 13 on 4.8M entries of 100K columns 99 -> 62.
template <int V, int KG, bool DEEP, bool RWR, template <int> class XR>
__global__ void __launch_bounds__(kB) k_tile_spmm(const Wl* __restrict__ wl, int64_t n_wl, int64_t n_lead,
                                                  int32_t pieces, int32_t slices, const int32_t* __restrict__ idx,
                                                  const float* __restrict__ val, const int32_t* __restrict__ rowid,
                                                  const float* __restrict__ X, int64_t n_cols, int32_t ldx,
                                                  float* __restrict__ Y, int32_t k,
                                                  double* __restrict__ partial, RwrEpi epi) {
  // fused restart: the seeds (k <= kB) in LDS, read only where rows are written
  __shared__ int32_t sd[RWR ? kB : 1];
  if constexpr (RWR) {
    if ((int32_t)threadIdx.x < k) sd[threadIdx.x] = epi.seeds[threadIdx.x];
    __syncthreads();
  }
  const int lane = lane_id();
  const int64_t w = (int64_t)blockIdx.x * kWpb + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t lead_items = n_lead * pieces, v = w - lead_items;
  if (v >= (n_wl - n_lead) * slices) return;
  const bool lead = v < 0;
  const Wl d = wl[lead ? w / pieces : n_lead + v / slices];
  const Cols<V, KG> c(lane, (int32_t)blockIdx.y * (V * KG), k);
  const XR<V> xr(X, n_cols, ldx);
  spmm_item<V, KG, DEEP, RWR>(d, (int32_t)(lead ? w % pieces : v % slices), lead ? pieces : slices, lead, idx, val, rowid,
                        xr, Y, k, c, lane, partial, epi, sd);
}

// Zero the rows no workload writes: block b takes rows b * rpb ..., thread
// (r, q) of the block row r's entries q, q + kk, ... (kk = min(k, kB))
// (with the fused restart, epi.seeds != NULL: the rows' restart values)
__global__ void k_begin_spmm(float* __restrict__ Y, const int32_t* __restrict__ empty, int64_t n_empty, int32_t k,
                             RwrEpi epi) {
  const int32_t kk = min(k, kB), rpb = kB / kk;
  const int32_t r = threadIdx.x / kk, q0 = threadIdx.x % kk;
  if (r >= rpb) return;
  for (int64_t i = (int64_t)blockIdx.x * rpb + r; i < n_empty; i += (int64_t)gridDim.x * rpb) {
    const int32_t e = empty[i];
    float* row = Y + (int64_t)e * k;
    for (int32_t q = q0; q < k; q += kk) row[q] = epi.seeds ? rwr_restart(epi.c, 0.0f, e == epi.seeds[q]) : 0.0f;
  }
}

__global__ void k_split_combine_mm(const SplitRow* __restrict__ sr, int64_t n, const double* __restrict__ partial,
                                   int32_t pieces, float* __restrict__ Y, int32_t k, RwrEpi epi) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * k) return;
  const int64_t i = t / k;
  const int32_t q = (int32_t)(t % k);
  const SplitRow s = sr[i];
  const int64_t u0 = (int64_t)s.slot_begin * pieces;
  const double acc = sum_slots(partial + u0 * k + q, (int64_t)s.n_slots * pieces, k);
  if (epi.seeds)  // fused restart (one tile: the chunks are all of the row)
    Y[(int64_t)s.row * k + q] = rwr_restart(epi.c, (float)acc, s.row == epi.seeds[q]);
  else if (s.store)
    Y[(int64_t)s.row * k + q] = (float)acc;
  else
    add_to_y(Y + (int64_t)s.row * k, q, acc);
}

// Leading chunk workloads of every tile, found once per handle from the host
// workload list.  pieces = 1 when some tile has a chunk after a non-chunk
// workload (those chunks are then done whole by k_tile_spmm).
void spmm_plan(tc_handle* h) {
  if (h->mm_planned) return;
  h->mm_lead.assign(h->n_tiles, 0);
  int64_t max_wpad = 0;
  bool lead_only = true;
  for (int t = 0; t < h->n_tiles; ++t) {
    const int64_t b = h->tile_wl_begin[t], e = h->tile_wl_begin[t + 1];
    int64_t i = b;
    while (i < e && h->wls[i].layout == kChunk) max_wpad = std::max<int64_t>(max_wpad, h->wls[i++].w_pad);
    h->mm_lead[t] = i - b;
    for (; i < e; ++i)
      if (h->wls[i].layout == kChunk) lead_only = false;
  }
  h->mm_pieces = lead_only && max_wpad > 0 ? (int32_t)((max_wpad + kPiece - 1) / kPiece) : 1;
  if (!lead_only) h->mm_lead.assign(h->n_tiles, 0);
  h->mm_planned = true;
}

// The passes of one tile over the k right-hand sides, 32 at a time (128 bytes
// of each X row, one cache line per gather), in one launch.  Wider passes spread
// the gathers over n * 4k bytes, past the 256 MB MALL at a million rows and k =
// 64 (measured on a 31M-entry power-law matrix, 1M rows: k = 64 1262 -> 1152 us,
// k = 128 2718 -> 2244 us per product; 16 per pass slows k = 32 by 40%).  The
// last pass has the lanes of a whole one: fewer lanes in a launch of their own
// measured 667 / 631 us at k = 36 on the R-MAT matrix of 2^20, 200 / 192 on a
// rectangle of 4.8M entries, 25.3 / 22.1 on one of 2^12 rows (whole / fewer).
//
// The form of the kernel (see Flight): deep for a tile with a long row, and for more than 16 right-hand sides where a
// pass reads more than 2^18 rows of X (32 MB, what the eight L2s hold): deep / not,
// us at k = 32 and 64, uniform and R-MAT matrices of 2^17 columns 75 / 60, 142 /
// 112, 57 / 54, 96 / 89; of 2^18 107 / 107, 206 / 208, 91 / 89, 166 / 163; of 2^20
// 377 / 387, 744 / 761, 336 / 355, 613 / 642.
constexpr int64_t kNearCols = (int64_t)1 << 18;
template <bool RWR, template <int> class XR>
void spmm_tile_x(tc_handle* h, int t, int64_t b, int64_t n, int64_t lead, int32_t pieces, int32_t slices,
                 const float* X, int32_t ldx, float* Y, int32_t k, double* partial, const RwrEpi& ep, hipStream_t st) {
  const bool lone = long_row(h, t);
  const unsigned gx = nblk(lead * pieces + (n - lead) * slices, kWpb);
  auto go = [&](auto near, auto deep, bool d) {
    launch_tile(h, d ? deep : near, dim3(gx, (unsigned)((k + 31) / 32)), dim3(kB), 0, st, (const Wl*)(h->d_wl + b), n,
                lead, pieces, slices, (const int32_t*)h->d_idx, (const float*)h->d_val, (const int32_t*)h->d_rowid, X,
                (int64_t)h->n_cols, ldx, Y, k, partial, ep);
  };
  if (k == 1) return go(k_tile_spmm<1, 1, false, RWR, XR>, k_tile_spmm<1, 1, true, RWR, XR>, lone);
  if (k == 2) return go(k_tile_spmm<2, 1, false, RWR, XR>, k_tile_spmm<2, 1, true, RWR, XR>, lone);
  if (k == 3) return go(k_tile_spmm<2, 2, false, RWR, XR>, k_tile_spmm<2, 2, true, RWR, XR>, lone);
  if (k == 4) return go(k_tile_spmm<4, 1, false, RWR, XR>, k_tile_spmm<4, 1, true, RWR, XR>, lone);
  if (k <= 8) return go(k_tile_spmm<4, 2, false, RWR, XR>, k_tile_spmm<4, 2, true, RWR, XR>, lone);
  if (k <= 16) return go(k_tile_spmm<4, 4, false, RWR, XR>, k_tile_spmm<4, 4, true, RWR, XR>, lone);
  go(k_tile_spmm<4, 8, false, RWR, XR>, k_tile_spmm<4, 8, true, RWR, XR>, lone || h->n_cols > kNearCols);
}

// out[c] = X[cperm[c]], rows of k floats into rows of 4 ld4 (the rest zeros)
__global__ void __launch_bounds__(kB) k_gather_pad(const float* __restrict__ X, const int32_t* __restrict__ cperm,
                                                   int64_t n, int32_t k, uint32_t ld4, v4f* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * kB + threadIdx.x;
  if (t >= n * ld4) return;
  const int64_t c = t / ld4;
  const int32_t q = 4 * (int32_t)(t - c * ld4);
  const float* p = X + (int64_t)cperm[c] * k;
  v4f v;
  if (q + 4 <= k) {
    v = *(const v4fu*)(p + q);
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = q + u < k ? p[q + u] : 0.0f;
  }
  out[t] = v;
}

// Floats between the rows of tc_spmm's own copy of X: rows of more than 4 lie in
// as few lines as they can.  us a product, unpadded / padded, on a rectangle of
// 4.8M entries and 100K columns: k = 7 61 / 58, 13 71 / 65, 23 108 / 91, 29 130 / 92,
// 37 229 / 208; on the 16M-entry R-MAT matrix of 2^20: 228 / 214, 281 / 249, 453 / 383,
// 545 / 418, 844 / 751.  17 and 18 would nearly double (17: 85 / 88 and 346 / 337), and
// a copy past the 256 MB MALL was not measured: both stay as they are.
int32_t padded_rows(int64_t n_cols, int32_t k) {
  int32_t ld = k;
  if (k > 32)
    ld = (k + 7) / 8 * 8;
  else if (k > 18)
    ld = 32;
  else if (k > 4 && k <= 16)
    ld = k <= 8 ? 8 : 16;
  return n_cols * ld * (int64_t)sizeof(float) <= ((int64_t)256 << 20) ? ld : k;
}

void spmm_tile(tc_handle* h, int t, int64_t b, int64_t n, int64_t lead, int32_t pieces, int32_t slices, const float* X,
               int32_t ldx, float* Y, int32_t k, double* partial, bool rwr, const RwrEpi& ep, hipStream_t st) {
  const bool small = h->n_cols <= ((int64_t)1 << 24) && h->n_cols * ldx < ((int64_t)1 << 29);
  auto f = rwr ? (small ? spmm_tile_x<true, SmallX> : spmm_tile_x<true, LargeX>)
               : (small ? spmm_tile_x<false, SmallX> : spmm_tile_x<false, LargeX>);
  f(h, t, b, n, lead, pieces, slices, X, ldx, Y, k, partial, ep, st);
}

}  // namespace

// epi (one tile, k <= kB): write the RWR restart of every row instead of
// the product.  skip_empty: the rows no workload writes already hold what
// this call would write there (0, or with epi their restart values).
size_t spmm_partial_doubles(tc_handle* h, int32_t k) {
  spmm_plan(h);
  return (size_t)h->n_slots * h->mm_pieces * k;
}

// Row slices of a workload: 4 (the kernel has the figures), 2 where the workloads
// are so small that wavefronts without a row to sum are most of the launch.
// Four / two, us at k = 5 by workload size: 22.1 / 17.8 at 54 (19,810 rows of 28
// entries), 28.3 / 25.6 at 108 (40,000 of 28), 27.1 / 27.6 at 128 (R-MAT 2^16),
// 16.1 / 17.2, 24.6 / 26.5 and 26.4 / 29.3 at 256.
constexpr int64_t kFewSlicesWl = 128;

void spmm_internal(tc_handle* h, const float* X, float* Y, int32_t k, hipStream_t st, bool skip_empty,
                   const RwrEpi* epi, double* partial_ext, int32_t ldx) {
  if (ldx == 0) ldx = k;
  if (epi && !(h->n_tiles == 1 && h->xcd_groups == 0 && k <= kB))
    throw Err{TC_EINVAL, "fused restart needs one tile and k <= 256"};
  const RwrEpi ep = epi ? *epi : RwrEpi{0.0, nullptr};
  spmm_plan(h);
  const int32_t pieces = h->mm_pieces;
  double* partial = nullptr;
  if (partial_ext) {
    partial = partial_ext;
  } else if (h->n_slots > 0) {
    const size_t need = sizeof(double) * (size_t)h->n_slots * pieces * k;
    if (need > h->mm_partial_bytes) {
      if (h->d_mm_partial) pool_free(h->d_mm_partial, st, false);
      h->d_mm_partial = nullptr;
      h->mm_partial_bytes = 0;
      if (!(h->d_mm_partial = (double*)pool_alloc(need, st)))
        throw Err{TC_ENOMEM, "SpMM partial sums: allocation of " + std::to_string(need) + " bytes failed"};
      h->mm_partial_bytes = need;
    }
    partial = h->d_mm_partial;
  }
  const bool timing = h->timing;
  if (partial_ext) h->timing = false;  // event creation is not for callers that cannot allocate
  if (h->n_empty > 0 && !skip_empty) {
    const int64_t rpb = kB / std::min(k, kB);
    hipLaunchKernelGGL(k_begin_spmm, dim3((unsigned)std::min<int64_t>(nblk(h->n_empty, rpb), 1 << 16)), dim3(kB), 0,
                       st, Y, (const int32_t*)h->d_empty, h->n_empty, k, ep);
    HIPC(hipGetLastError());
  }
  for (int t = 0; t < h->n_tiles; ++t) {
    const int64_t b = h->tile_wl_begin[t], e = h->tile_wl_begin[t + 1];
    const int64_t lead = h->mm_lead[t];
    const int32_t slices = h->tile_wl[t] <= kFewSlicesWl ? 2 : 4;
    if (e > b) spmm_tile(h, t, b, e - b, lead, pieces, slices, X, ldx, Y, k, partial, epi != nullptr, ep, st);
  }
  if (h->n_split_rows > 0) {
    hipLaunchKernelGGL(k_split_combine_mm, dim3(nblk(h->n_split_rows * k, kB)), dim3(kB), 0, st, h->d_split,
                       h->n_split_rows, (const double*)partial, pieces, Y, k, ep);
    HIPC(hipGetLastError());
  }
  h->timing = timing;
  h->spmv_calls++;
}

}  // namespace tc

using namespace tc;

extern "C" tc_status tc_spmm(const tc_handle* hc, const float* X, float* Y, int32_t k, tc_stream_t stream) {
  return guarded("tc_spmm", [&]() -> tc_status {
    if (!hc || (!X && hc->n_cols > 0) || (!Y && hc->n_rows > 0)) throw Err{TC_EINVAL, "NULL argument"};
    if (k < 1 || k > 256) throw Err{TC_EINVAL, "k must be in [1, 256]"};
    if ((const void*)X == (const void*)Y && hc->n_rows > 0) throw Err{TC_EINVAL, "X and Y must not alias"};
    tc_handle* h = const_cast<tc_handle*>(hc);
    hipStream_t st = (hipStream_t)stream;
    const size_t yb = sizeof(float) * (size_t)h->n_rows * k;
    auto x_bytes = [&](int32_t ld) { return (sizeof(float) * (size_t)h->n_cols * ld + 255) / 256 * 256; };
    int32_t ld = padded_rows(h->n_cols, k);
    char* ws = nullptr;
    try {
      ws = (char*)workspace(h, x_bytes(ld) + yb, st);
    } catch (const Err&) {
      if (ld == k) throw;
      ws = (char*)workspace(h, x_bytes(ld = k) + yb, st);
    }
    float* Xi = (float*)ws;
    float* Yi = (float*)(ws + x_bytes(ld));
    if (ld == k) {
      gather_rows(X, h->d_cperm, h->n_cols, k, Xi, st);
    } else if (h->n_cols > 0) {
      hipLaunchKernelGGL(k_gather_pad, dim3(nblk(h->n_cols * (ld / 4), kB)), dim3(kB), 0, st, X,
                         (const int32_t*)h->d_cperm, h->n_cols, k, (uint32_t)(ld / 4), (v4f*)Xi);
      HIPC(hipGetLastError());
    }
    if (h->relabel) {
      spmm_internal(h, Xi, Yi, k, st, false, nullptr, nullptr, ld);
      gather_rows(Yi, h->d_rowmap, h->n_rows, k, Y, st);
    } else {
      spmm_internal(h, Xi, Y, k, st, false, nullptr, nullptr, ld);
    }
    return TC_OK;
  });
}

// ---- SpMM for callers that cannot allocate (code under HIP graph capture,
// serving loops, harnesses that forbid hipMalloc): the split-row partial sums
// live in this file-scope device array instead of the handle's pool buffer.
// Every call on a device shares that device's copy (calls that overlap on one
// GPU race); nothing in it needs clearing, each product writes every slot it
// reads.  The array's address on each device comes from hipGetSymbolAddress
// on the first call with that device current.
namespace {
constexpr size_t kScratchDoubles = (size_t)1 << 21;  // 16 MiB per device
__device__ __align__(256) double scratch[kScratchDoubles];
std::mutex g_scratch_mu;
std::map<int, double*> g_scratch_ptr;

double* scratch_on_current_device() {
  int dev = 0;
  HIPC(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  auto it = g_scratch_ptr.find(dev);
  if (it != g_scratch_ptr.end()) return it->second;
  double* p = nullptr;
  HIPC(hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch)));
  g_scratch_ptr[dev] = p;
  return p;
}
}  // namespace

extern "C" tc_status tc_spmm_internal_noalloc(const tc_handle* hc, const float* X, float* Y, int32_t k,
                                              tc_stream_t stream) {
  return guarded("tc_spmm_internal_noalloc", [&]() -> tc_status {
    if (!hc || (!X && hc->n_cols > 0) || (!Y && hc->n_rows > 0)) throw Err{TC_EINVAL, "NULL argument"};
    if (k < 1 || k > 256) throw Err{TC_EINVAL, "k must be in [1, 256]"};
    if ((const void*)X == (const void*)Y && hc->n_rows > 0) throw Err{TC_EINVAL, "X and Y must not alias"};
    tc_handle* h = const_cast<tc_handle*>(hc);
    const size_t need = spmm_partial_doubles(h, k);
    if (need > kScratchDoubles)
      throw Err{TC_EINVAL, "split-row partial sums need " + std::to_string(need * sizeof(double)) +
                               " bytes, more than the " + std::to_string(kScratchDoubles * sizeof(double)) +
                               "-byte scratch of this call"};
    double* ptr = scratch_on_current_device();
    spmm_internal(h, X, Y, k, (hipStream_t)stream, false, nullptr, ptr);
    return TC_OK;
  });
}
