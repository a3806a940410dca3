// Differentiable RWR with learned edge weights (Appendix F, Eq. 9 with
// w = softplus(theta . f)): the weights and their column normalisation, the
// checkpointed forward iterations, the adjoint pass and the chain to theta.
#include <algorithm>
#include <cmath>
#include <memory>
#include <vector>

#include "tc_expand.h"
#include "tc_tile.h"

namespace tc {

namespace {

// ---- differentiable RWR: learned edge weights (Appendix F, Eq. 9)
//
// z_e = theta . f_e, w_e = softplus(z_e), W_e = w_e / S_j with S_j the sum of
// w over column j.  The per-entry arrays of the gradient (features, z, w, G)
// are kept in the order of A^T's CSR (the columns of A, each by increasing
// row), so every column quantity is a contiguous segmented pass; the values
// of W in A's own order are computed from A's copy of the features.
__device__ inline double softplus_d(double z) { return fmax(z, 0.0) + log1p(exp(-fabs(z))); }

// w of one entry; the same arithmetic in both orders, so W and W^T get
// bit-identical values
__device__ inline double edge_w(const float* __restrict__ f, const double* __restrict__ theta, int32_t nf,
                                double* z_out) {
  double a = 0.0;
  for (int32_t d = 0; d < nf; ++d) a = fma((double)f[d], theta[d], a);
  if (z_out) *z_out = a;
  return softplus_d(a);
}

__global__ void k_edge_softplus(const float* __restrict__ featsT, int64_t nnz, int32_t nf,
                                const double* __restrict__ theta, double* __restrict__ zT, double* __restrict__ wT) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= nnz) return;
  double z;
  wT[q] = edge_w(featsT + q * nf, theta, nf, &z);
  zT[q] = z;
}

// W in A's order: val_e = fl32(w_e / S_col(e))
__global__ void k_edge_values(const float* __restrict__ feats, const int32_t* __restrict__ col, int64_t nnz,
                              int32_t nf, const double* __restrict__ theta, const double* __restrict__ S,
                              float* __restrict__ val) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < nnz) val[e] = (float)(edge_w(feats + e * nf, theta, nf, nullptr) / S[col[e]]);
}

// Column sums over A^T's CSR: groups of kColLanes lanes take one column each,
// and the columns of more than kColLong entries go to a list whose columns
// take a block each (hubs sit next to each other, so a wavefront that sums
// those it meets is left with most of a graph's entries: S and cs of R-MAT 2^18
// symmetrised, 7.6M entries, 72 and 145 us that way, 50 and 86 so).  Every
// lane loads (a
// lane past the column's end at the column's first entry) and adds only its
// own entries.  The per-entry passes that need a column's sum are flat passes
// over the entries (the column of entry q: rowT[q]).
constexpr int kColLanes = 8;
constexpr int kColLong = 512;
constexpr int kGradBlocks = 1024;
constexpr int kMaxFeat = 16;

// sum over each aligned group of kColLanes lanes (every lane gets the same bits)
__device__ inline double group_sum8(double v) {
  v += __shfl_xor(v, 1, kWave);
  v += __shfl_xor(v, 2, kWave);
  v += __shfl_xor(v, 4, kWave);
  return v;
}

// this lane's part of the sum over q in [a, b) of f(q): LANES lanes from
// offset gl, U loads in flight
template <int LANES, int U, class F>
__device__ inline double seg_part(int64_t a, int64_t b, int gl, F f) {
  double s = 0.0;
  for (int64_t q0 = a + gl; q0 < b; q0 += U * LANES) {
    double t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t q = q0 + u * LANES;
      t[u] = f(q < b ? q : a);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) s += q0 + u * LANES < b ? t[u] : 0.0;
  }
  return s;
}

// Columns of more than kColLong entries: how many, and which.
struct LongCols {
  uint32_t* count;  // zero before the pass
  int32_t* list;
};

// out[j] = post(j, sum over column j's entries q of f(q)), short columns
template <class F, class P>
__device__ inline void col_sums(const int64_t* __restrict__ rpT, int64_t n_cols, F f, P post, const LongCols& lc,
                                double* __restrict__ out) {
  const int lane = lane_id(), gl = lane % kColLanes;
  const int64_t cg = (int64_t)blockIdx.x * kWpb + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t j0 = cg * (kWave / kColLanes);
  if (j0 >= n_cols) return;
  const int64_t j = j0 + lane / kColLanes;
  int64_t a = 0, b = 0;
  if (j < n_cols) {
    a = rpT[j];
    b = rpT[j + 1];
  }
  const bool lng = b - a > kColLong;
  const double s = group_sum8(lng || j >= n_cols ? 0.0 : seg_part<kColLanes, 4>(a, b, gl, f));
  if (gl != 0 || j >= n_cols) return;
  if (lng)
    lc.list[atomicAdd(lc.count, 1u)] = (int32_t)j;  // in any order: each has a sum of its own
  else
    out[j] = post(j, s);
}

// ... and the long ones
template <class F, class P>
__device__ inline void col_sums_long(const int64_t* __restrict__ rpT, F f, P post, const LongCols& lc,
                                     double* __restrict__ out) {
  const uint32_t n = *lc.count;
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int32_t j = lc.list[i];
    const double s = block_sum(seg_part<kB, 8>(rpT[j], rpT[j + 1], threadIdx.x, f));
    if (threadIdx.x == 0) out[j] = post(j, s);
  }
}

// S_j = sum of w over column j
template <bool LONG>
__global__ void __launch_bounds__(kB) k_col_norm(const int64_t* __restrict__ rpT, int64_t n_cols,
                                                 const double* __restrict__ wT, LongCols lc, double* __restrict__ S) {
  auto f = [&](int64_t q) { return wT[q]; };
  auto post = [](int64_t, double s) { return s; };
  if constexpr (LONG)
    col_sums_long(rpT, f, post, lc, S);
  else
    col_sums(rpT, n_cols, f, post, lc, S);
}

// W^T's values fl32(w / S_j)
__global__ void k_values_T(const int32_t* __restrict__ rowT, int64_t nnz, const double* __restrict__ wT,
                           const double* __restrict__ S, float* __restrict__ valT) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < nnz) valT[q] = (float)(wT[q] / S[rowT[q]]);
}

// r_next = fl32(c y + (1 - c) [i == seed]) (the same rounding as k_rwr_update)
__global__ void k_rwr_step(const float* __restrict__ y, float* __restrict__ r, int64_t n, int32_t seed, double c) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) r[i] = (float)(c * (double)y[i] + (i == seed ? 1.0 - c : 0.0));
}

// Rows for the per-entry sums: row u of dst (ROW floats) holds user id u's
// value in each of m <= ROW vectors.  inv: internal -> user id of the vectors
// (null: they are in user ids).  A wavefront reads 64 values of each vector
// and writes whole rows through LDS.
template <int ROW>
__global__ void __launch_bounds__(kB) k_step_rows(const float* __restrict__ src, int32_t m, int64_t n,
                                                  const int32_t* __restrict__ inv, float* __restrict__ dst) {
  constexpr int P = ROW + 1, L = ROW / 4, R = kWave / L;  // padded row; lanes per row, rows per store
  __shared__ float sm[kWpb][kWave * P];
  const int lane = lane_id();
  float* t = sm[threadIdx.x / kWave];
  const int64_t i0 = ((int64_t)blockIdx.x * kWpb + threadIdx.x / kWave) * kWave;
  if (i0 >= n) return;
  const int64_t i = i0 + lane < n ? i0 + lane : i0;
#pragma unroll 8
  for (int32_t q = 0; q < m; ++q) t[lane * P + q] = src[(int64_t)q * n + i];
  for (int32_t q = m; q < ROW; ++q) t[lane * P + q] = 0.0f;
  __builtin_amdgcn_wave_barrier();
  const int32_t u = inv ? inv[i] : (int32_t)i;
#pragma unroll
  for (int r = 0; r < kWave; r += R) {
    const int row = r + lane / L, c = 4 * (lane % L);
    const int64_t ur = __shfl(u, row, kWave);
    const float* p = t + row * P + c;
    if (i0 + row < n && c < m) *(v4f*)(dst + ur * ROW + c) = v4f{p[0], p[1], p[2], p[3]};
  }
}

// G_q (+)= sum over a batch of m <= ROW steps, latest first, of g^{k+1}_i r^k_j
// for the entry q = (i, j) of A (row j of A^T, column i of A^T: gidx = A^T's
// column array, ridx = A^T's row of every entry); the steps' values of i and j
// are the first m of their rows of gr and rr (k_step_rows).  The random rows,
// those of i, come through LDS: ROW / 4 lanes read a row (one 128-byte line for
// ROW = 32) at once, then each lane adds its own entry's steps.  Bound by those
// lines: 7.6M entries, 30 steps, 118 us (64 G lines/s); a pass per checkpoint
// segment of 6 read as many lines each time and took 5 x 174.
template <int ROW, bool FIRST>
__global__ void __launch_bounds__(kB) k_edge_accum(const int32_t* __restrict__ gidx, const int32_t* __restrict__ ridx,
                                                   int64_t nnz, const float* __restrict__ gr,
                                                   const float* __restrict__ rr, int32_t m, double* __restrict__ G) {
  constexpr int P = ROW + 1, L = ROW / 4, R = kWave / L;
  __shared__ float sm[kWpb][kWave * P];
  const int lane = lane_id();
  float* t = sm[threadIdx.x / kWave];
  const int64_t q0 = ((int64_t)blockIdx.x * kWpb + threadIdx.x / kWave) * kWave;
  if (q0 >= nnz) return;
  const int64_t q = q0 + lane < nnz ? q0 + lane : q0;
  const int32_t gi = gidx[q];
  const float* rp = rr + (int64_t)ridx[q] * ROW;
  double acc = FIRST ? 0.0 : G[q];
  const int c = 4 * (lane % L);
  v4f a[L];
#pragma unroll
  for (int u = 0; u < L; ++u) {  // R rows per load; pieces past m: the row's first
    const int32_t row = __shfl(gi, u * R + lane / L, kWave);
    a[u] = *(const v4f*)(gr + (int64_t)row * ROW + (c < m ? c : 0));
  }
#pragma unroll
  for (int u = 0; u < L; ++u) {
    float* p = t + (u * R + lane / L) * P + c;
    p[0] = a[u].x, p[1] = a[u].y, p[2] = a[u].z, p[3] = a[u].w;
  }
  __builtin_amdgcn_wave_barrier();
  const float* gp = t + lane * P;
  int32_t s = 0;
  for (; s + 4 <= m; s += 4) {
    const v4f r = *(const v4f*)(rp + s);
    acc = fma((double)gp[s], (double)r.x, acc);
    acc = fma((double)gp[s + 1], (double)r.y, acc);
    acc = fma((double)gp[s + 2], (double)r.z, acc);
    acc = fma((double)gp[s + 3], (double)r.w, acc);
  }
  for (; s < m; ++s) acc = fma((double)gp[s], (double)rp[s], acc);
  if (q0 + lane < nnz) G[q] = acc;
}

// The same without rows, where there is no memory for them: step t's values at
// g[t n + i] and r[t n + j], i and j by way of the maps to the vectors' ids (null:
// they are in user ids).
template <bool FIRST>
__global__ void __launch_bounds__(kB) k_edge_accum_vec(const int32_t* __restrict__ gidx,
                                                       const int32_t* __restrict__ ridx, int64_t nnz,
                                                       const float* __restrict__ g, const float* __restrict__ r,
                                                       const int32_t* __restrict__ gmap,
                                                       const int32_t* __restrict__ rmap, int64_t n, int32_t m,
                                                       double* __restrict__ G) {
  const int64_t q = (int64_t)blockIdx.x * kB + threadIdx.x;
  if (q >= nnz) return;
  const int32_t i = gmap ? gmap[gidx[q]] : gidx[q], j = rmap ? rmap[ridx[q]] : ridx[q];
  double acc = FIRST ? 0.0 : G[q];
#pragma unroll 4
  for (int32_t t = 0; t < m; ++t) acc = fma((double)g[t * n + i], (double)r[t * n + j], acc);
  G[q] = acc;
}

// a seed's internal id (no seed: -1)
__global__ void k_set_seed(int32_t* __restrict__ out, const int32_t* __restrict__ map, int32_t seed) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *out = seed < 0 ? -1 : map[seed];
}

__global__ void k_onehot(float* __restrict__ r, int64_t n, int32_t seed) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) r[i] = i == seed ? 1.0f : 0.0f;
}

// per column j: cs_j = sum over its entries of dL/dW W, with dL/dW = c G and
// W = w / S_j, taken as (c / S_j) sum G w
template <bool LONG>
__global__ void __launch_bounds__(kB) k_col_dot(const int64_t* __restrict__ rpT, int64_t n_cols,
                                                const double* __restrict__ GT, const double* __restrict__ wT,
                                                const double* __restrict__ S, double c, LongCols lc,
                                                double* __restrict__ cs) {
  auto f = [&](int64_t q) { return GT[q] * wT[q]; };
  auto post = [&](int64_t j, double s) { return c / S[j] * s; };
  if constexpr (LONG)
    col_sums_long(rpT, f, post, lc, cs);
  else
    col_sums(rpT, n_cols, f, post, lc, cs);
}

// dL/dz = (c G - cs_j) / S_j * sigmoid(z) per entry (column j = rowT[q]);
// per-block partial sums of dL/dz f (nf of them), combined afterwards in
// block order
__global__ void __launch_bounds__(kB) k_theta_grad(const int32_t* __restrict__ rowT, int64_t nnz, int32_t nf,
                                                   const float* __restrict__ featsT, const double* __restrict__ zT,
                                                   const double* __restrict__ S, const double* __restrict__ GT,
                                                   const double* __restrict__ cs, double c,
                                                   double* __restrict__ parts) {
  double acc[kMaxFeat];
#pragma unroll
  for (int d = 0; d < kMaxFeat; ++d) acc[d] = 0.0;
  for (int64_t q = (int64_t)blockIdx.x * kB + threadIdx.x; q < nnz; q += (int64_t)gridDim.x * kB) {
    const int32_t j = rowT[q];
    const double dz = (c * GT[q] - cs[j]) / S[j] / (1.0 + exp(-zT[q]));
#pragma unroll
    for (int d = 0; d < kMaxFeat; ++d)
      if (d < nf) acc[d] = fma(dz, (double)featsT[q * nf + d], acc[d]);
  }
  __shared__ double sm[kMaxFeat][kB / kWave];
  const int lane = lane_id(), wv = threadIdx.x / kWave;
#pragma unroll
  for (int d = 0; d < kMaxFeat; ++d) {
    const double t = wave_sum(acc[d]);
    if (lane == 0) sm[d][wv] = t;
  }
  __syncthreads();
  if ((int32_t)threadIdx.x < nf) {
    double t = 0.0;
    for (int q = 0; q < kB / kWave; ++q) t += sm[threadIdx.x][q];
    parts[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
  }
}

}  // namespace
}  // namespace tc

using namespace tc;

// ---- differentiable RWR (host)
namespace tc {
namespace {
struct PoolBuf {
  void* p = nullptr;
  hipStream_t st;
  PoolBuf(size_t bytes, hipStream_t s) : st(s) {
    p = pool_alloc(bytes ? bytes : 1, s);
    if (!p) throw Err{TC_ENOMEM, "device allocation of " + std::to_string(bytes) + " bytes failed"};
  }
  ~PoolBuf() { pool_free(p, st, false); }
  template <class T>
  T* as() const { return (T*)p; }
};

// the long columns of a pass over nnz entries (their count starts at zero)
constexpr unsigned kLongBlocks = 1024;
struct LongList {
  PoolBuf b;
  LongCols c;
  LongList(int64_t nnz, hipStream_t st) : b(256 + sizeof(int32_t) * (size_t)(nnz / kColLong + 1), st) {
    c = LongCols{b.as<uint32_t>(), (int32_t*)((char*)b.p + 256)};
    HIPC(hipMemsetAsync(b.p, 0, 4, st));
  }
};

// The power steps of W (or W^T) in the order its products work in: internal
// ids with the update written by the product (one tile), or the caller's ids
// with a product and an update.
struct Steps {
  tc_handle* h;
  double c;
  int32_t seed;  // caller's id, -1: none
  PoolBuf id;    // its internal id (one tile)
  PoolBuf tmp;   // a product (other formats)
  bool inner;
  hipStream_t st;
  Steps(tc_handle* hh, float cc, int32_t s, hipStream_t q)
      : h(hh), c((double)cc), seed(s), id(4, q), tmp(one_tile(hh) ? 1 : sizeof(float) * (size_t)hh->n_rows, q),
        inner(one_tile(hh)), st(q) {
    if (!inner) return;
    hipLaunchKernelGGL(k_set_seed, dim3(1), dim3(64), 0, st, id.as<int32_t>(), (const int32_t*)h->d_rowmap, seed);
    HIPC(hipGetLastError());
  }
  // working order -> caller's ids, or null
  const int32_t* inv() const { return inner ? h->d_rowinv : nullptr; }
  const int32_t* map() const { return inner ? h->d_rowmap : nullptr; }  // and back
  void copy(const float* v, const int32_t* perm, float* out) const {
    if (inner)
      gather_rows(v, perm, h->n_rows, 1, out, st);
    else if (h->n_rows > 0)
      HIPC(hipMemcpyAsync(out, v, sizeof(float) * h->n_rows, hipMemcpyDeviceToDevice, st));
  }
  void to_user(const float* v, float* out) const { copy(v, h->d_rowmap, out); }
  void from_user(const float* v, float* out) const { copy(v, h->d_rowinv, out); }
  // out = fl32(c fl32(A in) + (1 - c) [seed]); out may be in where the ids are the caller's
  void step(const float* in, float* out) const {
    if (inner) {
      run_tile(h, 0, RwrSpec{in, c, id.as<const int32_t>()}, out, st, tile_rest(h, true));
      h->spmv_calls++;
      return;
    }
    spmv_user(h, in, tmp.as<float>(), st);
    hipLaunchKernelGGL(k_rwr_step, dim3(nblk(h->n_rows, kB)), dim3(kB), 0, st, tmp.as<const float>(), out, h->n_rows,
                       seed, c);
    HIPC(hipGetLastError());
  }
};

// The adjoint pass: steps whose vectors are kept for one batch (whole segments),
// and floats of the rows that its passes over the entries read (0: no rows).
struct Batch {
  int32_t cap, row;
  int64_t vectors() const { return 2 * (int64_t)cap + 1 + 2 * row; }  // of n floats
};

// Scratch beyond what the caller's interval asks for: more than one segment, or
// rows of 32, only where all of it stays within this.
constexpr int64_t kBatchBytes = (int64_t)1 << 30;

// Rows of 32 (one line of 128 bytes) where they fit the bytes above, or what four
// vectors a step of a segment take; else rows of 8: at most 2 every + 17 vectors.
Batch plan_batch(int64_t n, int32_t K, int32_t seglen) {
  const int64_t room = std::max<int64_t>(kBatchBytes / (4 * std::max<int64_t>(n, 1)), 4 * (int64_t)seglen + 2);
  for (const int32_t row : {32, 8}) {
    const int64_t most = (room - 1 - 2 * row) / 2;
    if (most < seglen) continue;
    const int32_t cap = std::max<int32_t>(seglen, (int32_t)std::min<int64_t>(std::min(std::max(K, 1), 32), most));
    return Batch{cap, cap <= 8 ? 8 : row};
  }
  return Batch{seglen, 8};
}

struct BatchBufs {
  PoolBuf seg, gseg, rowr, rowg;
  BatchBufs(const Batch& b, int64_t n, bool rows, hipStream_t st)
      : seg(sizeof(float) * n * b.cap, st), gseg(sizeof(float) * n * (b.cap + 1), st),
        rowr(rows ? sizeof(float) * n * b.row : 1, st), rowg(rows ? sizeof(float) * n * b.row : 1, st) {}
};

int32_t n_checkpoints(int32_t K, int32_t every) { return K <= 0 ? 0 : (K + every - 1) / every; }
}  // namespace
}  // namespace tc

extern "C" tc_status tc_rwr_edge_weights(int64_t n_cols, int64_t nnz, const int32_t* d_col, const int64_t* d_rpT,
                                         int32_t nf, const float* d_feats, const float* d_featsT, const double* theta,
                                         double* d_zT, double* d_wT, double* d_S, float* d_val, float* d_valT,
                                         tc_stream_t stream) {
  return guarded("tc_rwr_edge_weights", [&]() -> tc_status {
    if (n_cols < 0 || nnz < 0 || nf < 1 || nf > kMaxFeat) throw Err{TC_EINVAL, "need sizes >= 0 and 1 <= nf <= 16"};
    if (!theta || !d_rpT || !d_S ||
        (nnz > 0 && (!d_col || !d_feats || !d_featsT || !d_zT || !d_wT || !d_val || !d_valT)))
      throw Err{TC_EINVAL, "NULL argument"};
    hipStream_t st = (hipStream_t)stream;
    PoolBuf th(sizeof(double) * nf, st);
    HIPC(hipMemcpyAsync(th.p, theta, sizeof(double) * nf, hipMemcpyHostToDevice, st));
    if (nnz > 0) {
      hipLaunchKernelGGL(k_edge_softplus, dim3(nblk(nnz, kB)), dim3(kB), 0, st, d_featsT, nnz, nf,
                         th.as<const double>(), d_zT, d_wT);
      HIPC(hipGetLastError());
    }
    if (n_cols > 0) {
      LongList lc(nnz, st);
      hipLaunchKernelGGL(k_col_norm<false>, dim3(nblk(nblk(n_cols, kWave / kColLanes), kWpb)), dim3(kB), 0, st, d_rpT,
                         n_cols, (const double*)d_wT, lc.c, d_S);
      HIPC(hipGetLastError());
      if (nnz > kColLong) {
        hipLaunchKernelGGL(k_col_norm<true>, dim3(kLongBlocks), dim3(kB), 0, st, d_rpT, n_cols, (const double*)d_wT,
                           lc.c, d_S);
        HIPC(hipGetLastError());
      }
    }
    if (nnz > 0) {
      PoolBuf rowT(sizeof(int32_t) * (size_t)nnz, st);
      rows_of(d_rpT, n_cols, nnz, rowT.as<int32_t>(), st);
      HIPC(hipGetLastError());
      hipLaunchKernelGGL(k_values_T, dim3(nblk(nnz, kB)), dim3(kB), 0, st, rowT.as<const int32_t>(), nnz,
                         (const double*)d_wT, (const double*)d_S, d_valT);
      HIPC(hipGetLastError());
      hipLaunchKernelGGL(k_edge_values, dim3(nblk(nnz, kB)), dim3(kB), 0, st, d_feats, d_col, nnz, nf,
                         th.as<const double>(), (const double*)d_S, d_val);
      HIPC(hipGetLastError());
      HIPC(hipStreamSynchronize(st));  // before rowT goes back to the pool
    }
    HIPC(hipStreamSynchronize(st));  // theta's staging copy is released below
    return TC_OK;
  });
}

extern "C" tc_status tc_rwr_iterates(const tc_handle* hc, int32_t seed, float c, int32_t K, int32_t every,
                                     float* d_ckpt, float* d_rK, tc_stream_t stream) {
  return guarded("tc_rwr_iterates", [&]() -> tc_status {
    if (!hc || (!d_rK && hc->n_rows > 0)) throw Err{TC_EINVAL, "NULL argument"};
    need_square(hc, "tc_rwr_iterates");
    if (K < 0 || every < 1 || !(c >= 0.0f && c <= 1.0f)) throw Err{TC_EINVAL, "need K >= 0, every >= 1, 0 <= c <= 1"};
    if (seed < 0 || seed >= hc->n_rows) throw Err{TC_EINVAL, "seed out of range"};
    if (K > 0 && !d_ckpt) throw Err{TC_EINVAL, "NULL checkpoint array"};
    tc_handle* h = const_cast<tc_handle*>(hc);
    hipStream_t st = (hipStream_t)stream;
    const int64_t n = h->n_rows;
    const Steps W(h, c, seed, st);
    // in internal ids the handle's two vectors in turn, else in place
    float *cur = W.inner ? h->d_xbuf : d_rK, *nxt = W.inner ? h->d_ybuf : d_rK;
    hipLaunchKernelGGL(k_onehot, dim3(nblk(n, kB)), dim3(kB), 0, st, d_rK, n, seed);
    HIPC(hipGetLastError());
    if (W.inner && K > 0) W.from_user(d_rK, cur);
    for (int32_t k = 0; k < K; ++k) {
      if (k % every == 0) W.to_user(cur, d_ckpt + (int64_t)(k / every) * n);
      W.step(cur, nxt);
      std::swap(cur, nxt);
    }
    if (W.inner && K > 0) W.to_user(cur, d_rK);
    return TC_OK;
  });
}

extern "C" tc_status tc_rwr_adjoint(const tc_handle* hc, const tc_handle* htc, const int64_t* d_rpT,
                                    const int32_t* d_colT, int32_t seed, float c, int32_t K, int32_t every,
                                    const float* d_ckpt, const float* d_gK, double* d_G, float* d_g0,
                                    tc_stream_t stream) {
  return guarded("tc_rwr_adjoint", [&]() -> tc_status {
    if (!hc || !htc || !d_rpT || (hc->n_rows > 0 && !d_gK)) throw Err{TC_EINVAL, "NULL argument"};
    need_square(hc, "tc_rwr_adjoint");
    need_square(htc, "tc_rwr_adjoint");
    if (htc->n_rows != hc->n_rows || htc->nnz != hc->nnz) throw Err{TC_EINVAL, "the second handle must hold A^T"};
    if (K < 0 || every < 1 || !(c >= 0.0f && c <= 1.0f)) throw Err{TC_EINVAL, "need K >= 0, every >= 1, 0 <= c <= 1"};
    if (seed < 0 || seed >= hc->n_rows) throw Err{TC_EINVAL, "seed out of range"};
    const int64_t n = hc->n_rows, nnz = hc->nnz;
    if (nnz > 0 && (!d_colT || !d_G)) throw Err{TC_EINVAL, "NULL argument"};
    if (K > 0 && !d_ckpt) throw Err{TC_EINVAL, "NULL checkpoint array"};
    tc_handle* h = const_cast<tc_handle*>(hc);
    tc_handle* ht = const_cast<tc_handle*>(htc);
    hipStream_t st = (hipStream_t)stream;
    const Steps W(h, c, seed, st), Wt(ht, c, -1, st);
    const int32_t seglen = std::min(every, std::max(K, 1));
    PoolBuf rows(sizeof(int32_t) * (size_t)std::max<int64_t>(nnz, 1), st);
    Batch batch = plan_batch(n, K, seglen);
    std::unique_ptr<BatchBufs> bufs;
    try {
      bufs = std::make_unique<BatchBufs>(batch, n, nnz > 0, st);
    } catch (const Err& e) {  // what one segment cannot do without
      if (e.st != TC_ENOMEM) throw;
      batch = Batch{seglen, 0};
      bufs = std::make_unique<BatchBufs>(batch, n, nnz > 0, st);
    }
    const int32_t cap = batch.cap, row = batch.row;
    if (nnz > 0) {
      rows_of(d_rpT, n, nnz, rows.as<int32_t>(), st);
      HIPC(hipGetLastError());
    }
    // steps in S and GS, latest first; GS's next slot holds the current g
    float *S = bufs->seg.as<float>(), *GS = bufs->gseg.as<float>();
    float *rowr = bufs->rowr.as<float>(), *rowg = bufs->rowg.as<float>();
    Wt.from_user(d_gK, GS);
    int32_t have = 0;
    bool first = true;
    auto flush = [&]() {
      if (row == 0 && have > 0 && nnz > 0) {
        hipLaunchKernelGGL(first ? k_edge_accum_vec<true> : k_edge_accum_vec<false>, dim3(nblk(nnz, kB)), dim3(kB), 0,
                           st, d_colT, rows.as<const int32_t>(), nnz, (const float*)GS, (const float*)S, Wt.map(),
                           W.map(), n, have, d_G);
        HIPC(hipGetLastError());
        first = false;
        return;
      }
      for (int32_t b = 0; b < have && nnz > 0; b += row) {
        const int32_t m = std::min(row, have - b);
        auto put = row == 8 ? k_step_rows<8> : k_step_rows<32>;
        hipLaunchKernelGGL(put, dim3(nblk(n, kB)), dim3(kB), 0, st, (const float*)(GS + (int64_t)b * n), m, n,
                           Wt.inv(), rowg);
        HIPC(hipGetLastError());
        hipLaunchKernelGGL(put, dim3(nblk(n, kB)), dim3(kB), 0, st, (const float*)(S + (int64_t)b * n), m, n, W.inv(),
                           rowr);
        HIPC(hipGetLastError());
        auto sum = row == 8 ? (first ? k_edge_accum<8, true> : k_edge_accum<8, false>)
                            : (first ? k_edge_accum<32, true> : k_edge_accum<32, false>);
        hipLaunchKernelGGL(sum, dim3(nblk(nnz, kB)), dim3(kB), 0, st, d_colT, rows.as<const int32_t>(), nnz,
                           (const float*)rowg, (const float*)rowr, m, d_G);
        HIPC(hipGetLastError());
        first = false;
      }
    };
    for (int32_t q = n_checkpoints(K, every) - 1; q >= 0; --q) {
      const int32_t k0 = q * every, m = std::min(K, k0 + every) - k0;
      if (have + m > cap) {
        flush();
        HIPC(hipMemcpyAsync(GS, GS + (int64_t)have * n, sizeof(float) * n, hipMemcpyDeviceToDevice, st));
        have = 0;
      }
      // r^k at slot have + (k0 + m - 1 - k), recomputed from the checkpoint, which
      // is the segment's last slot
      float* end = S + (int64_t)(have + m - 1) * n;
      W.from_user(d_ckpt + (int64_t)q * n, end);
      for (int32_t t = 1; t < m; ++t) W.step(end - (int64_t)(t - 1) * n, end - (int64_t)t * n);
      // g^{k+1} likewise; its product is g^k (g^0 only where it is asked for)
      const int32_t steps = q == 0 && !d_g0 ? m - 1 : m;
      for (int32_t t = 0; t < steps; ++t) Wt.step(GS + (int64_t)(have + t) * n, GS + (int64_t)(have + t + 1) * n);
      have += m;
    }
    flush();
    if (nnz > 0 && first) HIPC(hipMemsetAsync(d_G, 0, sizeof(double) * nnz, st));
    if (d_g0) Wt.to_user(GS + (int64_t)have * n, d_g0);
    return TC_OK;
  });
}

extern "C" tc_status tc_rwr_theta_grad(int64_t n_cols, int64_t nnz, const int64_t* d_rpT, int32_t nf,
                                       const float* d_featsT, const double* d_zT, const double* d_wT,
                                       const double* d_S, const double* d_G, float c, double* dtheta,
                                       tc_stream_t stream) {
  return guarded("tc_rwr_theta_grad", [&]() -> tc_status {
    if (n_cols < 0 || nnz < 0 || nf < 1 || nf > kMaxFeat) throw Err{TC_EINVAL, "need sizes >= 0 and 1 <= nf <= 16"};
    if (!dtheta || !d_rpT || !d_S || (nnz > 0 && (!d_featsT || !d_zT || !d_wT || !d_G)))
      throw Err{TC_EINVAL, "NULL argument"};
    hipStream_t st = (hipStream_t)stream;
    PoolBuf cs(sizeof(double) * (size_t)std::max<int64_t>(n_cols, 1), st),
        rowT(sizeof(int32_t) * (size_t)std::max<int64_t>(nnz, 1), st),
        parts(sizeof(double) * (size_t)kGradBlocks * nf, st), out(sizeof(double) * nf, st);
    if (n_cols > 0) {
      LongList lc(nnz, st);
      hipLaunchKernelGGL(k_col_dot<false>, dim3(nblk(nblk(n_cols, kWave / kColLanes), kWpb)), dim3(kB), 0, st, d_rpT,
                         n_cols, d_G, d_wT, d_S, (double)c, lc.c, cs.as<double>());
      HIPC(hipGetLastError());
      if (nnz > kColLong) {
        hipLaunchKernelGGL(k_col_dot<true>, dim3(kLongBlocks), dim3(kB), 0, st, d_rpT, n_cols, d_G, d_wT, d_S,
                           (double)c, lc.c, cs.as<double>());
        HIPC(hipGetLastError());
      }
      if (nnz > 0) rows_of(d_rpT, n_cols, nnz, rowT.as<int32_t>(), st);
      HIPC(hipGetLastError());
    }
    hipLaunchKernelGGL(k_theta_grad, dim3(kGradBlocks), dim3(kB), 0, st, rowT.as<const int32_t>(), nnz, nf, d_featsT,
                       d_zT, d_S, d_G, cs.as<const double>(), (double)c, parts.as<double>());
    HIPC(hipGetLastError());
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kB), 0, st, parts.as<const double>(), kGradBlocks, nf,
                       out.as<double>());
    HIPC(hipGetLastError());
    HIPC(hipMemcpyAsync(dtheta, out.p, sizeof(double) * nf, hipMemcpyDeviceToHost, st));
    HIPC(hipStreamSynchronize(st));
    return TC_OK;
  });
}

// dst row q = src row idx[q] (rows of `width` floats); idx is checked against
// the source's n_src rows first
__global__ void k_idx_check(const int32_t* __restrict__ idx, int64_t n, int64_t n_src, int32_t* __restrict__ bad) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n && (idx[q] < 0 || idx[q] >= n_src)) atomicOr(bad, 1);
}

extern "C" tc_status tc_gather_rows(const float* d_src, int64_t n_src, const int32_t* d_idx, int64_t n, int32_t width,
                                    float* d_dst, tc_stream_t stream) {
  return guarded("tc_gather_rows", [&]() -> tc_status {
    if (n < 0 || n_src < 0 || width < 1) throw Err{TC_EINVAL, "need n, n_src >= 0 and width >= 1"};
    if (n == 0) return TC_OK;
    if (!d_src || !d_idx || !d_dst) throw Err{TC_EINVAL, "NULL argument"};
    hipStream_t st = (hipStream_t)stream;
    PoolBuf bad(sizeof(int32_t), st);
    HIPC(hipMemsetAsync(bad.p, 0, sizeof(int32_t), st));
    hipLaunchKernelGGL(k_idx_check, dim3(nblk(n, kB)), dim3(kB), 0, st, d_idx, n, n_src, bad.as<int32_t>());
    HIPC(hipGetLastError());
    int32_t hbad = 0;
    HIPC(hipMemcpyAsync(&hbad, bad.p, sizeof(int32_t), hipMemcpyDeviceToHost, st));
    HIPC(hipStreamSynchronize(st));
    if (hbad) throw Err{TC_EINVAL, "row index out of range"};
    gather_rows(d_src, d_idx, n, width, d_dst, st);
    HIPC(hipStreamSynchronize(st));
    return TC_OK;
  });
}
