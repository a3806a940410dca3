// The power iterations on a built handle (Appendix F): PageRank (Eq. 6), HITS
// (Eq. 7-8) and RWR (Eq. 9), with their vector updates and reductions in FP64;
// one-tile formats and row panels write PageRank's update, and one-tile formats
// RWR's restart, from the product itself.
#include <algorithm>
#include <cmath>
#include <vector>

#include "tc_tile.h"

namespace tc {

namespace {

// Blocks of the reductions.  Partial sums that the next launch adds itself:
// 64 where every wavefront does (wave_parts), kB where a block does; and no
// more blocks draw a ticket, since 1024 of them took 19 us at one address.
constexpr int kSumBlocks = kB;
constexpr int kDangBlocks = 64;

// PageRank update (Eq. 6 with uniform dangling mass), fused with the L1
// change and the dangling mass of the new iterate:
//   p'_i = c (y_i + d/n) + (1-c)/n
// (ypriv, G): private copies of y of the XCD schedule still to be added, in
// g order, to y (G = 0 when there are none).
__global__ void __launch_bounds__(kB) k_pr_update(const float* __restrict__ y, const float* __restrict__ ypriv,
                                                  int32_t G, float* __restrict__ p, int64_t n, int64_t dang_begin,
                                                  double c, const double* __restrict__ dmass,
                                                  double* __restrict__ parts) {
  const double dn = *dmass / (double)n;
  const double tele = (1.0 - c) / (double)n;
  double v[2] = {0.0, 0.0};
  for (int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kB) {
    float yi = y[i];
    if (G > 0) {
      double s = (double)yi;
      for (int32_t g = 0; g < G; ++g) s += (double)ypriv[(int64_t)g * n + i];
      yi = (float)s;
    }
    const float pn = (float)(c * ((double)yi + dn) + tele);
    v[0] += fabs((double)pn - (double)p[i]);
    if (i >= dang_begin) v[1] += (double)pn;
    p[i] = pn;
  }
  block_sum_store<2>(v, parts + blockIdx.x, gridDim.x);
}

// PageRank start: p = 1/n, and its dangling mass nd v as the only partial sum
// (nd equal floats: their sum in FP64 is exact) and as mass
__global__ void k_pr_init(float* __restrict__ p, int64_t n, float v, double nd, double* __restrict__ dparts,
                          double* __restrict__ mass, uint32_t* __restrict__ ticket) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
  if (i < 64) dparts[i] = i == 0 ? nd * (double)v : 0.0;
  if (i == 0) {
    *mass = nd * (double)v;
    *ticket = 0;
  }
}

// Dangling mass of the new iterate by the first nd blocks (partial sums to
// dparts, added where they are used) and, by the others (if any), its L1
// change from the old one, final in this launch, in *res and *host.
__global__ void __launch_bounds__(kB) k_pr_sums(const float* __restrict__ pn, const float* __restrict__ pc, int64_t n,
                                                int64_t dang_begin, int32_t nd, double* __restrict__ dparts,
                                                double* __restrict__ parts, uint32_t* __restrict__ ticket,
                                                double* __restrict__ res, double* host) {
  const bool dang = (int32_t)blockIdx.x < nd;
  const int64_t step = (int64_t)(dang ? nd : (int32_t)gridDim.x - nd) * kB;
  const int64_t b = dang ? dang_begin + (int64_t)blockIdx.x * kB : (int64_t)((int32_t)blockIdx.x - nd) * kB;
  double v = 0.0;
  for (int64_t i0 = b + threadIdx.x; i0 < n; i0 += 8 * step) {
    float s[8], t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {  // eight elements in flight (past the end: the first, not added)
      const int64_t i = i0 + u * step < n ? i0 + u * step : i0;
      s[u] = pn[i];
      t[u] = dang ? 0.0f : pc[i];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v += i0 + u * step >= n ? 0.0 : dang ? (double)s[u] : fabs((double)s[u] - (double)t[u]);
  }
  v = block_sum(v);
  if ((int32_t)blockIdx.x < nd && threadIdx.x == 0) dparts[blockIdx.x] = v;
  if ((int32_t)gridDim.x == nd || !last_block(parts, v, ticket)) return;
  const double r = sum_parts(parts, nd, gridDim.x);
  if (threadIdx.x == 0) {
    *res = r;
    if (host) __hip_atomic_store(host, r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// HITS start: x = 1/n, the half of every internal id, the error flag and the ticket
__global__ void k_hits_init(float* __restrict__ x, const int32_t* __restrict__ rowinv, int64_t n2, int64_t n, float v,
                            uint8_t* __restrict__ half, double* __restrict__ res, uint32_t* __restrict__ ticket) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n2) {
    x[i] = v;
    half[i] = rowinv[i] >= n ? 1 : 0;
  }
  if (i == 0) {
    res[1] = 0.0;
    *ticket = 0;
  }
}

// HITS: partial sums of the two halves of y, authorities to parts[block], hubs
// to parts[kSumBlocks + block]; added where they are used
__global__ void __launch_bounds__(kB) k_hits_sums(const float* __restrict__ y, const uint8_t* __restrict__ half,
                                                  int64_t n2, double* __restrict__ parts) {
  double a = 0.0, h = 0.0;
  const int64_t step = (int64_t)gridDim.x * kB;
  for (int64_t i0 = (int64_t)blockIdx.x * kB + threadIdx.x; i0 < n2; i0 += 8 * step) {
    float t[8];
    uint8_t f[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {  // eight elements in flight (past the end: the first, not added)
      t[u] = y[i0 + u * step < n2 ? i0 + u * step : i0];
      f[u] = half[i0 + u * step < n2 ? i0 + u * step : i0];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double v = i0 + u * step < n2 ? (double)t[u] : 0.0;
      a += f[u] ? 0.0 : v;
      h += f[u] ? v : 0.0;
    }
  }
  a = block_sum(a);
  h = block_sum(h);
  if (threadIdx.x == 0) {
    parts[blockIdx.x] = a;
    parts[kSumBlocks + blockIdx.x] = h;
  }
}

// HITS: x' = y / (sum of its half), from the partial sums of np blocks; RES:
// the L1 change, final in this launch (res[0]; the change and the zero-sum
// flag res[1] also to host[0..1])
template <bool RES>
__global__ void __launch_bounds__(kB) k_hits_update(const float* __restrict__ y, float* __restrict__ x,
                                                    const uint8_t* __restrict__ half, int64_t n2,
                                                    const double* __restrict__ sums, int np,
                                                    double* __restrict__ parts, uint32_t* __restrict__ ticket,
                                                    double* __restrict__ res, double* host) {
  const double sa = block_sum((int)threadIdx.x < np ? sums[threadIdx.x] : 0.0);
  const double sh = block_sum((int)threadIdx.x < np ? sums[kSumBlocks + threadIdx.x] : 0.0);
  const bool zero = sa == 0.0 || sh == 0.0;
  if (zero && blockIdx.x == 0 && threadIdx.x == 0) res[1] = 1.0;
  double v = 0.0;
  const int64_t step = (int64_t)gridDim.x * kB;
  for (int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x; i < n2; i += step) {
    const double s = half[i] ? sh : sa;
    const float xn = s != 0.0 ? (float)((double)y[i] / s) : 0.0f;
    if (RES) v += fabs((double)xn - (double)x[i]);
    x[i] = xn;
  }
  if (!RES) return;
  if (!last_block(parts, block_sum(v), ticket)) return;
  v = sum_parts(parts, 0, gridDim.x);
  if (threadIdx.x == 0) {
    res[0] = v;
    if (host) {
      __hip_atomic_store(host, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(host + 1, zero ? 1.0 : res[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

// Fused PageRank step with row panels, the split rows: their unsplit
// segments' sum (yraw, from the panel pass) plus their chunks, then the same
// formula as the panel pass; the rows without entries were written by it.
__global__ void __launch_bounds__(kB) k_pr_split_panel(const SplitRow* __restrict__ sr, int64_t n_split,
                                                        const double* __restrict__ partial,
                                                        const float* __restrict__ yraw, float* __restrict__ pn,
                                                        double c, const double* __restrict__ dparts, int32_t nd,
                                                        int64_t n) {
  // one wavefront per split row
  const int lane = lane_id();
  const int64_t t = (int64_t)blockIdx.x * kWpb + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (t >= n_split) return;
  __shared__ double buf[kWpb][4 * kWave];
  const SplitRow s = sr[t];
  const double mass = wave_parts(dparts, nd);
  const double acc = sum_slots_wave(partial + s.slot_begin, s.n_slots, lane, buf[threadIdx.x / kWave]);
  if (lane == 0) {
    const double dn = mass / (double)n, tele = (1.0 - c) / (double)n;
    const float yv = (float)((double)yraw[t] + acc);
    pn[s.row] = (float)(c * ((double)yv + dn) + tele);
  }
}

// RWR: R' = c Y + (1-c) E, per-column L1 change (nq columns of k at q0)
__global__ void __launch_bounds__(kB) k_rwr_update(const float* __restrict__ Y, float* __restrict__ R, int64_t n,
                                                   int32_t k, double c, const int32_t* __restrict__ seeds,
                                                   double* __restrict__ parts, int nblocks) {
  // thread layout: each thread owns one column q (threadIdx.x % k) of rows
  // spaced by the grid; k <= 256
  const int32_t q = threadIdx.x % k;
  const int32_t rpb = kB / k;  // rows per block step
  const int32_t rr = threadIdx.x / k;
  __shared__ double sm[kB];
  double s = 0.0;
  if (rr < rpb) {
    const int32_t seed = seeds[q];
    const int64_t step = (int64_t)gridDim.x * rpb;
    for (int64_t i0 = (int64_t)blockIdx.x * rpb + rr; i0 < n; i0 += 4 * step) {
      float y[4], r[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {  // four rows' loads together (past n: row i0, not used)
        const int64_t e = (i0 + u * step < n ? i0 + u * step : i0) * k + q;
        y[u] = Y[e];
        r[u] = R[e];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t i = i0 + u * step;
        if (i < n) {
          const float rn = (float)(c * (double)y[u] + (i == seed ? (1.0 - c) : 0.0));
          s += fabs((double)rn - (double)r[u]);
          R[i * k + q] = rn;
        }
      }
    }
  }
  sm[threadIdx.x] = s;
  __syncthreads();
  if ((int32_t)threadIdx.x < k) {
    double t = 0.0;
    for (int32_t u = 0; u < rpb; ++u) t += sm[u * k + threadIdx.x];
    parts[(int64_t)threadIdx.x * nblocks + blockIdx.x] = t;
  }
}

// per-column L1 change from Ra to Rb (the restart is in the product)
__global__ void __launch_bounds__(kB) k_rwr_change(const float* __restrict__ Ra, const float* __restrict__ Rb,
                                                   int64_t n, int32_t k, double* __restrict__ parts, int nblocks) {
  const int32_t q = threadIdx.x % k, rpb = kB / k, rr = threadIdx.x / k;  // as in k_rwr_update
  __shared__ double sm[kB];
  double s = 0.0;
  if (rr < rpb) {
    const int64_t step = (int64_t)gridDim.x * rpb;
    for (int64_t i0 = (int64_t)blockIdx.x * rpb + rr; i0 < n; i0 += 8 * step) {
      float a[8], b[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {  // eight rows' loads together (past n: row i0, no change)
        const int64_t e = (i0 + u * step < n ? i0 + u * step : i0) * k + q;
        a[u] = Ra[e];
        b[u] = Rb[e];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) s += i0 + u * step < n ? fabs((double)a[u] - (double)b[u]) : 0.0;
    }
  }
  sm[threadIdx.x] = s;
  __syncthreads();
  if ((int32_t)threadIdx.x < k) {
    double t = 0.0;
    for (int32_t u = 0; u < rpb; ++u) t += sm[u * k + threadIdx.x];
    parts[(int64_t)threadIdx.x * nblocks + blockIdx.x] = t;
  }
}

// Largest over k columns of each column's partial sums (np of them), one
// wavefront per column; the largest final in this launch, also to *host.
__global__ void __launch_bounds__(kB) k_cols_max(const double* __restrict__ parts, int np, int32_t k,
                                                 double* __restrict__ best, uint32_t* __restrict__ ticket,
                                                 double* __restrict__ out, double* host) {
  const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int32_t q = (int32_t)blockIdx.x * kWpb + wv;
  __shared__ double sm[kWpb];
  double s = 0.0;
  if (q < k) {
    const double* pq = parts + (int64_t)q * np;
    for (int i0 = lane; i0 < np; i0 += 8 * kWave) {  // eight loads in flight (past the end: pq[0], not added)
      double t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = pq[i0 + u * kWave < np ? i0 + u * kWave : 0];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += i0 + u * kWave < np ? t[u] : 0.0;
    }
    s = wave_sum(s);
  }
  if (lane == 0) sm[wv] = s;
  __syncthreads();
  double m = 0.0;
  for (int w = 0; w < kWpb; ++w) m = fmax(m, sm[w]);
  if (!last_block(best, m, ticket) || threadIdx.x != 0) return;
  m = 0.0;
  for (int b = 0; b < (int)gridDim.x; ++b)
    m = fmax(m, __hip_atomic_load(best + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  *out = m;
  if (host) __hip_atomic_store(host, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ void k_zero(v4f* __restrict__ a, int64_t n4) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n4) a[i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
}

// The seeds' internal ids, R = their one-hot rows (R is zero), the ticket
struct SeedArg {
  int32_t s[kB];
};
__global__ void __launch_bounds__(kB) k_rwr_seeds(SeedArg seeds, const int32_t* __restrict__ map, int32_t k,
                                                  int32_t* __restrict__ out, float* __restrict__ R,
                                                  uint32_t* __restrict__ ticket) {
  const int32_t q = threadIdx.x;
  if (q < k) {
    const int32_t i = map[seeds.s[q]];
    out[q] = i;
    R[(int64_t)i * k + q] = 1.0f;
  }
  if (q == 0) *ticket = 0;
}

}  // namespace
}  // namespace tc

using namespace tc;

extern "C" tc_status tc_pagerank(const tc_handle* hc, float c, float tol, int32_t max_iter, int32_t check_every,
                                 float* p_out, int32_t* iters, double* resid, tc_stream_t stream) {
  return guarded("tc_pagerank", [&]() -> tc_status {
    if (!hc || (!p_out && hc->n_rows > 0)) throw Err{TC_EINVAL, "NULL argument"};
    if (!(c >= 0.0f && c <= 1.0f) || max_iter < 0) throw Err{TC_EINVAL, "need 0 <= c <= 1 and max_iter >= 0"};
    need_square(hc, "tc_pagerank");
    tc_handle* h = const_cast<tc_handle*>(hc);
    hipStream_t st = (hipStream_t)stream;
    const int64_t n = h->n_rows;
    if (check_every < 1) check_every = 1;
    float* p = h->d_xbuf;
    float* y = h->d_ybuf;
    double* parts = h->d_red;                  // 2 * kRedBlocks
    double* res = h->d_red + 2 * kRedBlocks;   // [resid, dangling mass]
    uint32_t* ticket = (uint32_t*)(res + 2);
    double* dparts = res + 8;                  // kDangBlocks
    int32_t it = 0;
    double r = 0.0;
    bool conv = false;
    if (n > 0) {
      HostResult change(res, st);
      hipLaunchKernelGGL(k_pr_init, dim3(nblk(n, kB)), dim3(kB), 0, st, p, n, (float)(1.0 / (double)n),
                         (double)h->n_dangling, dparts, res + 1, ticket);
      HIPC(hipGetLastError());
      const bool xcd = h->xcd_groups > 0 && h->n_tiles > 1;
      const int32_t G = xcd ? h->n_tiles - 1 : 0;
      // One tile and row panels: every iteration writes the update from the
      // product into the other buffer; the dangling mass of the new iterate and,
      // where it is read, its change come from a pass over the two.  The other
      // formats run the product into the other buffer, then the update in place.
      const bool fuse = one_tile(h) || h->n_panels > 0;
      const int32_t nd = (int32_t)std::min<int64_t>(nblk(h->n_dangling, 2 * kB), kDangBlocks);
      const int32_t nr = (int32_t)std::min<int64_t>(nblk(n, 4 * kB), kSumBlocks);
      float* buf[2] = {p, y};
      bool zero_rows = false;  // y's rows without entries hold 0 (formats whose buffers stay)
      int cur = 0;
      for (it = 0; it < max_iter;) {
        const bool need_res = it + 1 == max_iter || (tol > 0.0f && (it + 1) % check_every == 0);
        float* pc = buf[cur];
        float* pn = buf[1 - cur];
        if (fuse) {
          if (h->n_panels > 0) {
            const PanelPr pr{(double)c, (const double*)dparts, kDangBlocks, n, (const int64_t*)h->d_panel_split_begin,
                             (const SplitRow*)h->d_split, h->d_panel_yraw};
            panel_pass(h, pc, pn, st, &pr);
            if (h->n_split_rows > 0) {
              hipLaunchKernelGGL(k_pr_split_panel, dim3(nblk(h->n_split_rows, kWpb)), dim3(kB), 0, st, h->d_split,
                                 h->n_split_rows, (const double*)h->d_partial, (const float*)h->d_panel_yraw, pn,
                                 (double)c, (const double*)dparts, (int32_t)kDangBlocks, n);
              HIPC(hipGetLastError());
            }
          } else {
            run_tile(h, 0, PrSpec{pc, (double)c, dparts, kDangBlocks, n}, pn, st, tile_rest(h, true));
          }
          if (nd > 0 || need_res) {
            hipLaunchKernelGGL(k_pr_sums, dim3(nd + (need_res ? nr : 0)), dim3(kB), 0, st, (const float*)pn,
                               (const float*)pc, n, n - h->n_dangling, nd, dparts, parts, ticket, res,
                               need_res ? change.h() : nullptr);
            HIPC(hipGetLastError());
          }
          h->spmv_calls++;
          cur = 1 - cur;
        } else {
          spmv_internal(h, pc, pn, st, xcd, zero_rows);
          zero_rows = true;
          hipLaunchKernelGGL(k_pr_update, dim3(kRedBlocks), dim3(kB), 0, st, (const float*)pn,
                             (const float*)h->d_ypriv, G, pc, n, n - h->n_dangling, (double)c,
                             (const double*)(res + 1), parts);
          HIPC(hipGetLastError());
          hipLaunchKernelGGL(k_finish, dim3(1), dim3(kB), 0, st, (const double*)parts, kRedBlocks, 2, res);
          HIPC(hipGetLastError());
        }
        ++it;
        if (tol > 0.0f && need_res) {
          r = fuse ? change.read() : read_f64(res, st);
          if (r <= (double)tol) {
            conv = true;
            break;
          }
        }
      }
      // the residual of the last iteration (every loop end has it queued)
      gather_rows(buf[cur], h->d_rowmap, n, 1, p_out, st);
      if (it > 0 && !(tol > 0.0f)) r = fuse ? change.read() : read_f64(res, st);
    }
    if (iters) *iters = it;
    if (resid) *resid = r;
    if (tol > 0.0f && !conv && n > 0) {
      set_error("tc_pagerank: tolerance not reached in max_iter iterations");
      return TC_ENOTCONV;
    }
    return TC_OK;
  });
}

extern "C" tc_status tc_hits(const tc_handle* hc, float tol, int32_t max_iter, int32_t check_every, float* auth,
                             float* hub, int32_t* iters, double* resid, tc_stream_t stream) {
  return guarded("tc_hits", [&]() -> tc_status {
    if (!hc || ((!auth || !hub) && hc->n_rows > 0)) throw Err{TC_EINVAL, "NULL argument"};
    if (max_iter < 0) throw Err{TC_EINVAL, "max_iter < 0"};
    need_square(hc, "tc_hits");
    if (hc->n_rows % 2) throw Err{TC_EINVAL, "the HITS matrix must be 2n x 2n"};
    tc_handle* h = const_cast<tc_handle*>(hc);
    hipStream_t st = (hipStream_t)stream;
    const int64_t n2 = h->n_rows, n = n2 / 2;
    if (check_every < 1) check_every = 1;
    float* x = h->d_xbuf;
    float* y = h->d_ybuf;
    double* parts = h->d_red;
    double* sums = h->d_red + kRedBlocks;           // 2 * kSumBlocks partial sums
    double* res = h->d_red + 2 * kRedBlocks;        // [resid, a sum was zero]
    uint32_t* ticket = (uint32_t*)(res + 2);
    uint8_t* half = (uint8_t*)workspace(h, (size_t)std::max<int64_t>(n2, 1), st);
    int32_t it = 0;
    double r = 0.0;
    bool conv = false;
    if (n2 > 0) {
      HostResult result(res, st);
      hipLaunchKernelGGL(k_hits_init, dim3(nblk(n2, kB)), dim3(kB), 0, st, x, (const int32_t*)h->d_rowinv, n2, n,
                         (float)(1.0 / (double)n), half, res, ticket);
      HIPC(hipGetLastError());
      const unsigned nb = (unsigned)std::min<int64_t>(nblk(n2, 4 * kB), kSumBlocks);
      const unsigned ub = (unsigned)std::min<int64_t>(nblk(n2, 4 * kB), 2 * kRedBlocks);  // update without the change
      double zero_sum = 0.0;
      // the change and the zero-sum flag of the iterations so far
      auto read_back = [&]() {
        r = result.read();
        zero_sum = result.b.pinned ? ((volatile double*)result.b.p)[1] : read_f64(res + 1, st);
      };
      bool zero_rows = false;
      for (it = 0; it < max_iter;) {
        const bool check = tol > 0.0f && (it + 1) % check_every == 0;
        const bool need_res = it + 1 == max_iter || check;
        spmv_internal(h, x, y, st, false, zero_rows);
        zero_rows = !(h->xcd_groups > 0 && h->n_tiles > 1);  // nothing else writes y
        hipLaunchKernelGGL(k_hits_sums, dim3(nb), dim3(kB), 0, st, (const float*)y, (const uint8_t*)half, n2, sums);
        HIPC(hipGetLastError());
        hipLaunchKernelGGL(need_res ? k_hits_update<true> : k_hits_update<false>, dim3(need_res ? nb : ub), dim3(kB), 0, st,
                           (const float*)y, x, (const uint8_t*)half, n2, (const double*)sums, (int)nb, parts, ticket, res,
                           need_res ? result.h() : nullptr);
        HIPC(hipGetLastError());
        ++it;
        if (need_res && tol > 0.0f) {
          read_back();
          if (r <= (double)tol) {
            conv = true;
            break;
          }
        }
      }
      if (it > 0 && !(tol > 0.0f)) read_back();
      if (zero_sum != 0.0) throw Err{TC_EINVAL, "a half of the iterate sums to zero (graph without edges?)"};
      gather_rows(x, h->d_rowmap, n, 1, auth, st);
      gather_rows(x, h->d_rowmap + n, n, 1, hub, st);
    }
    if (iters) *iters = it;
    if (resid) *resid = r;
    if (tol > 0.0f && !conv && n2 > 0) {
      set_error("tc_hits: tolerance not reached in max_iter iterations");
      return TC_ENOTCONV;
    }
    return TC_OK;
  });
}

extern "C" tc_status tc_rwr(const tc_handle* hc, const int32_t* seeds, int32_t k, float c, float tol,
                            int32_t max_iter, int32_t check_every, float* R_out, int32_t* iters, double* resid,
                            tc_stream_t stream) {
  return guarded("tc_rwr", [&]() -> tc_status {
    if (!hc || !seeds || (!R_out && hc->n_rows > 0)) throw Err{TC_EINVAL, "NULL argument"};
    if (k < 1 || k > 256) throw Err{TC_EINVAL, "k must be in [1, 256]"};
    if (!(c >= 0.0f && c <= 1.0f) || max_iter < 0) throw Err{TC_EINVAL, "need 0 <= c <= 1 and max_iter >= 0"};
    need_square(hc, "tc_rwr");
    tc_handle* h = const_cast<tc_handle*>(hc);
    hipStream_t st = (hipStream_t)stream;
    const int64_t n = h->n_rows;
    for (int32_t q = 0; q < k; ++q)
      if (seeds[q] < 0 || seeds[q] >= n) throw Err{TC_EINVAL, "seed out of range"};
    if (check_every < 1) check_every = 1;
    // blocks of the change (one partial per block and column)
    const int nb = (int)std::min<int64_t>(2048, nblk(std::max<int64_t>(n, 1), 8 * std::max(kB / k, 1)));
    const size_t vb = ((sizeof(float) * (size_t)n * k + 255) / 256) * 256;
    const size_t need = 2 * vb + sizeof(double) * ((size_t)nb * k + k + 8) + sizeof(int32_t) * k;
    char* ws = (char*)workspace(h, need, st);
    float* Rm = (float*)ws;
    float* Ym = (float*)(ws + vb);
    double* parts = (double*)(ws + 2 * vb);
    double* best = parts + (size_t)nb * k;
    double* mx = best + k;
    uint32_t* ticket = (uint32_t*)(mx + 1);
    int32_t* dseeds = (int32_t*)(mx + 8);
    int32_t it = 0;
    double r = 0.0;
    bool conv = false;
    if (n > 0) {
      HostResult change(mx, st);
      SeedArg sa;
      std::copy(seeds, seeds + k, sa.s);
      hipLaunchKernelGGL(k_zero, dim3(nblk((int64_t)(vb / 16), kB)), dim3(kB), 0, st, (v4f*)Rm, (int64_t)(vb / 16));
      HIPC(hipGetLastError());
      hipLaunchKernelGGL(k_rwr_seeds, dim3(1), dim3(kB), 0, st, sa, (const int32_t*)h->d_rowmap, k, dseeds, Rm,
                         ticket);
      HIPC(hipGetLastError());
      // One tile: every iteration writes the restart from the product into the
      // other buffer, and the change, where it is read, comes from a pass over
      // the two.  Several tiles (and one query on TILE-COO): the product, then
      // the update in place with its per-column change.
      const bool fuse = h->n_tiles == 1 && h->xcd_groups == 0 && (k > 1 || one_tile(h));
      const RwrEpi epi{(double)c, dseeds};
      float* buf[2] = {Rm, Ym};
      bool rest[2] = {false, false};  // the buffer's rows without entries hold what this loop writes there
      int cur = 0;
      for (it = 0; it < max_iter;) {
        const bool need_res = it + 1 == max_iter || (tol > 0.0f && (it + 1) % check_every == 0);
        float* Rcur = buf[cur];
        float* Yb = buf[1 - cur];
        if (fuse && k > 1) {
          spmm_internal(h, Rcur, Yb, k, st, rest[1 - cur], &epi);
        } else if (fuse) {
          run_tile(h, 0, RwrSpec{Rcur, (double)c, dseeds}, Yb, st, tile_rest(h, !rest[1 - cur]));
          h->spmv_calls++;
        } else if (k == 1) {
          spmv_internal(h, Rcur, Yb, st, false, rest[1 - cur]);
        } else {
          spmm_internal(h, Rcur, Yb, k, st, rest[1 - cur]);
        }
        rest[1 - cur] = true;
        if (!fuse) {
          hipLaunchKernelGGL(k_rwr_update, dim3(nb), dim3(kB), 0, st, (const float*)Yb, Rcur, n, k, (double)c,
                             (const int32_t*)dseeds, parts, nb);
          HIPC(hipGetLastError());
        } else {
          if (need_res) {
            hipLaunchKernelGGL(k_rwr_change, dim3(nb), dim3(kB), 0, st, (const float*)Rcur, (const float*)Yb, n, k,
                               parts, nb);
            HIPC(hipGetLastError());
          }
          cur = 1 - cur;
        }
        if (need_res) {
          hipLaunchKernelGGL(k_cols_max, dim3(nblk(k, kWpb)), dim3(kB), 0, st, (const double*)parts, nb, k, best,
                             ticket, mx, change.h());
          HIPC(hipGetLastError());
        }
        ++it;
        if (tol > 0.0f && need_res) {
          r = change.read();
          if (r <= (double)tol) {
            conv = true;
            break;
          }
        }
      }
      gather_rows(buf[cur], h->d_rowmap, n, k, R_out, st);
      if (it > 0 && !(tol > 0.0f)) r = change.read();
    }
    if (iters) *iters = it;
    if (resid) *resid = r;
    if (tol > 0.0f && !conv && n > 0) {
      set_error("tc_rwr: tolerance not reached in max_iter iterations");
      return TC_ENOTCONV;
    }
    return TC_OK;
  });
}
