// rounds.hip -- per-query bookkeeping of the batched LO-RANSAC rounds (ImLoc
// Sec. 3.3: batches of minimal sets; stop after the sample cap or once the
// probability of having missed the best model is small), plus small utility
// kernels.  One thread per query unless noted.
#include "imloc_device.h"
#include "imloc_kernels.h"

#include <algorithm>

namespace imloc {

__global__ void fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

// Samples of the coming round: the rest of the budget, at most one batch;
// none once the query stopped.
__device__ inline int64_t round_samples(const QueryDesc& d, const BestState& b) {
  if (!b.active) return 0;
  const int64_t left = d.total - b.drawn;
  return left < d.batch ? left : d.batch;
}

// The start of a call (of a round, in a server): one launch brings the table
// and the rigs from (pinned) host memory, gathers the scoring subsets, clears the
// mailboxes and resets the states, where a copy or a launch each took 3 to 5 us
// (a query on 2,000 points 6.6 -> 3.1 us, with a subset of 10,000 of 50,000 12.6
// -> 6.0, a four-camera query 11 -> 5.7, a server's round 9 -> 5.2).
// Grid: a query's rows in x (the gather of a large set has more than the 65,536
// that y can hold), the queries in y.  Row 0: one workgroup of 1024 threads copies
// the descriptor and, if the query is fresh, resets the state.  With `begin`, it
// also sets up the round (samples, candidate counter).  The next rows sum a fresh
// query's scoring-set weights in float64, in kWeightParts parts whatever the number
// of rows: one compute unit loads at 14 GB/s what another kernel has just written
// (126,000 weights in one workgroup took the launch 41 us, now 7.2; 50,000 that
// were read before 11.1, now 4.9); who needs the total adds the parts.  Without
// weights it is the number of points (one query on 50,000 6.7 -> 4.8), and a call
// of Gauss-Newton alone needs none (20,000 points 7.0 -> 4.2).
// Then come the rows that clear a fresh query's mailboxes, and the others gather
// its scoring set, S_j = point floor(j * n / m).
// No workgroup reads what another one writes: all read the host's table.
constexpr int kInitThreads = 1024;
constexpr int kSumGroups = 512;  // workgroups of a launch that sum weights, about (two per compute unit)
// Rows that clear, a row for 16 words per thread, at most this many per query or
// those that make two workgroups per compute unit: 4,096 starts on 20,000 points
// (84 MB of mailboxes) 143 us with eight rows, 15.5 with 512.
constexpr int kClearRows = 8;

__device__ inline void clear_words(uint64_t* p, int64_t n, int row, int rows) {
  for (int64_t i = (int64_t)row * kInitThreads + threadIdx.x; i < n; i += (int64_t)rows * kInitThreads) p[i] = 0;
}

__global__ __launch_bounds__(kInitThreads) void init_queries_kernel(QueryTables t, BestState* __restrict__ st,
                                                                    CandBuf cb, int begin, int sum_rows,
                                                                    GNClear clear, int clear_rows) {
  const int q = blockIdx.y;
  // the descriptor in one read over the bus (about 1.5 us), not field by field
  constexpr int kWords = sizeof(QueryDesc) / sizeof(uint64_t), kB = offsetof(QueryDesc, B) / sizeof(uint64_t);
  static_assert(sizeof(QueryDesc) % sizeof(uint64_t) == 0, "copied by words");
  __shared__ uint64_t s_desc[kWords];
  if (threadIdx.x < kWords) {
    const uint64_t w = reinterpret_cast<const uint64_t*>(t.host + q)[threadIdx.x];
    s_desc[threadIdx.x] = w;
    if (blockIdx.x == 0 && !(begin && threadIdx.x == kB))  // (B of a round: below)
      reinterpret_cast<uint64_t*>(t.dev + q)[threadIdx.x] = w;
  }
  lds_barrier();
  const QueryDesc& d = *reinterpret_cast<const QueryDesc*>(s_desc);
  const bool subset = d.S.u != d.full.u;
  const int64_t m = d.m, n = d.n;
  // floor(j n / m) < n < 2^31: the float64 quotient is off by less than one
  const double inv_m = 1.0 / (double)m;
  auto source = [&](int64_t j) {
    const int64_t jn = j * n;
    int64_t s = (int64_t)((double)jn * inv_m);
    const int64_t r = jn - s * m;
    s += r >= m ? 1 : 0;
    return s - (r < 0 ? 1 : 0);
  };
  const int row = (int)blockIdx.x - 1 - sum_rows;
  if (row >= clear_rows) {
    const int64_t j = (int64_t)(row - clear_rows) * kInitThreads + threadIdx.x;
    if (!d.fresh || !subset || j >= m) return;
    const int64_t i = source(j);
    float* dst = const_cast<float*>(d.S.u);
    dst[j] = d.full.u[i];
    dst[m + j] = d.full.v[i];
    dst[2 * m + j] = d.full.X[i];
    dst[3 * m + j] = d.full.Y[i];
    dst[4 * m + j] = d.full.Z[i];
    dst[5 * m + j] = d.full.w ? d.full.w[i] : 1.0f;
    return;
  }
  if (row >= 0) {
    if (!d.fresh) return;
    if (clear.lo && (clear.all || d.lo_team > 1))
      clear_words(clear.lo + q * clear.lo_words, clear.lo_words, row, clear_rows);
    if (clear.fin && (clear.all || d.fin_team > 1))
      clear_words(clear.fin + q * clear.fin_words, clear.fin_words, row, clear_rows);
    return;
  }
  if (blockIdx.x > 0) {
    const float* __restrict__ w = d.full.w;
    if (!d.fresh || !w) return;
    __shared__ double sw[kInitThreads / kWave];
    // (a small set has few parts: sixteen in turn took 100 points 11.0 us, one 4.2)
    if (blockIdx.x == 1 && threadIdx.x < kWeightParts && (int64_t)threadIdx.x * kInitThreads >= m)
      cb.wsum[q * kWeightParts + threadIdx.x] = 0.0;
    for (int u = (int)blockIdx.x - 1; u < kWeightParts && (int64_t)u * kInitThreads < m; u += sum_rows) {
      double p = 0.0;
      for (int64_t i0 = (int64_t)u * kInitThreads + threadIdx.x; i0 < m; i0 += 8 * kWeightParts * kInitThreads) {
        float x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int64_t i = i0 + (int64_t)k * kWeightParts * kInitThreads;
          x[k] = i < m ? w[subset ? source(i) : i] : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) p += (double)x[k];
      }
      p = wave_sum(p);
      if ((threadIdx.x & (kWave - 1)) == 0) sw[threadIdx.x / kWave] = p;
      __syncthreads();
      if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int k = 0; k < kInitThreads / kWave; ++k) tot += sw[k];
        cb.wsum[q * kWeightParts + u] = tot;
      }
      __syncthreads();
    }
    return;
  }
  if (q == 0 && threadIdx.x < 2) clear.tickets[threadIdx.x] = 0;
  if (threadIdx.x == 2) cb.sel_done[q] = 0;
  if (t.rig_host && (int)threadIdx.x < 16 * d.ncam) {
    const int64_t o = d.rig - t.rig_dev;
    t.rig_dev[o + threadIdx.x] = t.rig_host[o + threadIdx.x];
  }
  if (!d.fresh) {
    if (begin && threadIdx.x == 0) {
      if (st[q].finished == 1) st[q].finished = 2;  // refined in the round before: the query has left
      t.dev[q].B = round_samples(d, st[q]);
      cb.n[q] = 0;
    }
    return;
  }
  if (threadIdx.x == 0) {
    BestState& b = st[q];
    for (int e = 0; e < 12; ++e) b.pose[e] = (e == 0 || e == 4 || e == 8) ? 1.0 : 0.0;
    b.cost = __builtin_inf();
    b.count = 0;
    b.h = -1;
    b.j = -1;
    b.have = 0;
    b.lo_runs = 0;
    b.candidates = 0;
    b.inlier_residuals = 0;
    b.final_cost = 0.0;
    b.full_count = 0;
    b.drawn = 0;
    b.batches = 0;
    const bool can = d.m >= 3 && d.total > 0;
    b.active = can ? 1 : 0;
    b.finished = can ? 0 : 1;
    if (begin) {
      t.dev[q].B = round_samples(d, b);
      cb.n[q] = 0;
    }
  }
}

// max_m bounds the scoring subsets of the fresh queries (0: there is none)
hipError_t launch_init_queries(const QueryTables& t, BestState* st, CandBuf cb, int nq, int64_t max_m, bool begin,
                               const GNClear& clear, hipStream_t s) {
  if (nq <= 0) return hipSuccess;
  const int64_t words = (clear.lo ? clear.lo_words : 0) + (clear.fin ? clear.fin_words : 0);
  const int64_t rows = (words + 16 * kInitThreads - 1) / (16 * kInitThreads);
  const int clear_rows = (int)std::min<int64_t>(rows, std::max(kClearRows, kSumGroups / nq));
  const int64_t gather_rows = (max_m + kInitThreads - 1) / kInitThreads;
  // rows for the sums: a part each while the launch has room for them and the sets have points for them
  int64_t weighted = 0;
  for (int q = 0; t.weights && q < nq; ++q)
    if (t.host[q].fresh && t.host[q].full.w) weighted = std::max(weighted, t.host[q].m);
  const int64_t parts = std::min<int64_t>((weighted + kInitThreads - 1) / kInitThreads, kWeightParts);
  const int sum_rows = (int)std::min<int64_t>(parts, std::max(1, kSumGroups / nq));
  hipLaunchKernelGGL(init_queries_kernel, dim3((unsigned)(1 + sum_rows + clear_rows + gather_rows), nq),
                     dim3(kInitThreads), 0, s, t, st, cb, begin ? 1 : 0, sum_rows, clear, clear_rows);
  return hipGetLastError();
}

__global__ void retire_kernel(BestState* __restrict__ st, int nq) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < nq && st[q].finished == 1) st[q].finished = 2;
}

hipError_t launch_retire(BestState* st, int nq, hipStream_t s) {
  if (nq <= 0) return hipSuccess;
  hipLaunchKernelGGL(retire_kernel, dim3((nq + 255) / 256), dim3(256), 0, s, st, nq);
  return hipGetLastError();
}

// Stopping rule: samples needed for inlier ratio eps with minimal sets of 3.
__device__ inline int64_t required_samples(double eps, double conf, int64_t cap) {
  if (!(eps > 0.0)) return cap;
  if (eps >= 1.0) return 0;
  const double denom = log1p(-eps * eps * eps);
  if (!(denom < 0.0)) return cap;
  const double k = ceil(log(1.0 - conf) / denom);
  if (!(k < (double)cap)) return cap;
  if (k < 0.0) return 0;
  return (int64_t)k;
}

// The end of a round for every query, in one workgroup: the round's local
// optimisations update the running best (in selection order, a strictly
// lower refined cost replaces it), the sample count advances, the stopping
// rule runs, and with `begin_next` the next round is set up (samples,
// candidate counter).  The number of queries still sampling is summed in the
// workgroup and written to *active_count (nothing to clear beforehand).
__global__ __launch_bounds__(1024) void round_end_kernel(QueryDesc* __restrict__ qd, CandBuf cb,
                                                         const int32_t* __restrict__ sel,
                                                         const int32_t* __restrict__ n_sel,
                                                         const double* __restrict__ lo_pose,
                                                         const double* __restrict__ lo_cost,
                                                         const int64_t* __restrict__ lo_count, int nq, int kmax,
                                                         BestState* __restrict__ st, int32_t* __restrict__ active_count,
                                                         int32_t* __restrict__ tickets, int begin_next) {
  if (begin_next && threadIdx.x < 2) tickets[threadIdx.x] = 0;
  long long act = 0;
  for (int q = threadIdx.x; q < nq; q += blockDim.x) {
    QueryDesc& d = qd[q];
    BestState& b = st[q];
    if (d.B > 0) {
      const int ns = n_sel[q];
      for (int slot = 0; slot < ns; ++slot) {
        const int p = q * kmax + slot;
        if (lo_cost[p] < b.cost) {
          b.cost = lo_cost[p];
          b.count = lo_count[p];
          for (int e = 0; e < 12; ++e) b.pose[e] = lo_pose[12 * (int64_t)p + e];
          const int64_t o = d.cand_off + sel[q * kMaxTopK + slot];
          b.h = cb.h[o];
          b.j = cb.j[o];
          b.have = 1;
        }
      }
      b.lo_runs += ns;
      b.drawn += d.B;
      b.batches += 1;
      bool more;
      if (d.fixed) {
        more = b.drawn < d.total;
      } else {
        int64_t need = required_samples((double)b.count / (double)d.m, d.confidence, d.total);
        if (need < d.min_iters) need = d.min_iters;
        if (need > d.total) need = d.total;
        more = b.drawn < need;
      }
      if (!more) {
        b.active = 0;
        b.finished = 1;
      }
    }
    act += b.active;
    if (begin_next) {
      d.B = round_samples(d, b);
      cb.n[q] = 0;
      cb.sel_done[q] = 0;
    }
  }
  act = wave_sum(act);
  __shared__ long long s_act[1024 / kWave];
  if ((threadIdx.x & (kWave - 1)) == 0) s_act[threadIdx.x / kWave] = act;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long t = 0;
    for (int w = 0; w < (int)(blockDim.x / kWave); ++w) t += s_act[w];
    *active_count = (int32_t)t;
  }
}

hipError_t launch_round_end(QueryDesc* qd, CandBuf cb, const int32_t* sel, const int32_t* n_sel,
                            const double* lo_pose, const double* lo_cost, const int64_t* lo_count, int nq, int kmax,
                            BestState* st, int32_t* active_count, int32_t* tickets, bool begin_next, hipStream_t s) {
  hipLaunchKernelGGL(round_end_kernel, dim3(1), dim3(1024), 0, s, qd, cb, sel, n_sel, lo_pose, lo_cost, lo_count, nq,
                     kmax, st, active_count, tickets, begin_next ? 1 : 0);
  return hipGetLastError();
}

}  // namespace imloc
