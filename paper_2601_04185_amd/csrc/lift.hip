// lift.hip -- a world point for every query-to-database match, through the
// stored depth maps (ImLoc Sec. 3.3 "Query Time Matching and 2D-3D Lifting": bilinear depth
// at sub-pixel database coordinates, plain lookup otherwise; keep matches with
// valid depth and confidence above the threshold).
//
// One launch, 1,024 matches per workgroup, four per thread.  The output is a
// stable compaction in match order: a workgroup publishes how many of its
// matches it keeps and adds up what the workgroups before it published.  The
// arithmetic is float64, rounded once to the float32 outputs; the work is a
// gather of four depth texels per match, bound by the latency of its three
// dependent loads (match, texels and view, the counts before).  20 views x
// 8,000 matches: 20.1 us in three launches (count, scan, lift again and write)
// -> 13.4, 50 x 5,000 through codes 27.8 -> 16.6; with one or two matches per
// thread 14.9 and 14.4, 22.3 and 18.1.  Of that about one microsecond is the
// wait for the counts.
//
// Depth maps come as float32 metres or as 8-bit log-depth codes (Sec. 3.3
// "Data Compression": depth clipped to [0.25, 128] m, quantised uniformly in
// log depth; code 0 = no depth, code c >= 1 = 0.25 * 512^((c - 1) / 254)).
// Code maps are decoded through a 256-entry float64 table each workgroup
// builds in LDS, so a tap costs one byte of HBM instead of four.
#include "imloc_device.h"
#include "imloc_kernels.h"

namespace imloc {

constexpr int kLiftBlock = 256;
constexpr int kLiftPer = 4;  // matches per thread, kLiftBlock apart

__device__ inline bool depth_ok(float d) { return d > 0.0f && d <= 3.402823466e38f; }  // finite and positive

// Depth texel idx of view map D; false if it holds no valid depth.
template <bool kCodes>
__device__ inline bool tap(const LiftArgs& a, int64_t idx, const double* lut, double& d) {
  if constexpr (kCodes) {
    const int c = a.codes[idx];
    d = lut[c];
    return c != 0;
  } else {
    const float f = a.depth[idx];
    d = f;
    return depth_ok(f);
  }
}

// A match, loaded whether it will be kept or not: one memory latency.
struct LiftMatch {
  float conf, qu, qv, fu, fv;
  int view;
};

__device__ inline LiftMatch lift_load(const LiftArgs& a, int64_t i) {
  return LiftMatch{a.conf[i], a.q_u[i], a.q_v[i], a.db_u[i], a.db_v[i], a.view[i]};
}

template <bool kCodes>
__device__ inline bool lift_one(const LiftArgs& a, const LiftMatch& m, const double* lut, float out[6]) {
  const float conf = m.conf;
  if (!(conf > a.min_conf)) return false;
  const int k = m.view;
  if (k < 0 || k >= a.n_views) return false;
  const float qu = m.qu, qv = m.qv, fu = m.fu, fv = m.fv;
  if (!isfinite(qu) || !isfinite(qv) || !isfinite(fu) || !isfinite(fv)) return false;
  const int64_t base = (int64_t)k * a.H * a.W;
  const double du = fu, dv = fv;
  double d;
  if (a.subpixel) {
    const double x = du - 0.5, y = dv - 0.5;
    const double x0 = floor(x), y0 = floor(y);
    if (x0 < 0.0 || y0 < 0.0 || x0 + 1.0 > (double)(a.W - 1) || y0 + 1.0 > (double)(a.H - 1)) return false;
    const int64_t c0 = (int64_t)x0, r0 = (int64_t)y0;
    double d00, d01, d10, d11;
    const bool ok00 = tap<kCodes>(a, base + r0 * a.W + c0, lut, d00);
    const bool ok01 = tap<kCodes>(a, base + r0 * a.W + c0 + 1, lut, d01);
    const bool ok10 = tap<kCodes>(a, base + (r0 + 1) * a.W + c0, lut, d10);
    const bool ok11 = tap<kCodes>(a, base + (r0 + 1) * a.W + c0 + 1, lut, d11);
    if (!(ok00 && ok01 && ok10 && ok11)) return false;
    const double ax = x - x0, ay = y - y0;
    d = (1.0 - ay) * ((1.0 - ax) * d00 + ax * d01) + ay * ((1.0 - ax) * d10 + ax * d11);
  } else {
    const double cf = floor(du), rf = floor(dv);
    if (cf < 0.0 || rf < 0.0 || cf > (double)(a.W - 1) || rf > (double)(a.H - 1)) return false;
    if (!tap<kCodes>(a, base + (int64_t)rf * a.W + (int64_t)cf, lut, d)) return false;
  }
  const double* cam = a.cams + 4 * k;
  const double* T = a.poses + 12 * k;
  const double xc = d * (du - cam[2]) / cam[0] - T[9];
  const double yc = d * (dv - cam[3]) / cam[1] - T[10];
  const double zc = d - T[11];
  // X_w = R^T (x_c - t)
  out[0] = qu;
  out[1] = qv;
  out[2] = (float)(T[0] * xc + T[3] * yc + T[6] * zc);
  out[3] = (float)(T[1] * xc + T[4] * yc + T[7] * zc);
  out[4] = (float)(T[2] * xc + T[5] * yc + T[8] * zc);
  out[5] = conf;
  return true;
}

// decode table of the code maps (kLiftBlock == 256: one entry per thread)
template <bool kCodes>
__device__ inline void fill_lut(double* lut) {
  static_assert(kLiftBlock == 256, "one table entry per thread");
  if constexpr (kCodes) lut[threadIdx.x] = log8_level((int)threadIdx.x);
}

// What a workgroup publishes: 1 and its own count, then 2 and the count up to
// its end.  A word is complete in itself, so no fence is needed.
__device__ inline void lift_publish(uint64_t* word, unsigned kind, unsigned value) {
  __hip_atomic_store(word, ((uint64_t)kind << 32) | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Kept matches of one tile, counted by this workgroup.
template <bool kCodes>
__device__ inline unsigned lift_count(const LiftArgs& a, int tile, const double* lut) {
  unsigned c = 0;
  for (int j = 0; j < kLiftPer; ++j) {
    const int64_t i = (int64_t)tile * (kLiftBlock * kLiftPer) + j * kLiftBlock + threadIdx.x;
    float o[6];
    c += (unsigned)__syncthreads_count(i < a.n && lift_one<kCodes>(a, lift_load(a, i), lut, o));
  }
  return c;
}

// Kept matches before workgroup `tile`, from the words of those before it, 256
// at a time from the nearest on, up to the first that knows its end.  Every
// workgroup publishes its own count before it waits for another; what has not
// come after a.polls polls (its workgroup may have no room to start) is counted
// here instead, so every wait ends.
template <bool kCodes>
__device__ inline unsigned lift_before(const LiftArgs& a, int tile, const double* lut) {
  __shared__ unsigned s_sum[kLiftBlock / kWave];
  __shared__ int s_end[kLiftBlock / kWave];
  __shared__ int s_miss;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  unsigned before = 0;
  for (int hi = tile; hi > 0; hi -= kLiftBlock) {
    const int p = hi - 1 - tid;
    uint64_t v = 0;
    bool got = p < 0;
    for (int n = 0; !got && n < a.polls; ++n) {
      v = __hip_atomic_load(a.state + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      got = (v >> 32) != 0;
      if (!got) __builtin_amdgcn_s_sleep(1);
    }
    while (__syncthreads_or(!got)) {
      if (tid == 0) s_miss = -1;
      __syncthreads();
      if (!got) atomicMax(&s_miss, p);
      __syncthreads();
      const int q = s_miss;
      const unsigned c = lift_count<kCodes>(a, q, lut);  // (its barriers also free s_miss)
      if (p == q) {
        v = (1ull << 32) | c;
        got = true;
      }
    }
    // the nearest word of kind 2: lanes after it do not count
    const uint64_t ends = __ballot((v >> 32) == 2);
    const int end = ends ? __ffsll((unsigned long long)ends) - 1 : kWave;
    unsigned c = lane <= end ? (unsigned)v : 0u;
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) c += __shfl_xor(c, off, kWave);
    if (lane == 0) {
      s_sum[wave] = c;
      s_end[wave] = ends != 0;
    }
    __syncthreads();
    bool done = false;
#pragma unroll
    for (int w = 0; w < kLiftBlock / kWave; ++w) {
      if (!done) before += s_sum[w];
      done |= s_end[w] != 0;
    }
    __syncthreads();
    if (done) break;
  }
  return before;
}

template <bool kCodes>
__global__ __launch_bounds__(kLiftBlock) void lift_kernel(LiftArgs a) {
  __shared__ double lut[kCodes ? 256 : 1];
  __shared__ unsigned s_kept[kLiftPer * kLiftBlock / kWave];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int nb = gridDim.x, tile = blockIdx.x;
  const int64_t i0 = (int64_t)tile * (kLiftBlock * kLiftPer) + tid;
  LiftMatch m[kLiftPer];
#pragma unroll
  for (int j = 0; j < kLiftPer; ++j) {
    const int64_t i = i0 + j * kLiftBlock;
    m[j] = lift_load(a, i < a.n ? i : a.n - 1);
  }
  fill_lut<kCodes>(lut);
  __syncthreads();
  float o[kLiftPer][6];
  uint64_t keep[kLiftPer];
#pragma unroll
  for (int j = 0; j < kLiftPer; ++j) {
    const bool k = i0 + j * kLiftBlock < a.n && lift_one<kCodes>(a, m[j], lut, o[j]);
    keep[j] = __ballot(k);
    if (lane == 0) s_kept[j * (kLiftBlock / kWave) + wave] = (unsigned)__popcll(keep[j]);
  }
  __syncthreads();
  // rank of the thread's matches inside the workgroup
  unsigned own = 0, rank[kLiftPer];
#pragma unroll
  for (int e = 0; e < kLiftPer * kLiftBlock / kWave; ++e) {
    if (e % (kLiftBlock / kWave) == wave) rank[e / (kLiftBlock / kWave)] = own;
    own += s_kept[e];
  }
  if (tid == 0 && tile < nb - 1) lift_publish(a.state + tile, tile == 0 ? 2 : 1, own);
  const unsigned before = lift_before<kCodes>(a, tile, lut);
  if (tid == 0) {
    if (tile > 0 && tile < nb - 1) lift_publish(a.state + tile, 2, before + own);
    if (tile == nb - 1) *a.n_out = *a.n_host = (int32_t)(before + own);
  }
#pragma unroll
  for (int j = 0; j < kLiftPer; ++j) {
    if (!((keep[j] >> lane) & 1u)) continue;
    const int64_t dst = (int64_t)before + rank[j] + __popcll(keep[j] & ((1ull << lane) - 1));
    if (dst >= a.capacity) continue;
    a.out_u[dst] = o[j][0];
    a.out_v[dst] = o[j][1];
    a.out_X[dst] = o[j][2];
    a.out_Y[dst] = o[j][3];
    a.out_Z[dst] = o[j][4];
    if (a.out_w) a.out_w[dst] = o[j][5];
    if (a.out_src) a.out_src[dst] = (int32_t)(i0 + j * kLiftBlock);
  }
}

static int lift_blocks(int64_t n) { return (int)((n + kLiftBlock * kLiftPer - 1) / (kLiftBlock * kLiftPer)); }

int64_t lift_words(int64_t n) {  // the last workgroup publishes nothing
  const int nb = lift_blocks(n);
  return nb > 1 ? nb - 1 : 0;
}

hipError_t launch_lift(const LiftArgs& a, hipStream_t s) {
  const int nb = lift_blocks(a.n);
  if (nb == 0) return launch_fill_i32(a.n_out, 1, 0, s);
  if (a.codes) {
    hipLaunchKernelGGL(lift_kernel<true>, dim3(nb), dim3(kLiftBlock), 0, s, a);
  } else {
    hipLaunchKernelGGL(lift_kernel<false>, dim3(nb), dim3(kLiftBlock), 0, s, a);
  }
  return hipGetLastError();
}

constexpr int kEncodeQuads = 4;

// Encoder of the code maps: nearest level in log depth (halves away from
// zero), depth clipped to [0.25, 128] m, code 0 for depth not finite or <= 0.
// Four depths per load (float4) and store (32 bits) over the first 4 * n4
// entries, one per thread over the rest (n4 = 0 when the arrays are not 16- and
// 4-byte aligned).  A thread takes four such quads, 256 apart, loaded together,
// and the float64 logarithm is the exception (log8_code): a call on 20 maps of
// 480 x 640 20.0 -> 8.7 us (31 MB: 6 us at the rate of a copy), on 20 million
// depths 71 -> 19.5 us.  With one quad per thread, 6,000 short workgroups, the
// faster logarithm alone gains nothing.
__global__ __launch_bounds__(256) void log8_encode_kernel(const float* __restrict__ depth, int64_t n, int64_t n4,
                                                           uint8_t* __restrict__ codes) {
  constexpr int Q = kEncodeQuads;
  const int64_t q0 = (int64_t)blockIdx.x * (256 * Q) + threadIdx.x;
  if (q0 - threadIdx.x < n4) {
    float4 v[Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int64_t q = q0 + 256 * j;
      v[j] = reinterpret_cast<const float4*>(depth)[q < n4 ? q : n4 - 1];
    }
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int64_t q = q0 + 256 * j;
      const uint32_t w = (uint32_t)log8_code(v[j].x) | ((uint32_t)log8_code(v[j].y) << 8) |
                         ((uint32_t)log8_code(v[j].z) << 16) | ((uint32_t)log8_code(v[j].w) << 24);
      if (q < n4) reinterpret_cast<uint32_t*>(codes)[q] = w;
    }
  }
#pragma unroll
  for (int j = 0; j < Q; ++j) {  // the rest: entries past the last quad
    const int64_t i = 4 * n4 + (q0 + 256 * j - n4);
    if (q0 + 256 * j >= n4 && i < n) codes[i] = log8_code(depth[i]);
  }
}

hipError_t launch_log8_encode(const float* depth, int64_t n, uint8_t* codes, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const bool vec = reinterpret_cast<uintptr_t>(depth) % 16 == 0 && reinterpret_cast<uintptr_t>(codes) % 4 == 0;
  const int64_t n4 = vec ? n / 4 : 0;
  const int64_t threads = n4 + (n - 4 * n4);
  constexpr int kPer = 256 * kEncodeQuads;
  hipLaunchKernelGGL(log8_encode_kernel, dim3((unsigned)((threads + kPer - 1) / kPer)), dim3(256), 0, s, depth, n, n4,
                     codes);
  return hipGetLastError();
}

}  // namespace imloc
