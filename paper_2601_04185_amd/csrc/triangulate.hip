// triangulate.hip -- mapping-time depth of every pixel of a mapping image by
// 1-DoF triangulation of dense matches (ImLoc Sec. 3.3 "Depth Estimation by
// Dense Matching").
//
// Poses are known, so the point of pixel (row i, col j) lies on its ray
// X(l) = C0 + l r0, r0 = R0^T K0^-1 [j + 0.5, i + 0.5, 1]^T (l is the z-depth).
// Each match of the pixel in covisible view k (confidence >= 0.05) is a unit
// ray rk from the view's centre Ck; the angular error of depth l for it is the
// angle between X(l) - Ck and rk.  Per pixel:
//   1. every match gives one depth hypothesis: the depth minimising its own
//      angular error, in closed form (the cosine's derivative along the ray
//      vanishes at one depth); it counts if that is a minimum at l > 0;
//   2. each hypothesis counts the matches within 2 degrees; the most inliers
//      win, ties going to the lowest view;
//   3. the depth is refined on that inlier set by minimising the
//      confidence-weighted sum of squared angular errors (1-D Newton, step
//      halving while the cost rises, to a step below 1e-9 l);
//   4. it is kept if the inlier set has at least min_inliers (4) members.
//
// Two launches, float64 throughout (on MI355X the
// float64 vector rate equals the non-packed float32 rate):
//   - triangulate_kernel: steps 1, 2 and 4, a lane per pixel; a pixel whose
//     depth needs refinement is appended to a queue (one atomic per workgroup);
//   - tri_refine_kernel: step 3, a quad of lanes per queued pixel.
// Refinement is most of the arithmetic, but only the pixels with enough
// inliers (about half of a mapping image) need it, and each runs its own
// number of Newton steps; run in place, every wave would pay for its slowest
// lane while its other lanes idle.  Compacted, the waves of the second launch
// are full.
//
// Both launches are bound by float64 instructions.  Along the pixel's ray
// everything an angle needs is a polynomial of l with coefficients that are
// fixed per match (b = C0 - Ck, r the match's ray):
//   a . r = b.r + l r0.r            |a|^2 = b.b + 2 l b.r0 + l^2 r0.r0
// so a hypothesis tests a match with 6 instructions from three values, and the
// refinement evaluates a match without its ray (below).
// 560 x 560 pixels, ten views: triangulate_kernel 84 -> 36 us, tri_refine_kernel
// 411 -> 55 us against loops over cross products, three gradients by atan2 and
// a cost per Newton step (the first kernel's floor, 38 MB of matches, is 8 us;
// both now issue float64 instructions in 60 to 85 % of their cycles).
// Match arrays are [view][H][W], so the loads of the first launch are
// coalesced; the second recomputes the rays of its pixel's inliers with the
// same arithmetic.
#include "imloc_device.h"
#include "imloc_kernels.h"

namespace imloc {

struct TriViewDev {
  double ifx, ify, cx, cy;  // 1 / fx, 1 / fy
  double Rt[9];   // R^T row-major: world direction = Rt * K^-1 [u, v, 1]^T
  double b[3];    // C0 - Ck
  double ga;      // b . b
};

__device__ inline void tri_ray(const TriViewDev& v, double u, double w, double r[3]) {
  const double dx = (u - v.cx) * v.ifx, dy = (w - v.cy) * v.ify;
  for (int c = 0; c < 3; ++c) r[c] = v.Rt[3 * c] * dx + v.Rt[3 * c + 1] * dy + v.Rt[3 * c + 2];
}

constexpr int kTriBlock = 256;  // most threads per workgroup of the first launch

// Dynamic LDS of one workgroup: per-view constants [V + 1] (entry 0: the
// mapping camera), then for the hypotheses two values per match, each
// [V][threads].
size_t tri_lds_bytes(int V, int threads) {
  return (size_t)(V + 1) * sizeof(TriViewDev) + (size_t)V * threads * 2 * sizeof(double);
}

struct TriLds {
  TriViewDev* view;
  double *al, *be;
};

// carve the dynamic LDS and load the per-view constants (every lane of the
// workgroup takes part)
__device__ inline TriLds tri_lds_setup(const TriArgs& a) {
  extern __shared__ double s_dyn[];
  TriLds L;
  L.view = reinterpret_cast<TriViewDev*>(s_dyn);
  L.al = s_dyn + (size_t)(a.V + 1) * (sizeof(TriViewDev) / sizeof(double));
  L.be = L.al + a.V * blockDim.x;
  for (int e = threadIdx.x; e <= a.V; e += blockDim.x) {
    const double* src = a.views + 16 * e;
    TriViewDev v;
    v.ifx = 1.0 / src[0]; v.ify = 1.0 / src[1]; v.cx = src[2]; v.cy = src[3];
    for (int c = 0; c < 9; ++c) v.Rt[c] = src[4 + c];
    for (int c = 0; c < 3; ++c) v.b[c] = src[13 + c];
    v.ga = v.b[0] * v.b[0] + v.b[1] * v.b[1] + v.b[2] * v.b[2];
    L.view[e] = v;
  }
  __syncthreads();
  return L;
}

// The refinement runs on a quad of lanes per pixel: lane j of the quad takes
// the views k = j, j + 4, ... of the inlier set, and the sums are added over
// the quad by DPP.  The butterfly gives every lane of the quad the same bits
// ((x0 + x1) + (x2 + x3) up to commutation), so the four lanes take the same
// decisions.  A pixel's Newton chain is a quarter as long, and four times as
// many waves hide each other's latency.
constexpr int kTriQuad = 4;
constexpr int kTriLoadGroup = 16;  // match loads issued together

__host__ __device__ inline int tri_quad_rows(int V) { return (V + kTriQuad - 1) / kTriQuad; }

__device__ __forceinline__ double quad_sum(double x) {
  x += dpp_f64<0xb1>(x);  // quad_perm [1, 0, 3, 2]
  x += dpp_f64<0x4e>(x);  // quad_perm [2, 3, 0, 1]
  return x;
}

// What the refinement keeps of a match.  In the plane normal to its unit ray r,
// with the axes e1 = y / |y|, y = r0 x r, and r x e1, the point a = b + l r0 has
// the coordinates p + l Y and m, of which only the first moves:
//   S^2 = |a x r|^2 = (p + l Y)^2 + m^2,    s = a . r = al + l be,
// Y = |y|, p = (b x r) . e1, m = (b x r) . (r x e1); the angle is atan2(S, s).
struct TriSlot {
  double p, Y, m2, al, be, w;
};

__device__ inline TriSlot tri_slot(const double b[3], const double r0[3], const double r[3], double w) {
  const double y0 = r0[1] * r[2] - r0[2] * r[1], y1 = r0[2] * r[0] - r0[0] * r[2], y2 = r0[0] * r[1] - r0[1] * r[0];
  const double c0 = b[1] * r[2] - b[2] * r[1], c1 = b[2] * r[0] - b[0] * r[2], c2 = b[0] * r[1] - b[1] * r[0];
  TriSlot t;
  const double yy = y0 * y0 + y1 * y1 + y2 * y2;
  if (yy > 0.0) {
    const double i = rsqrt(yy);
    t.Y = yy * i;
    t.p = (c0 * y0 + c1 * y1 + c2 * y2) * i;
    const double m = (c0 * (r[1] * y2 - r[2] * y1) + c1 * (r[2] * y0 - r[0] * y2) + c2 * (r[0] * y1 - r[1] * y0)) * i;
    t.m2 = m * m;
  } else {  // the ray of the match is the pixel's: its angle's sine does not depend on l but for |a|
    t.Y = 0.0;
    t.p = sqrt(c0 * c0 + c1 * c1 + c2 * c2);
    t.m2 = 0.0;
  }
  t.al = b[0] * r[0] + b[1] * r[1] + b[2] * r[2];
  t.be = r0[0] * r[0] + r0[1] * r[1] + r0[2] * r[2];
  t.w = w;
  return t;
}

// A squared angle th^2, f = th dth/dl = (th^2 / 2)' and f' at depth l.
//
// With z = S^2 / s^2 (the squared tangent), th^2 = z A(z)^2, A = atan(sqrt z) /
// sqrt z = 1 - z / 3 + z^2 / 5 - ..., and th dth/dz = A / (2 (1 + z)): rational
// in l but for A, no root and no arc tangent.  Below z = 0.01 (5.7 degrees;
// inliers start below 2) the terms up to z^7 leave 0.01^8 / 17 < 2^-56.  A match
// beyond that takes atan2.
struct TriEval {
  double e, g, c;
};

constexpr double kTriSeries = 0.01;
constexpr double kTriLastStep = 1e-9;

__device__ __forceinline__ TriEval tri_eval_wide(const TriSlot& t, double l) {
  const double x1 = fma(l, t.Y, t.p), S2 = fma(x1, x1, t.m2), s = fma(l, t.be, t.al), q = fma(s, s, S2);
  const double S = sqrt(S2), th = atan2(S, s);
  TriEval o{th * th, 0.0, 0.0};
  if (S2 > 1e-24 * q) {
    const double dS = x1 * t.Y / S, J = (s * dS - S * t.be) / q;
    o.g = th * J;
    o.c = J * J + th * (s * ((t.Y * t.Y - dS * dS) / S) - J * 2.0 * (x1 * t.Y + s * t.be)) / q;
  } else {  // the limit where the angle vanishes
    const double J = s * t.Y / q;
    o.g = th * J;
    o.c = J * J;
  }
  return o;
}

__device__ __forceinline__ TriEval tri_eval(const TriSlot& t, double l) {
  const double x1 = fma(l, t.Y, t.p), S2 = fma(x1, x1, t.m2), s = fma(l, t.be, t.al), q = fma(s, s, S2);
  if (!(s > 0.0 && S2 <= kTriSeries * (s * s))) return tri_eval_wide(t, l);
  const double r = 1.0 / (s * q), i = r * q, h = s * s * (r * s);  // 1 / s, 1 / (1 + z)
  const double i2 = i * i, z = S2 * i2;
  double A = -1.0 / 15.0, D = 0.0;  // A and dA/dz by Horner's rule
  auto term = [&](double c) {
    D = fma(D, z, A);
    A = fma(A, z, c);
  };
  term(1.0 / 13.0);
  term(-1.0 / 11.0);
  term(1.0 / 9.0);
  term(-1.0 / 7.0);
  term(1.0 / 5.0);
  term(-1.0 / 3.0);
  term(1.0);
  const double x1Y = x1 * t.Y, S2b = S2 * t.be;
  const double zp = 2.0 * (s * x1Y - S2b) * (i * i2);
  const double zpp = 2.0 * (t.Y * t.Y * (s * s) + t.be * (3.0 * S2b - 4.0 * x1Y * s)) * (i2 * i2);
  const double F1 = 0.5 * A * h, F2 = 0.5 * D * h - F1 * h;  // d/dz and d2/dz2 of th^2 / 2
  return TriEval{z * A * A, F1 * zp, F2 * zp * zp + F1 * zpp};
}

// (dth/dl)^2, for the Gauss-Newton curvature
__device__ inline double tri_slope2(const TriSlot& t, double l) {
  const double x1 = fma(l, t.Y, t.p), S2 = fma(x1, x1, t.m2), s = fma(l, t.be, t.al), q = fma(s, s, S2);
  if (!(S2 > 1e-24 * q)) return (s * t.Y / q) * (s * t.Y / q);
  const double N = s * (x1 * t.Y) - S2 * t.be;
  return N * N / (S2 * q * q);
}

// the ray of pixel p of the mapping image (unnormalised: its z-component in
// the camera is 1, so that l is the z-depth)
__device__ inline void tri_pixel_ray(const TriArgs& a, const TriViewDev& v0, int64_t p, double r0[3]) {
  const int i = (int)(p / a.W), j = (int)(p - (int64_t)i * a.W);
  tri_ray(v0, (double)j + 0.5, (double)i + 0.5, r0);
}

// Steps 1, 2 and 4: a lane per pixel.  Of each match LDS holds al = b . r and be
// = r0 . r ([view][lane], so the lanes of a wave hit distinct banks), r scaled
// so that the inlier test is (a . r)^2 > |a|^2; the other terms do not depend
// on r's length.  Hypotheses are formed kTriGroup at a time and tested
// together, so that a match's values are read from LDS once per group.  The
// loops run over all views with the same view in every lane (the view constants
// are broadcast reads); a lane without a match in a view drops that view's
// results.  A pixel to refine is queued with its hypothesis and inlier set.
// Hypotheses per group: the rest of the last group is tested for nothing, and more
// take registers.  560 x 560 pixels, groups of 3 / 4 / 5 / 6 / 8 / 10, us: 3 views
// 11.7 / 12.8 / 12.9 / 13.8 / 15.5 / 16.7, 7 views 27.1 / 26.4 / 27.5 / 28.2 / 26.3 /
// 27.0, 10 views 40.2 / 39.1 / 36.5 / 38.1 / 43.1 / 35.1, 13 views 59.1 / 59.0 / 57.0
// / 60.4 / 56.7 / 62.4, 20 views 137 / 127 / 127 / 137 / 135 / 118: five is within 10 %
// of the best at each of them.
constexpr int kTriGroup = 5;

__global__ __launch_bounds__(kTriBlock) void triangulate_kernel(TriArgs a) {
  const TriLds L = tri_lds_setup(a);
  const int tid = threadIdx.x, nt = blockDim.x;
  const int64_t HW = (int64_t)a.H * a.W;
  const int64_t p = (int64_t)blockIdx.x * nt + tid;
  const bool pix = p < HW;  // the lanes past the image take part in the queue's ballot only
  double r0[3];
  tri_pixel_ray(a, L.view[0], pix ? p : 0, r0);
  const double ep = r0[0] * r0[0] + r0[1] * r0[1] + r0[2] * r0[2];

  // the pixel's matches.  The loads of a group of views are issued together,
  // so that the group waits for one memory latency, not one per view.
  uint32_t ok = 0;
  for (int k0 = 0; pix && k0 < a.V; k0 += kTriLoadGroup) {
    float mu[kTriLoadGroup], mv[kTriLoadGroup], cf[kTriLoadGroup];
#pragma unroll
    for (int j = 0; j < kTriLoadGroup; ++j) {
      const int64_t o = (int64_t)min(k0 + j, a.V - 1) * HW + p;
      mu[j] = a.mu[o]; mv[j] = a.mv[o]; cf[j] = a.conf[o];
    }
#pragma unroll
    for (int j = 0; j < kTriLoadGroup; ++j) {
      const int k = k0 + j;
      if (k < a.V && cf[j] >= a.min_conf && isfinite(mu[j]) && isfinite(mv[j])) {
        const double* b = L.view[k + 1].b;
        double r[3];
        tri_ray(L.view[k + 1], mu[j], mv[j], r);
        const double inv = rsqrt(a.cos2_thr * (r[0] * r[0] + r[1] * r[1] + r[2] * r[2]));
        const int o = k * nt + tid;
        L.al[o] = (b[0] * r[0] + b[1] * r[1] + b[2] * r[2]) * inv;
        L.be[o] = (r0[0] * r[0] + r0[1] * r[1] + r0[2] * r[2]) * inv;
        ok |= 1u << k;
      }
    }
  }

  // hypotheses, in view order
  int best_n = 0;
  double best_l = 0.0;
  uint32_t best_set = 0;
  for (int h0 = 0; h0 < a.V; h0 += kTriGroup) {
    double l[kTriGroup];
    uint32_t set[kTriGroup], valid = 0;
#pragma unroll
    for (int j = 0; j < kTriGroup; ++j) {
      const int h = min(h0 + j, a.V - 1);
      const double* b = L.view[h + 1].b;
      const int o = h * nt + tid;
      const double al = L.al[o], be = L.be[o], de = b[0] * r0[0] + b[1] * r0[1] + b[2] * r0[2];
      const double ga = L.view[h + 1].ga;
      const double den = be * de - al * ep;
      l[j] = (al * de - be * ga) / den;
      set[j] = 0;
      // a minimum: the cosine there, c / sqrt(q) |r|, exceeds its limits at l -> +-inf, +-be / sqrt(ep) |r|
      const double c = al + l[j] * be, q = ga + l[j] * (2.0 * de + l[j] * ep);
      if (h0 + j < a.V && ((ok >> h) & 1u) && den != 0.0 && l[j] > 0.0 && isfinite(l[j]) && c > 0.0 &&
          c * c * ep > be * be * q)
        valid |= 1u << j;
    }
    if (!__ballot(valid != 0)) continue;
    // inliers: angle < thr  <=>  a.r > 0 and (a.r)^2 > cos^2(thr) |a|^2 |r|^2
    for (int k = 0; k < a.V; ++k) {
      const double* b = L.view[k + 1].b;
      const int o = k * nt + tid;
      const double al = L.al[o], be = L.be[o], de2 = 2.0 * (b[0] * r0[0] + b[1] * r0[1] + b[2] * r0[2]);
      const double ga = L.view[k + 1].ga;
#pragma unroll
      for (int j = 0; j < kTriGroup; ++j) {
        const double s = fma(l[j], be, al), q = fma(l[j], fma(l[j], ep, de2), ga);
        if (s * fabs(s) > q) set[j] |= 1u << k;
      }
    }
#pragma unroll
    for (int j = 0; j < kTriGroup; ++j) {
      set[j] &= ok;
      const int cnt = __popc(set[j]);
      if (((valid >> j) & 1u) && cnt > best_n) {
        best_n = cnt;
        best_l = l[j];
        best_set = set[j];
      }
    }
  }

  const bool refine = pix && best_n > 0 && best_n >= a.min_inliers;
  // queue the pixels to refine: one counter add per workgroup (adds to one
  // address take about 10 ns each), slots in thread order
  __shared__ int s_first[kTriBlock / kWave + 1];
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  const uint64_t bal = __ballot(refine);
  if (lane == 0) s_first[wave] = __popcll(bal);
  __syncthreads();
  if (tid == 0) {
    int sum = 0;
    for (int w = 0; w < nt / kWave; ++w) {
      const int c = s_first[w];
      s_first[w] = sum;
      sum += c;
    }
    s_first[kTriBlock / kWave] = sum ? atomicAdd(a.n_tasks, sum) : 0;
  }
  __syncthreads();
  if (refine) {
    const int slot = s_first[kTriBlock / kWave] + s_first[wave] + __popcll(bal & ((1ull << lane) - 1));
    a.tasks[slot] = TriTask{best_l, (int32_t)p, best_set};
  }
  if (!pix) return;
  if (a.inliers) a.inliers[p] = best_n;
  if (!refine) {
    if (a.depth) a.depth[p] = 0.0f;
    if (a.codes) a.codes[p] = 0;
  }
}

// Step 3 for the queued pixels, a quad of lanes each: Newton's method on the
// confidence-weighted sum of squared angular errors over the inlier set (the
// Gauss-Newton curvature where the second derivative is not positive), a step
// that raises the cost halved up to 30 times, until the step is below 1e-12 l
// or max_iters steps.  A step below 1e-12 l is not taken while being halved
// either.  A Newton step below 1e-9 l is the last and needs no trial: the one
// after it is of the order of its square, and its decrease of the cost is
// below the cost's rounding noise, which made a wave halve such steps down to
// 1e-12 l for its unluckiest lane.  Each depth tried is evaluated once, cost and both
// derivatives together.  Lane i of the quad keeps the members i, i + 4, ... of
// the inlier set in registers (KQ = ceil(V / 4) bounds them, a template, so
// the loops unroll; slots that no pixel of the wave fills are passed over).
// Launched over the largest possible queue; waves past its length return at
// once.
template <int KQ>
__global__ __launch_bounds__(kWave) void tri_refine_kernel(TriArgs a) {
  constexpr int kPerWave = kWave / kTriQuad;  // pixels per wave
  const int n = *a.n_tasks;
  if ((int64_t)blockIdx.x * kPerWave >= n) return;
  const TriLds L = tri_lds_setup(a);
  const int lane = threadIdx.x;
  const int64_t t = (int64_t)blockIdx.x * kPerWave + lane / kTriQuad;
  if (t >= n) return;  // the whole quad
  const TriTask task = a.tasks[t];
  const int64_t HW = (int64_t)a.H * a.W;
  const int64_t p = task.p;
  double r0[3];
  tri_pixel_ray(a, L.view[0], p, r0);
  // this lane's members (-1: none), loads issued together
  int view[KQ];
  uint32_t rest = task.set;
#pragma unroll
  for (int j = 0; j < KQ; ++j) {
    view[j] = -1;
#pragma unroll
    for (int i = 0; i < kTriQuad; ++i) {
      if ((lane & (kTriQuad - 1)) == i && rest) view[j] = __ffs(rest) - 1;
      rest &= rest - 1;
    }
  }
  float mu[KQ], mv[KQ], cf[KQ];
#pragma unroll
  for (int j = 0; j < KQ; ++j) {
    const int64_t o = (int64_t)max(view[j], 0) * HW + p;  // view 0 always exists
    mu[j] = a.mu[o]; mv[j] = a.mv[o]; cf[j] = a.conf[o];
  }
  bool used[KQ];  // by a pixel of the wave
  TriSlot slot[KQ];
#pragma unroll
  for (int j = 0; j < KQ; ++j) {
    used[j] = __ballot(view[j] >= 0) != 0;
    if (!used[j]) continue;
    const TriViewDev& v = L.view[max(view[j], 0) + 1];
    double r[3];
    tri_ray(v, mu[j], mv[j], r);
    const double inv = rsqrt(r[0] * r[0] + r[1] * r[1] + r[2] * r[2]);
    r[0] *= inv;
    r[1] *= inv;
    r[2] *= inv;
    slot[j] = tri_slot(v.b, r0, r, cf[j]);
    if (view[j] < 0) slot[j] = TriSlot{0.0, 0.0, 0.0, 1.0, 0.0, 0.0};  // an exact 0
  }
  auto evaluate = [&](double l) {
    TriEval o{0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < KQ; ++j) {
      if (!used[j]) continue;
      const TriEval v = tri_eval(slot[j], l);
      o.e += slot[j].w * v.e;
      o.g += slot[j].w * v.g;
      o.c += slot[j].w * v.c;
    }
    return TriEval{quad_sum(o.e), quad_sum(o.g), quad_sum(o.c)};
  };
  // (one evaluation in the code: at the first depth, then at each one tried)
  double l = task.l, ln = l, step = 0.0;
  TriEval cur{};
  for (int it = -1, half = 0;;) {
    const TriEval v = evaluate(ln);
    if (it < 0 || v.e <= cur.e) {
      const bool moved = ln != l;
      l = ln;
      cur = v;
      if (it >= 0 && (!moved || fabs(step) <= 1e-12 * l)) break;
      if (++it >= a.max_iters || cur.g == 0.0) break;
      double curv = cur.c;
      if (!(curv > 0.0)) {
        curv = 0.0;
#pragma unroll
        for (int j = 0; j < KQ; ++j)
          if (used[j]) curv += slot[j].w * tri_slope2(slot[j], l);
        curv = quad_sum(curv);
        if (!(curv > 0.0)) break;
      }
      step = -cur.g / curv;
      half = 0;
      if (cur.c > 0.0 && fabs(step) <= kTriLastStep * l) {
        if (fabs(step) > 1e-12 * l) l += step;
        break;
      }
    } else {
      step *= 0.5;
      ++half;
    }
    bool tried = false;  // the next depth to try: in front of the camera, a step that counts
    for (; half < 30 && !tried && !(fabs(step) <= 1e-12 * l); ) {
      ln = l + step;
      tried = ln > 0.0;
      if (!tried) {
        step *= 0.5;
        ++half;
      }
    }
    if (!tried) break;
  }
  const double depth = l > 0.0 ? l : 0.0;
  const float d32 = (float)depth;
  if ((lane & (kTriQuad - 1)) == 0) {
    if (a.depth) a.depth[p] = d32;
    if (a.codes) a.codes[p] = depth > 0.0 ? log8_code(d32) : (uint8_t)0;
  }
}

hipError_t launch_triangulate(const TriArgs& a, hipStream_t s) {
  const int64_t HW = (int64_t)a.H * a.W;
  if (HW <= 0) return hipSuccess;
  int block = kTriBlock;  // as many waves as 64 KiB of LDS hold
  while (block > kWave && tri_lds_bytes(a.V, block) > 65536 - 256) block /= 2;
  const dim3 grid((unsigned)((HW + block - 1) / block));
  hipLaunchKernelGGL(triangulate_kernel, grid, dim3(block), tri_lds_bytes(a.V, block), s, a);
  const dim3 grid_refine((unsigned)((HW * kTriQuad + kWave - 1) / kWave));
  const size_t lds = tri_lds_bytes(a.V, 0);
  switch (tri_quad_rows(a.V)) {  // slots per lane, 1..8 for 1..32 views
    case 1: hipLaunchKernelGGL(tri_refine_kernel<1>, grid_refine, dim3(kWave), lds, s, a); break;
    case 2: hipLaunchKernelGGL(tri_refine_kernel<2>, grid_refine, dim3(kWave), lds, s, a); break;
    case 3: hipLaunchKernelGGL(tri_refine_kernel<3>, grid_refine, dim3(kWave), lds, s, a); break;
    case 4: hipLaunchKernelGGL(tri_refine_kernel<4>, grid_refine, dim3(kWave), lds, s, a); break;
    case 5: hipLaunchKernelGGL(tri_refine_kernel<5>, grid_refine, dim3(kWave), lds, s, a); break;
    case 6: hipLaunchKernelGGL(tri_refine_kernel<6>, grid_refine, dim3(kWave), lds, s, a); break;
    case 7: hipLaunchKernelGGL(tri_refine_kernel<7>, grid_refine, dim3(kWave), lds, s, a); break;
    default: hipLaunchKernelGGL(tri_refine_kernel<8>, grid_refine, dim3(kWave), lds, s, a); break;
  }
  return hipGetLastError();
}

}  // namespace imloc
