// refine.hip -- float64 Gauss-Newton of LO-RANSAC (ImLoc Sec. 3.3, "Pose
// Estimation"):
//   local optimisation: Gauss-Newton on the truncated cost over the scoring
//     set, started from a candidate that beats the running best; the inlier
//     set is taken again at every iterate;
//   final refinement: IRLS on the Cauchy loss, each point weighted by its
//     confidence, over the inliers of the full set at the best pose (that set
//     stays fixed).
//
// One launch runs every iteration of every problem.  A problem is worked on
// by a team of workgroups: its points are cut into groups (2,048 points each
// up to 262,144 points, see gn_group_points), every member evaluates its
// groups at the current pose -- the 6x6 normal equations (upper triangle), the
// gradient, the cost and the inlier count of a group, in float64 -- and the
// members exchange the groups' sums, add them in group order and take the
// same decision.  The sums of a group and their order depend on the problem
// alone, so a result does not depend on the team's size or on the batch
// around it.  Residual r = pi(R X + t) - x; left update on SO(3).
//
// Why a team inside one launch: a run is a chain of short, dependent steps
// (evaluate, sum, decide).  A launch per iteration cost 4.3 to 10 us each, and
// twelve launches however early a run ended; the exchange below costs 0.9 us
// between 2 members, 1.5 us among 10 or 16 and 1.8 us among 32 (29 sums each),
// and a run that ends frees its workgroups at once.  Measured (MI355X, both
// launches): a query of 2,000 points with one start 117 -> 77 us, of 50,000
// points with eight starts 155 -> 109 us, a four-camera query of 20,000 points
// 152 -> 120 us; 256 queries of 5,000 to 80,000 points 4.24 -> 3.91 ms, a burst
// of 192 queries at the server 9.1 -> 5.0 ms.  What bounds it: for one query,
// issue by a lone wave per SIMD (5.4 cycles per float64 instruction) and the
// exchange, about half each; for a batch, float64 issue (4.3 cycles).
//
// The exchange: a group's 29 sums go to its mailbox as 58 words of 64 bits,
// each half of a value with a tag that names the evaluation, written and read
// by relaxed agent-scope atomics.  A word carries its own tag, so no fence
// and no counter is needed: a reader polls the words themselves.  Mailboxes
// alternate between two buffers: a member writes evaluation j + 2 only after
// it has read everyone's j + 1, which a member writes after reading everyone's
// j.  They are cleared before the first use (init_queries_kernel), and tags
// count on from round to round.
//
// Every wait ends.  Workgroups take their role from a ticket drawn at their
// start, so the members of every team but the last one started are running,
// and only that one can be short of members while workgroup slots are taken.
// A wait is also bounded: a member that has polled GNLaunch::polls times evaluates
// the missing groups itself (the same sums, bit for bit) and does not wait
// again in this launch.
#include "imloc_device.h"
#include "imloc_kernels.h"

namespace imloc {

constexpr int kAcc = 29;  // 21 (H upper) + 6 (g) + cost + count
constexpr double kStepTol2 = 1e-20;  // squared length of a step that ends a run
constexpr int kGNThreads = 256;
constexpr int kGNWaves = kGNThreads / kWave;
constexpr int kGNGroup = 2048;          // points of a group that stays in LDS, at most: eight per thread
constexpr int kGNGroupMost = 32768;     // of the largest (offsets in a group are 16 bits, 0xffff is none)
constexpr int kGNHalfGroups = 32;        // groups of half that size, at most
constexpr int kGNGroupsWanted = 128;     // groups of a problem, until their size grows past kGNGroup
constexpr int kGNBox = 64;              // mailbox words of a group (58 used)
constexpr int kGNInBlock = 64;          // groups read together (a bit each in a word)
constexpr uint16_t kGNNone = 0xffff;
// waves per SIMD where the points are read from memory (the local optimisation
// of 256 queries took 3.3 ms with two, 2.73 with three, 3.96 with four, which
// spill); with the points in LDS two workgroups fit a compute unit
constexpr int kGNWavesMany = 3;
constexpr int kGNRig = 18;              // LDS doubles of a rig camera: R, t, 1/fx, 1/fy, -cx/fx, -cy/fy, fx^2, fy^2

// 1 / z for the per-point work of an evaluation (z > 0 and finite): the
// hardware reciprocal and two Newton steps, within about an ulp of the
// rounded quotient, in 5 instructions where a rounded division takes about
// 10.
__device__ __forceinline__ double recip_pos(double z) {
  double r = __builtin_amdgcn_rcp(z);
  r = fma(r, fma(-z, r, 1.0), r);
  return fma(r, fma(-z, r, 1.0), r);
}

// ln(1 + t) for t >= 0: 1 + t = 2^e m with m in [1/sqrt 2, sqrt 2), and ln m =
// 2 atanh(f / (2 + f)), f = m - 1, by the series of atanh (|s| < 0.172, so its
// terms are below 3e-17 from s^21 on; for e = 0, f is t itself).  Within 5e-16
// relative of ln(1 + t); about 35 instructions where the library's log1p took
// most of an evaluation step of the refinement (1,820 cycles a step with it,
// see the kernel).
__device__ __forceinline__ double log1p_pos(double t) {
#pragma clang fp contract(off)
  const double y = 1.0 + t;
  int e = __builtin_amdgcn_frexp_exp(y);      // y = 2^e * mant, mant in [0.5, 1)
  double m = __builtin_amdgcn_frexp_mant(y);
  const bool low = m < 0.70710678118654757;
  e = low ? e - 1 : e;
  m = low ? m + m : m;
  const double f = e == 0 ? t : m - 1.0;
  const double s = f * recip_pos(2.0 + f);
  const double z = s * s;
  double p = 1.0 / 19.0;
  p = fma(p, z, 1.0 / 17.0);
  p = fma(p, z, 1.0 / 15.0);
  p = fma(p, z, 1.0 / 13.0);
  p = fma(p, z, 1.0 / 11.0);
  p = fma(p, z, 1.0 / 9.0);
  p = fma(p, z, 1.0 / 7.0);
  p = fma(p, z, 1.0 / 5.0);
  p = fma(p, z, 1.0 / 3.0);
  const double s2 = s + s;
  return fma((double)e, 0.69314718055994531, fma(s2 * z, p, s2));
}

// A value that every lane holds alike, in scalar registers.
__device__ __forceinline__ double uniform(double x) {
  const long long b = __double_as_longlong(x);
  const unsigned lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Points of a group of a problem of n points: one group up to 2,048 points,
// then 1,024 points each while that makes at most 32 groups, then 2,048, and
// past 128 groups a 128th of the points (in steps of 2,048) up to 32,768.  More
// groups are more compute units for one problem (a lone wave per SIMD issues a
// float64 instruction every 5.4 cycles, so four points per thread take 2,600
// cycles of an evaluation), but each evaluation ends with an exchange of about
// 3,500 cycles once there are two, and 32 mailboxes take 5,000.  Larger groups
// would not stay in LDS: with a 32nd of the points from 65,536 points on, both
// stages on 66,000 / 90,000 / 200,000 points from one start took 223 / 225 /
// 352 us, now 159 / 170 / 234.
__host__ __device__ inline int gn_group_points(int64_t n) {
  if (n <= kGNGroup) return kGNGroup;
  if (n <= (int64_t)kGNHalfGroups * kGNGroup / 2) return kGNGroup / 2;
  int64_t s = (n + kGNGroupsWanted - 1) / kGNGroupsWanted;
  s = (s + kGNGroup - 1) / kGNGroup * kGNGroup;
  return (int)(s > kGNGroupMost ? kGNGroupMost : s);
}

__host__ __device__ inline int groups_for(int64_t n) {
  const int s = gn_group_points(n);
  const int64_t g = (n + s - 1) / s;
  return g > 0 ? (int)g : 1;
}

int gn_groups(int64_t n) { return groups_for(n); }

// the most groups that a problem of up to n points has (more points can make
// fewer groups: 32,768 make 32, 32,769 make 17)
int gn_most_groups(int64_t n) {
  int g = groups_for(n);
  if (n > (int64_t)kGNHalfGroups * kGNGroup / 2 && g < kGNHalfGroups) g = kGNHalfGroups;
  if (n > (int64_t)kGNGroupsWanted * kGNGroup && g < kGNGroupsWanted) g = kGNGroupsWanted;
  return g;
}

// The final refinement's in-set where its points do not stay in LDS: 16-bit
// offsets in the group, in point order, up to a kGNNone (512 entries per 512
// points).
int64_t gn_inset_bytes(int64_t n) {
  const int64_t c = (n + 511) / 512;
  return 1024 * (c > 0 ? c : 1);
}

// Mailboxes of nprob problems of at most `groups` groups (two buffers each).
int64_t gn_box_words(int groups) { return groups > 1 ? (int64_t)2 * kGNBox * groups : 0; }
size_t gn_scratch_bytes(int nprob, int groups) {
  return (size_t)(nprob > 0 ? nprob : 1) * (size_t)gn_box_words(groups) * sizeof(uint64_t) + 256;
}

// Team size of a problem of `groups` groups when a launch holds `total`
// groups and the chip `slots` workgroups: a member per group while all fit;
// else each member takes several groups, at most `most`.
int gn_team(int groups, int64_t total, int slots, int most, int mode) {
  if (mode == 2 || groups <= 1) return 1;
  int64_t r = 1;
  if (mode == 0 && total > slots) r = (total + slots - 1) / slots;
  if (r > most) r = most;
  const int t = (int)((groups + r - 1) / r);
  return t < kGNGroupsWanted ? t : kGNGroupsWanted;
}

// Exchange of lanes 32..63 of x with lanes 0..31 of y (swap16: odd 16-lane
// rows of x with even rows of y); then x + y holds, in a lane with that lane
// bit clear, the pair sum of x, and with it set, the pair sum of y.
__device__ __forceinline__ void swap32_f64(double& x, double& y) {
  const long long bx = __double_as_longlong(x), by = __double_as_longlong(y);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)bx, (unsigned)by, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(bx >> 32), (unsigned)(by >> 32), false, false);
  x = __longlong_as_double(((long long)hi[0] << 32) | (unsigned)lo[0]);
  y = __longlong_as_double(((long long)hi[1] << 32) | (unsigned)lo[1]);
}

__device__ __forceinline__ void swap16_f64(double& x, double& y) {
  const long long bx = __double_as_longlong(x), by = __double_as_longlong(y);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)bx, (unsigned)by, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(bx >> 32), (unsigned)(by >> 32), false, false);
  x = __longlong_as_double(((long long)hi[0] << 32) | (unsigned)lo[0]);
  y = __longlong_as_double(((long long)hi[1] << 32) | (unsigned)lo[1]);
}

// One halving level on lane bit B with the partner given by a DPP control:
// a lane keeps the lower half of the list if its bit is clear, the upper
// half if set, and adds what the partner (bit flipped) did not keep.
template <int CTRL, int H>
__device__ __forceinline__ void halve_dpp(double* v, bool upper) {
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const double send = upper ? v[i] : v[i + H];
    const double keep = upper ? v[i + H] : v[i];
    v[i] = keep + dpp_f64<CTRL>(send);
  }
}

// Wave sums of the 29 accumulators by recursive halving (about 125
// instructions instead of 29 separate reductions): after the six levels, lane
// l holds the wave total of entry l >> 1 (entries 29..31 are zero padding).
// Partners: lane ^ 32 and lane ^ 16 by the swap instructions, lane ^ 8
// (row_ror 8), lane ^ 7 (row_half_mirror: bit 2 flips, and the lanes already
// merged on bits 0..1 are all covered after the last two levels), lane ^ 2,
// lane ^ 1 (quad_perm).  The order of additions depends on the lane only.
__device__ __forceinline__ double wave_sum29(const double* a) {
  double v[32];
#pragma unroll
  for (int e = 0; e < 32; ++e) v[e] = e < kAcc ? a[e] : 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    double x = v[i], y = v[i + 16];
    swap32_f64(x, y);
    v[i] = x + y;
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    double x = v[i], y = v[i + 8];
    swap16_f64(x, y);
    v[i] = x + y;
  }
  const int lane = threadIdx.x & (kWave - 1);
  halve_dpp<0x128, 4>(v, (lane & 8) != 0);   // row_ror 8: lane ^ 8
  halve_dpp<0x141, 2>(v, (lane & 4) != 0);   // row_half_mirror: lane ^ 7
  halve_dpp<0x4e, 1>(v, (lane & 2) != 0);    // quad_perm [2, 3, 0, 1]: lane ^ 2
  return v[0] + dpp_f64<0xb1>(v[0]);         // quad_perm [1, 0, 3, 2]: lane ^ 1
}

// Inlier test of point i of the full set at a final pose (float64, through
// the point's rig camera for a rig query): depth > 0 and squared pixel
// residual below tau^2.
__device__ __forceinline__ bool mask_test(const QueryDesc& d, const double* pose, double X, double Y, double Z,
                                          double u, double v, int64_t i) {
  double x = pose[0] * X + pose[1] * Y + pose[2] * Z + pose[9];
  double y = pose[3] * X + pose[4] * Y + pose[5] * Z + pose[10];
  double z = pose[6] * X + pose[7] * Y + pose[8] * Z + pose[11];
  double fx = d.fx, fy = d.fy, cx = d.cx, cy = d.cy;
  if (d.ncam > 0) {  // through the point's rig camera
    const double* rc = d.rig + 16 * cam_of(d.segF, d.ncam, i);
    const double* Rc = rc + 4;
    const double xr[3] = {x, y, z};
    x = Rc[0] * xr[0] + Rc[1] * xr[1] + Rc[2] * xr[2] + rc[13];
    y = Rc[3] * xr[0] + Rc[4] * xr[1] + Rc[5] * xr[2] + rc[14];
    z = Rc[6] * xr[0] + Rc[7] * xr[1] + Rc[8] * xr[2] + rc[15];
    fx = rc[0]; fy = rc[1]; cx = rc[2]; cy = rc[3];
  }
  if (!(z > 0.0)) return false;
  const double du = fx * x / z + cx - u;
  const double dv = fy * y / z + cy - v;
  return du * du + dv * dv < d.tau * d.tau;
}

// Uniform values of one problem.
struct GNView {
  CorrF32 c;
  int64_t n;
  double ifx, ify, ucx, vcy;   // normalised observation: u ifx + ucx
  double fx2, fy2;
  double tau2, inv_s2;
  int ncam;
  const int64_t* seg;
};

// A point in registers (past the end of a group: u is NaN, w is 0).
struct GNPt {
  float X, Y, Z, u, v, w;
  int cam;
  bool use;
};

// Normal equations of one point of a single camera, in normalised image
// coordinates p = x / z, q = y / z, iz = 1 / z: the rows of d(p, q)/d(dw, dt)
// are J0 = (-p q, 1 + p^2, -q, iz, 0, -p iz) and J1 = (-(1 + q^2), p q, p, 0,
// iz, -q iz); the pixel scales and the weight are in w0 = w fx^2 and w1 = w
// fy^2.  The products with the structural zeros are left out (H[3][4] gets
// nothing).
__device__ __forceinline__ void acc_point(double* a, double p, double q, double iz, double du, double dv, double w0,
                                          double w1) {
  const double pq = p * q;
  const double J0[6] = {-pq, fma(p, p, 1.0), -q, iz, 0.0, -(p * iz)};
  const double J1[6] = {-fma(q, q, 1.0), pq, p, 0.0, iz, -(q * iz)};
  double W0[6], W1[6];
#pragma unroll
  for (int r = 0; r < 6; ++r) {
    W0[r] = w0 * J0[r];
    W1[r] = w1 * J1[r];
  }
  int k = 0;
#pragma unroll
  for (int r = 0; r < 6; ++r) {
#pragma unroll
    for (int c = r; c < 6; ++c) {
      const bool z0 = r == 4 || c == 4, z1 = r == 3 || c == 3;
      if (!z0 && !z1) a[k] = fma(W0[r], J0[c], fma(W1[r], J1[c], a[k]));
      else if (!z0) a[k] = fma(W0[r], J0[c], a[k]);
      else if (!z1) a[k] = fma(W1[r], J1[c], a[k]);
      ++k;
    }
  }
#pragma unroll
  for (int r = 0; r < 6; ++r) {
    if (r == 4) a[21 + r] = fma(W1[r], dv, a[21 + r]);
    else if (r == 3) a[21 + r] = fma(W0[r], du, a[21 + r]);
    else a[21 + r] = fma(W0[r], du, fma(W1[r], dv, a[21 + r]));
  }
}

// The same for a rig camera: x_c = R_c x_r + t_c with the rig-frame point x_r
// moving under the left update of the rig pose, so the rows of d(p, q)/dx_c
// are carried through R_c: J = [x_r x r, r] with r0 = (R_c row 0 - p R_c row
// 2) iz, r1 = (R_c row 1 - q R_c row 2) iz.
__device__ __forceinline__ void acc_point_rig(double* a, const double xr[3], double p, double q, double iz,
                                              const double* Rc, double du, double dv, double w0, double w1) {
  double J0[6], J1[6];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    J0[3 + c] = fma(-p, Rc[6 + c], Rc[c]) * iz;
    J1[3 + c] = fma(-q, Rc[6 + c], Rc[3 + c]) * iz;
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
    J0[c] = fma(xr[c1], J0[3 + c2], -(xr[c2] * J0[3 + c1]));
    J1[c] = fma(xr[c1], J1[3 + c2], -(xr[c2] * J1[3 + c1]));
  }
  int k = 0;
#pragma unroll
  for (int r = 0; r < 6; ++r) {
    const double W0 = w0 * J0[r], W1 = w1 * J1[r];
#pragma unroll
    for (int c = r; c < 6; ++c) {
      a[k] = fma(W0, J0[c], fma(W1, J1[c], a[k]));
      ++k;
    }
    a[21 + r] = fma(W0, du, fma(W1, dv, a[21 + r]));
  }
}

// One point at pose P into the sums; `take` is left true if it counts (local
// optimisation: an inlier; first evaluation of the refinement: an inlier,
// which puts it in the set; later ones: in the set).  Every product and sum
// is written as it is rounded (no contraction is left to the compiler), so
// the point gives the same bits wherever this is inlined.
template <int MODE, bool RIG>
__device__ __forceinline__ bool gn_point(const GNView& g, const double* s_rig, const double* P, bool first,
                                         const GNPt& pt, double* a) {
#pragma clang fp contract(off)
  const double X = pt.X, Y = pt.Y, Z = pt.Z, w = pt.w;
  double x = fma(P[0], X, fma(P[1], Y, fma(P[2], Z, P[9])));
  double y = fma(P[3], X, fma(P[4], Y, fma(P[5], Z, P[10])));
  double z = fma(P[6], X, fma(P[7], Y, fma(P[8], Z, P[11])));
  double ifx = g.ifx, ify = g.ify, ucx = g.ucx, vcy = g.vcy, fx2 = g.fx2, fy2 = g.fy2;
  const double xr[3] = {x, y, z};
  const double* rc = nullptr;
  if (RIG && g.ncam > 0) {  // through the point's camera: x_c = R_c x_r + t_c
    rc = s_rig + kGNRig * pt.cam;
    ifx = rc[12]; ify = rc[13]; ucx = rc[14]; vcy = rc[15]; fx2 = rc[16]; fy2 = rc[17];
    x = fma(rc[0], xr[0], fma(rc[1], xr[1], fma(rc[2], xr[2], rc[9])));
    y = fma(rc[3], xr[0], fma(rc[4], xr[1], fma(rc[5], xr[2], rc[10])));
    z = fma(rc[6], xr[0], fma(rc[7], xr[1], fma(rc[8], xr[2], rc[11])));
  }
  const bool front = z > 0.0;
  const double iz = recip_pos(z);
  const double p = x * iz, q = y * iz;
  const double du = p - fma((double)pt.u, ifx, ucx), dv = q - fma((double)pt.v, ify, vcy);
  const double r2 = fma(fx2, du * du, fy2 * (dv * dv));
  const bool in = front && r2 < g.tau2;  // never of an unused point
  if (MODE == 0) {
    a[27] = fma(w, in ? r2 : g.tau2, a[27]);
    if (in) {
      const double w0 = w * fx2, w1 = w * fy2;
      if (RIG && g.ncam > 0) acc_point_rig(a, xr, p, q, iz, rc, du, dv, w0, w1);
      else acc_point(a, p, q, iz, du, dv, w0, w1);
    }
    return in;
  }
  const bool take = first ? in : pt.use;  // (an unused point may hold anything)
  if (take) {
    // a point of the set that has gone behind the camera costs as much as one at the threshold
    const double t = (front ? r2 : g.tau2) * g.inv_s2;
    a[27] = fma(w, log1p_pos(t), a[27]);  // times s^2 after the last sum
    if (front) {
      const double wc = w * recip_pos(1.0 + t);  // the Cauchy weight
      const double w0 = wc * fx2, w1 = wc * fy2;
      if (RIG && g.ncam > 0) acc_point_rig(a, xr, p, q, iz, rc, du, dv, w0, w1);
      else acc_point(a, p, q, iz, du, dv, w0, w1);
    }
  }
  return take;
}

struct GNArgs {
  const QueryDesc* qd;
  CandBuf cb;
  const int32_t* sel;
  const int32_t* n_sel;
  const double* start_direct;
  BestState* bst;
  uint64_t* box;       // mailboxes [problem][2][box_groups][kGNBox]
  uint8_t* in_set_all;
  double* out_pose;
  double* out_cost;
  int64_t* out_count;
  int32_t* ticket;     // null: no team has more than one member
  int nq, kmax, box_groups;
  int team_direct;     // start_direct: members of every problem
  int polls;           // polls of a wait before a member works alone
  int write_mask;      // final refinement: the inlier mask and its count at the final pose
};

struct GNShared {
  double cur[12], eval[12], start[12];
  int done;
};

// H d = -g for the 6x6 normal equations given by tot (upper triangle of H,
// packed by rows, then g), through the Schur complement of the rotation
// block: H = [A B; B^T C], d_t = S^-1 (b_t - B^T A^-1 b_r) with S = C - B^T
// A^-1 B, d_r = A^-1 b_r - A^-1 B d_t; the 3x3 inverses by adjugates.  H is
// positive definite exactly when A and S are (leading minors checked); false
// otherwise.  Every lane solves it in its own registers: no lane exchanges,
// two divisions on the dependency chain.
__device__ __forceinline__ bool solve6_schur(const double* t, double x[6]) {
  const double h00 = t[0], h01 = t[1], h02 = t[2], h03 = t[3], h04 = t[4], h05 = t[5];
  const double h11 = t[6], h12 = t[7], h13 = t[8], h14 = t[9], h15 = t[10];
  const double h22 = t[11], h23 = t[12], h24 = t[13], h25 = t[14];
  const double h33 = t[15], h34 = t[16], h35 = t[17], h44 = t[18], h45 = t[19], h55 = t[20];
  const double br[3] = {-t[21], -t[22], -t[23]}, bt[3] = {-t[24], -t[25], -t[26]};
  // A^-1 by its adjugate
  const double c00 = fma(h11, h22, -h12 * h12), c01 = fma(h02, h12, -h01 * h22), c02 = fma(h01, h12, -h02 * h11);
  const double c11 = fma(h00, h22, -h02 * h02), c12 = fma(h01, h02, -h00 * h12), c22 = fma(h00, h11, -h01 * h01);
  const double detA = fma(h00, c00, fma(h01, c01, h02 * c02));
  const bool okA = h00 > 0.0 && c22 > 0.0 && detA > 0.0;
  const double ia = recip_pos(detA);
  const double I[3][3] = {{c00 * ia, c01 * ia, c02 * ia}, {c01 * ia, c11 * ia, c12 * ia}, {c02 * ia, c12 * ia, c22 * ia}};
  const double B[3][3] = {{h03, h04, h05}, {h13, h14, h15}, {h23, h24, h25}};
  const double C[3][3] = {{h33, h34, h35}, {h34, h44, h45}, {h35, h45, h55}};
  // T = A^-1 B, u = A^-1 b_r
  double T[3][3], u[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
#pragma unroll
    for (int c = 0; c < 3; ++c) T[r][c] = fma(I[r][0], B[0][c], fma(I[r][1], B[1][c], I[r][2] * B[2][c]));
    u[r] = fma(I[r][0], br[0], fma(I[r][1], br[1], I[r][2] * br[2]));
  }
  // S = C - B^T T, r = b_t - B^T u
  double S[3][3], rt[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
#pragma unroll
    for (int c = 0; c < 3; ++c) S[r][c] = C[r][c] - fma(B[0][r], T[0][c], fma(B[1][r], T[1][c], B[2][r] * T[2][c]));
    rt[r] = bt[r] - fma(B[0][r], u[0], fma(B[1][r], u[1], B[2][r] * u[2]));
  }
  const double d00 = fma(S[1][1], S[2][2], -S[1][2] * S[1][2]), d01 = fma(S[0][2], S[1][2], -S[0][1] * S[2][2]);
  const double d02 = fma(S[0][1], S[1][2], -S[0][2] * S[1][1]), d11 = fma(S[0][0], S[2][2], -S[0][2] * S[0][2]);
  const double d12 = fma(S[0][1], S[0][2], -S[0][0] * S[1][2]), d22 = fma(S[0][0], S[1][1], -S[0][1] * S[0][1]);
  const double detS = fma(S[0][0], d00, fma(S[0][1], d01, S[0][2] * d02));
  const bool okS = S[0][0] > 0.0 && d22 > 0.0 && detS > 0.0;
  const double is = recip_pos(detS);
  const double J[3][3] = {{d00 * is, d01 * is, d02 * is}, {d01 * is, d11 * is, d12 * is}, {d02 * is, d12 * is, d22 * is}};
#pragma unroll
  for (int r = 0; r < 3; ++r) x[3 + r] = fma(J[r][0], rt[0], fma(J[r][1], rt[1], J[r][2] * rt[2]));
#pragma unroll
  for (int r = 0; r < 3; ++r) x[r] = u[r] - fma(T[r][0], x[3], fma(T[r][1], x[4], T[r][2] * x[5]));
  return okA && okS;
}

// Decision j of a run, on the sums of evaluation j at s.eval: the evaluated
// pose becomes the accepted one if its cost did not rise (at j = 0 it is the
// start); unless the iteration budget is spent, the normal equations at the
// accepted pose give the pose of evaluation j + 1.  A cost-raising step, or a
// system that is not positive definite, ends the run with the accepted pose.
// Run by the 64 lanes of wave 0 (every lane takes the same branches): every
// lane solves the 6 x 6 system itself (solve6_schur), and lane e < 12 forms
// element e of the next pose.  The accepted cost and count stay in the wave's
// registers; s.done says whether this decision ends the run.
__device__ __forceinline__ void gn_decide_wave(int j, int iters, const double* tot, GNShared& s, double& best_cost,
                                               double& best_count) {
  const int lane = threadIdx.x;
  const double cur_l = s.eval[lane < 12 ? lane : 0];
  const int rr = lane < 9 ? lane / 3 : lane - 9, cc = lane < 9 ? lane % 3 : 3;
  // column cc of the evaluated pose (its translation for cc = 3)
  const int at = cc < 3 ? cc : 9, by = cc < 3 ? 3 : 1;
  const double p0 = s.eval[at], p1 = s.eval[at + by], p2 = s.eval[at + 2 * by];
  const double cost = tot[27], count = tot[28];
  double d[6];
  const bool solved = solve6_schur(tot, d);
  bool done = true;
  if (j == 0 || cost <= best_cost) {  // accept the evaluated pose
    if (lane < 12) s.cur[lane] = cur_l;
    best_cost = cost;
    best_count = count;
    // converged: a step shorter than 1e-10 (norm of (dw, dt)) is not taken and
    // ends the run (every lane holds d; the sum in element order)
    double d2 = 0.0;
#pragma unroll
    for (int e = 0; e < 6; ++e) d2 += d[e] * d[e];
    if (j < iters && solved && !(d2 < kStepTol2)) {
      // left update: R' = Exp(dw) R, t' = Exp(dw) t + dt, element `lane` (< 12)
      double E[9];
      so3_exp(d, E);
      // row rr of E and entry rr of the translation step by selects (a lane-indexed
      // register array would be placed in scratch memory)
      const double er0 = rr == 0 ? E[0] : (rr == 1 ? E[3] : E[6]);
      const double er1 = rr == 0 ? E[1] : (rr == 1 ? E[4] : E[7]);
      const double er2 = rr == 0 ? E[2] : (rr == 1 ? E[5] : E[8]);
      const double dt = rr == 0 ? d[3] : (rr == 1 ? d[4] : d[5]);
      const double v = fma(er0, p0, fma(er1, p1, er2 * p2)) + (cc < 3 ? 0.0 : dt);
      if (lane < 12) s.eval[lane] = v;
      done = false;
    }
  }
  if (lane == 0) s.done = done;
}

// LDS of a workgroup.
struct GNLds {
  double rows[2][kGNWaves][kAcc];
  double in[kGNInBlock][kAcc];
  double tot[kAcc];
  GNShared s;
  int kept[kGNGroup / kGNThreads][kGNWaves];
  unsigned long long miss;
  int alone, role;
};

// The points of a member's only group -- in the refinement, after its first
// evaluation, those of its in-set -- stay in (dynamic) LDS, so that an
// evaluation reads no memory.  Unused slots of the last slice have u = NaN and
// w = 0.
struct GNResident {
  float pt[6][kGNGroup];
  uint8_t cam[kGNGroup];
};

// Entry i of a uniform array, addressed from scalar registers.
__device__ __forceinline__ float at_u32(const float* base, unsigned i) {
  return *(const __attribute__((address_space(1))) float*)((const __attribute__((address_space(1))) char*)base +
                                                           (size_t)(i * 4u));
}

// A resident group into LDS: every load is in flight before the first is
// waited for (the first evaluation took 2,300 cycles per slice of 256 points
// when it loaded them itself, one slice ahead).
template <bool RIG>
__device__ __forceinline__ void gn_load_resident(GNResident& R, const GNView& g, int64_t g0, int pts) {
  constexpr int kSlices = kGNGroup / kGNThreads;
  const float* src[6] = {g.c.X + g0, g.c.Y + g0, g.c.Z + g0, g.c.u + g0, g.c.v + g0, g.c.w ? g.c.w + g0 : g.c.X + g0};
  float x[6][kSlices];
#pragma unroll
  for (int k = 0; k < kSlices; ++k) {
    if (k * kGNThreads >= pts) break;
    const int i = k * kGNThreads + (int)threadIdx.x;
#pragma unroll
    for (int c = 0; c < 6; ++c) x[c][k] = at_u32(src[c], i < pts ? i : pts - 1);
  }
#pragma unroll
  for (int k = 0; k < kSlices; ++k) {
    if (k * kGNThreads >= pts) break;
    const int i = k * kGNThreads + (int)threadIdx.x;
    const bool use = i < pts;
    R.pt[0][i] = x[0][k]; R.pt[1][i] = x[1][k]; R.pt[2][i] = x[2][k];
    R.pt[3][i] = use ? x[3][k] : __builtin_nanf("");
    R.pt[4][i] = x[4][k];
    R.pt[5][i] = use ? (g.c.w ? x[5][k] : 1.0f) : 0.0f;
    if (RIG) R.cam[i] = g.ncam > 0 ? (uint8_t)cam_of(g.seg, g.ncam, g0 + i) : 0;
  }
}

// Keep a resident group's in-set alone, in point order: bit k of `taken` says
// whether this thread's point k (index 256 k + thread) is in it.  The points
// pass through registers, as their new places may be other threads' old ones.
// Returns their number.
template <bool RIG>
__device__ __forceinline__ int gn_keep_resident(GNLds& L, GNResident& R, unsigned taken, int steps) {
  constexpr int kSlices = kGNGroup / kGNThreads;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  float x[6][kSlices];
  int cam[kSlices], at[kSlices];
#pragma unroll
  for (int k = 0; k < kSlices; ++k) {
    if (k >= steps) break;
    const int i = k * kGNThreads + (int)threadIdx.x;
#pragma unroll
    for (int c = 0; c < 6; ++c) x[c][k] = R.pt[c][i];
    cam[k] = RIG ? R.cam[i] : 0;
    const uint64_t bal = __ballot((taken >> k) & 1u);
    at[k] = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) L.kept[k][wave] = __popcll(bal);
  }
  lds_barrier();
  int base = 0;
#pragma unroll
  for (int k = 0; k < kSlices; ++k) {
    if (k >= steps) break;
    int mine = base + at[k];
#pragma unroll
    for (int w = 0; w < kGNWaves; ++w) {
      const int c = L.kept[k][w];
      mine += w < wave ? c : 0;
      base += c;
    }
    if ((taken >> k) & 1u) {
#pragma unroll
      for (int c = 0; c < 6; ++c) R.pt[c][mine] = x[c][k];
      if (RIG) R.cam[mine] = (uint8_t)cam[k];
    }
  }
  return __builtin_amdgcn_readfirstlane(base);
}

// One evaluation of one group at pose P: accumulate per thread in point
// order, across the wave by recursive halving, then the waves in wave order.
// Threads 0..28 return the sums.  The refinement's first evaluation lists the
// group's in-set in point order (in LDS or in `list`); later ones read that:
// thread t takes its points t, t + 256, ...  n_in: the set's size (resident).
// `turn` alternates between calls.
template <int MODE, bool RIG, bool RES>
__device__ __forceinline__ double gn_eval_group(GNLds& L, GNResident& R, const GNView& g, const double* s_rig,
                                                const double* P, int grp, bool first, bool in_lds, uint16_t* list,
                                                int& n_in, int turn) {
  const bool resident = RES && in_lds;
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int S = gn_group_points(g.n);
  const int64_t g0 = (int64_t)grp * S;
  const int64_t left = g.n - g0;
  const int pts = (int)(left < S ? (left > 0 ? left : 0) : S);
  const bool from_set = MODE == 1 && !first;
  const int items = from_set && resident ? n_in : pts;
  const int steps = __builtin_amdgcn_readfirstlane((items + kGNThreads - 1) / kGNThreads);
  const float *GX = g.c.X + g0, *GY = g.c.Y + g0, *GZ = g.c.Z + g0, *GU = g.c.u + g0, *GV = g.c.v + g0,
              *GW = g.c.w ? g.c.w + g0 : GX;
  const bool has_w = g.c.w != nullptr;
  const int last = items > 0 ? items - 1 : 0;
  double pose[12];
#pragma unroll
  for (int e = 0; e < 12; ++e) pose[e] = e < 9 ? uniform(P[e]) : P[e];  // (one scalar operand per multiply-add)
  double a[kAcc];
#pragma unroll
  for (int e = 0; e < kAcc; ++e) a[e] = 0.0;
  int count = 0, kept = 0;
  if (resident) {
    // the loop of a latency-bound run: a lone wave per SIMD pays for every
    // scalar instruction too, so nothing but the points is in it (MODE 1 with
    // the general loop's control: 1,350 cycles per step, with this 950)
    int i = threadIdx.x;
    unsigned taken = 0;  // bit k: this thread's point k
    auto load = [&](GNPt& t, int at) {
      at &= kGNGroup - 1;
      t.X = R.pt[0][at]; t.Y = R.pt[1][at]; t.Z = R.pt[2][at]; t.u = R.pt[3][at]; t.v = R.pt[4][at]; t.w = R.pt[5][at];
      t.cam = RIG ? R.cam[at] : 0;
    };
    GNPt next;
    load(next, i);
    for (int k = 0; k < steps; ++k) {
      GNPt t = next;
      load(next, i + kGNThreads);
      t.use = MODE == 0 || i < items;
      if (RIG && MODE == 1) t.cam = t.use ? t.cam : 0;
      const bool take = gn_point<MODE, RIG>(g, s_rig, pose, first, t, a);
      count += __popcll(__ballot(take));
      if (MODE == 1) taken |= (unsigned)take << k;
      i += kGNThreads;
    }
    if (MODE == 1 && first) n_in = gn_keep_resident<RIG>(L, R, taken, steps);
  } else {
    // The camera of a point of a group (rig): most groups have points of one or two,
    // so one compare tells (a search among the cameras' starts per point and
    // evaluation took both stages 434 us on 300,000 points of eight cameras, this 321).
    int cam0 = 0, cam_next = 0x7fffffff;  // of the group's first point; where the next one's begin
    bool cams_more = false;
    if (RIG && g.ncam > 0) {
      cam0 = cam_of(g.seg, g.ncam, g0);
      if (cam0 + 1 < g.ncam && g.seg[cam0 + 1] - g0 < pts) cam_next = (int)(g.seg[cam0 + 1] - g0);
      cams_more = cam0 + 2 < g.ncam && g.seg[cam0 + 2] - g0 < pts;
    }
    // point k of this thread; past the end some other one, not used
    auto fetch = [&](int k) {
      GNPt t;
      t.cam = 0;
      const int item = k * kGNThreads + (int)threadIdx.x;
      t.use = item < items;
      if (pts > 0) {
        unsigned i = t.use ? item : last;
        if (from_set) {
          i = list[i];
          t.use = t.use && i != kGNNone;
          i = t.use ? i : 0;
        }
        t.X = at_u32(GX, i); t.Y = at_u32(GY, i); t.Z = at_u32(GZ, i); t.u = at_u32(GU, i); t.v = at_u32(GV, i);
        t.w = at_u32(GW, i);
        if (RIG && g.ncam > 0)
          t.cam = cams_more ? cam_of(g.seg, g.ncam, g0 + i) : cam0 + ((int)i >= cam_next ? 1 : 0);
      }
      return t;
    };
    GNPt next = fetch(0);
    for (int k = 0; k < steps; ++k) {
      GNPt t = next;
      next = fetch(k + 1);
      t.u = t.use ? t.u : __builtin_nanf("");
      t.w = t.use ? (has_w ? t.w : 1.0f) : 0.0f;
      const bool take = gn_point<MODE, RIG>(g, s_rig, pose, first, t, a);
      const uint64_t bal = __ballot(take);
      count += __popcll(bal);
      if (MODE == 1 && first) {  // rank in point order: the waves' counts of this slice
        int* cnt = L.kept[k & 1];
        if (lane == 0) cnt[wave] = __popcll(bal);
        lds_barrier();
        int at = kept + __popcll(bal & ((1ull << lane) - 1ull));
  #pragma unroll
        for (int w = 0; w < kGNWaves; ++w) {
          at += w < wave ? cnt[w] : 0;
          kept += cnt[w];
        }
        if (take) list[at] = (uint16_t)(k * kGNThreads + (int)threadIdx.x);
      } else if (from_set && bal == 0) {
        break;  // (past the end of the list: it is dense)
      }
    }
  }
  if (MODE == 1 && first && !resident)
    for (int e = kept + (int)threadIdx.x; e < pts; e += kGNThreads) list[e] = kGNNone;
  a[28] = lane == 0 ? (double)count : 0.0;
  const double tot = wave_sum29(a);
  double (*rows)[kAcc] = L.rows[turn & 1];
  if ((lane & 1) == 0 && (lane >> 1) < kAcc) rows[wave][lane >> 1] = tot;
  if (MODE == 1 && first) __syncthreads();  // (also publishes the in-set to the other waves)
  else lds_barrier();
  double sum = 0.0;
  if ((int)threadIdx.x < kAcc) {
#pragma unroll
    for (int w = 0; w < kGNWaves; ++w) sum += rows[w][threadIdx.x];
  }
  return sum;
}

// A word pair of a mailbox: one value and the tag of its evaluation (the low
// halves of all values, then the high ones: whole cache lines per load).
constexpr int kBoxHigh = 32;
__device__ __forceinline__ void box_put(uint64_t* w, double v, unsigned tag) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  __hip_atomic_store(w, (b << 32) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(w + kBoxHigh, (b & 0xffffffff00000000ull) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The sums of groups [b0, b0 + nb) into L.in: every thread polls its values
// together (one memory latency, not one per value).  A group that has not
// come after `most` polls is marked in L.miss.
__device__ __forceinline__ void box_get(GNLds& L, const uint64_t* box, int b0, int nb, unsigned tag, int most) {
  constexpr int kPer = (kGNInBlock * kAcc + kGNThreads - 1) / kGNThreads;  // values per thread
  bool need[kPer];
  int at[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int e = (int)threadIdx.x + u * kGNThreads;
    need[u] = e < nb * kAcc;
    const int gi = e / kAcc;
    at[u] = gi * kGNBox + (e - gi * kAcc);
  }
  const int per = (nb * kAcc + kGNThreads - 1) / kGNThreads;
  for (int n = 0;; ++n) {
    uint64_t lo[kPer], hi[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      if (u >= per) break;
      const uint64_t* w = box + (int64_t)b0 * kGNBox + (need[u] ? at[u] : 0);
      lo[u] = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      hi[u] = __hip_atomic_load(w + kBoxHigh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    bool wait = false;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      if (u >= per || !need[u]) continue;
      if ((unsigned)lo[u] == tag && (unsigned)hi[u] == tag) {
        const int gi = at[u] / kGNBox;
        L.in[gi][at[u] - gi * kGNBox] =
            __longlong_as_double((long long)((hi[u] & 0xffffffff00000000ull) | (lo[u] >> 32)));
        need[u] = false;
      } else {
        wait = true;
      }
    }
    if (!wait) break;
    if (n >= most) {
#pragma unroll
      for (int u = 0; u < kPer; ++u)
        if (need[u]) atomicOr(&L.miss, 1ull << (at[u] / kGNBox));
      break;
    }
  }
}

// A member's whole run.  Tickets count query by query, problem by problem,
// member by member (QueryDesc::lo_team0 / fin_team0 are the running totals).
template <int MODE, bool RIG, bool RES>
__global__ __launch_bounds__(kGNThreads)
__attribute__((amdgpu_waves_per_eu(RES || RIG ? 2 : kGNWavesMany, RES || RIG ? 2 : kGNWavesMany))) void gn_team_kernel(
    GNArgs g) {
  __shared__ GNLds L;
  __shared__ double s_rig[RIG ? kMaxCams * kGNRig : 1];
  extern __shared__ GNResident s_resident[];
  GNResident& R = s_resident[0];
  const int tid = threadIdx.x;
  if (tid == 0) {
    L.role = g.ticket ? atomicAdd(g.ticket, 1) : (int)blockIdx.x;
    L.miss = 0;
    L.alone = 0;
  }
  __syncthreads();
  const int role = __builtin_amdgcn_readfirstlane(L.role);  // (uniform: descriptors come by scalar loads)
  int q = 0;
  // the last query whose first ticket is not above this one: 256 probes a step
  // (one look at every query took both launches 51 ms on 65,535 queries of 100
  // points, this 7.0; on 16,384 of 200 points 4.0, 1.9; on 4,096 of 300 0.65, 0.53)
  if (g.nq > 1) {
    int n = g.nq;
    do {
      const int step = (n + kGNThreads - 1) / kGNThreads, i = tid * step;
      const int t0 = i < n ? (MODE == 0 ? g.qd[q + i].lo_team0 : g.qd[q + i].fin_team0) : 0x7fffffff;
      const int below = __syncthreads_count(t0 <= role) - 1;
      q = __builtin_amdgcn_readfirstlane(q + below * step);
      n = min(step, n - below * step);
    } while (n > 1);
  }
  const QueryDesc& d = g.qd[q];
  const int T = g.start_direct ? g.team_direct : (MODE == 0 ? d.lo_team : d.fin_team);
  const int local = role - (g.start_direct ? 0 : (MODE == 0 ? d.lo_team0 : d.fin_team0));
  const int slot = local / T, member = local - slot * T;
  const int p = MODE == 0 ? q * g.kmax + slot : q;  // the problem: its mailboxes and outputs
  bool live = true;
  if (!g.start_direct) live = MODE == 0 ? slot < g.n_sel[q] : (g.bst[q].finished == 1) & (g.bst[q].have != 0);
  GNView v;
  v.c = MODE == 0 ? d.S : d.full;
  v.n = MODE == 0 ? d.m : d.n;
  const int G = groups_for(v.n), S = gn_group_points(v.n);
  if (!live) {
    // a finished query without a pose gets an all-zero mask
    if (MODE == 1 && g.write_mask && d.mask && g.bst[q].finished == 1)
      for (int grp = member; grp < G; grp += T)
        for (int e = tid; e < S; e += kGNThreads)
          if ((int64_t)grp * S + e < v.n) d.mask[(int64_t)grp * S + e] = 0;
    return;
  }
  v.ncam = d.ncam;
  v.seg = MODE == 0 ? d.segS : d.segF;
  v.ifx = uniform(1.0 / d.fx);
  v.ify = uniform(1.0 / d.fy);
  v.ucx = uniform(-d.cx * v.ifx);
  v.vcy = uniform(-d.cy * v.ify);
  v.fx2 = uniform(d.fx * d.fx);
  v.fy2 = uniform(d.fy * d.fy);
  v.tau2 = uniform(d.tau * d.tau);
  const double s2 = uniform(d.cauchy_s * d.cauchy_s);
  v.inv_s2 = uniform(1.0 / s2);
  const bool resident = RES && G <= T && S <= kGNGroup;
  const int iters = MODE == 0 ? d.lo_iters : d.final_iters;
  if (resident && v.n > 0) {
    const int64_t g0 = (int64_t)member * S;
    gn_load_resident<RIG>(R, v, g0, (int)(v.n - g0 < S ? v.n - g0 : S));
  }
  const double* start = g.start_direct ? g.start_direct + 12 * (int64_t)p
                        : MODE == 0    ? g.cb.pose + 12 * (d.cand_off + g.sel[q * kMaxTopK + slot])
                                       : g.bst[q].pose;
  if (tid < 12) L.s.cur[tid] = L.s.eval[tid] = L.s.start[tid] = start[tid];
  if (RIG && tid < d.ncam) {  // R, t, then the camera's scales
    const double* rc = d.rig + 16 * tid;
    double* o = s_rig + kGNRig * tid;
    for (int e = 0; e < 12; ++e) o[e] = rc[4 + e];
    o[12] = 1.0 / rc[0];
    o[13] = 1.0 / rc[1];
    o[14] = -rc[2] * o[12];
    o[15] = -rc[3] * o[13];
    o[16] = rc[0] * rc[0];
    o[17] = rc[1] * rc[1];
  }
  __syncthreads();
  uint16_t* lists = MODE == 1 ? reinterpret_cast<uint16_t*>(g.in_set_all + d.in_set_off) : nullptr;
  // tags of this round's evaluations (the mailboxes hold those of earlier rounds)
  const unsigned tag0 = MODE == 0 && g.bst ? (unsigned)g.bst[q].batches * 1024u : 0u;
  int n_in = 0, other_in = 0, turn = 0;
  double best_cost = 0.0, best_count = 0.0;  // (wave 0)
  for (int j = 0;; ++j) {
    uint64_t* box = g.box + ((int64_t)p * 2 + (j & 1)) * g.box_groups * kGNBox;
    const unsigned tag = tag0 + (unsigned)j + 1u;
    double tot = 0.0;
    // The groups of this evaluation: the member's own, then (T > 1) block by
    // block those of the others from their mailboxes, and of these the
    // missing ones from their points (alone; the refinement lists their set
    // first).  One loop, so that the evaluation is in the code once.
    int grp = member, b0 = -kGNInBlock, nb = 0;
    unsigned long long miss = 0;
    bool own = true, listed = MODE == 0 || j == 0;
    for (;;) {
      if (own ? grp < G : miss != 0) {
        const int gi = own ? 0 : __builtin_ctzll(miss);
        const int at = own ? grp : b0 + gi;
        const bool list_only = !own && !listed;
        const double sum = gn_eval_group<MODE, RIG, RES>(L, R, v, s_rig, list_only ? L.s.start : L.s.eval, at,
                                                    j == 0 || list_only, own && resident,
                                                    MODE == 1 ? lists + (int64_t)at * S : nullptr,
                                                    own ? n_in : other_in, turn++);
        if (own) {
          if (tid < kAcc) {
            if (T == 1) tot += sum;
            else box_put(box + (int64_t)grp * kGNBox + tid, sum, tag);
          }
          grp += T;
        } else if (list_only) {
          listed = true;
        } else {
          if (tid < kAcc) L.in[gi][tid] = sum;
          miss &= miss - 1;
          listed = MODE == 0 || j == 0;
        }
        continue;
      }
      if (T == 1) break;
      if (!own) {  // a block is complete
        if (tid < kAcc)
          for (int g0 = 0; g0 < nb; g0 += 8) {  // eight reads in flight, added in order
            double x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = L.in[g0 + u][tid];  // (kGNInBlock is a multiple of 8)
#pragma unroll
            for (int u = 0; u < 8; ++u)
              if (g0 + u < nb) tot += x[u];
          }
        if (b0 + kGNInBlock >= G) break;
        __syncthreads();  // before its slots are used again
      }
      own = false;
      b0 += kGNInBlock;
      nb = G - b0 < kGNInBlock ? G - b0 : kGNInBlock;
      box_get(L, box, b0, nb, tag, L.alone ? 0 : g.polls);
      __syncthreads();
      miss = L.miss;
      if (miss) {
        __syncthreads();
        if (tid == 0) {
          L.miss = 0;
          L.alone = 1;
        }
      }
    }
    if (tid < kWave) {  // wave 0: the same decision in every member
      if (tid < kAcc) L.tot[tid] = MODE == 1 && tid == 27 ? tot * s2 : tot;
      __builtin_amdgcn_wave_barrier();
      gn_decide_wave(j, iters, L.tot, L.s, best_cost, best_count);
    }
    __syncthreads();
    if (L.s.done) break;
  }
  if (member == 0) {
    if (tid < 12 && g.out_pose) g.out_pose[12 * (int64_t)p + tid] = L.s.cur[tid];
    if (tid == 0) {
      if (g.out_cost) g.out_cost[p] = best_cost;
      if (g.out_count) g.out_count[p] = (int64_t)best_count;
    }
  }
  if (MODE == 1 && g.write_mask) {
    long long cnt = 0;
    for (int grp = member; grp < G; grp += T)
      for (int e = tid; e < S; e += kGNThreads) {
        const int64_t i = (int64_t)grp * S + e;
        if (i >= v.n) break;
        const bool in = mask_test(d, L.s.cur, gmem(v.c.X)[i], gmem(v.c.Y)[i], gmem(v.c.Z)[i], gmem(v.c.u)[i],
                                  gmem(v.c.v)[i], i);
        if (d.mask) d.mask[i] = in ? 1 : 0;
        cnt += in ? 1 : 0;
      }
    // one add per member to the query's counter (same-address atomics serialise)
    __shared__ long long s_cnt[kGNWaves];
    cnt = wave_sum(cnt);
    if ((tid & (kWave - 1)) == 0) s_cnt[tid / kWave] = cnt;
    __syncthreads();
    if (tid == 0) {
      long long sum = 0;
#pragma unroll
      for (int w = 0; w < kGNWaves; ++w) sum += s_cnt[w];
      if (sum) atomicAdd((unsigned long long*)&g.bst[q].full_count, (unsigned long long)sum);
    }
  }
}

template <int MODE>
static void launch_team(const GNArgs& g, const GNLaunch& t, bool any_rig, hipStream_t s) {
  const dim3 grid(t.members), block(kGNThreads);
  const size_t lds = t.resident ? sizeof(GNResident) : 0;
  if (any_rig) {
    if (t.resident) hipLaunchKernelGGL((gn_team_kernel<MODE, true, true>), grid, block, lds, s, g);
    else hipLaunchKernelGGL((gn_team_kernel<MODE, true, false>), grid, block, lds, s, g);
  } else {
    if (t.resident) hipLaunchKernelGGL((gn_team_kernel<MODE, false, true>), grid, block, lds, s, g);
    else hipLaunchKernelGGL((gn_team_kernel<MODE, false, false>), grid, block, lds, s, g);
  }
}

hipError_t launch_lo(const QueryDesc* qd, const BestState* st, CandBuf cb, const int32_t* sel, const int32_t* n_sel,
                     const double* start_direct, int nq, int kmax, const GNLaunch& t, double* out_pose,
                     double* out_cost, int64_t* out_count, bool any_rig, hipStream_t s) {
  if (t.members <= 0) return hipSuccess;
  GNArgs g{};
  g.qd = qd;
  g.cb = cb;
  g.sel = sel;
  g.n_sel = n_sel;
  g.start_direct = start_direct;
  g.bst = const_cast<BestState*>(st);
  g.box = t.box;
  g.out_pose = out_pose;
  g.out_cost = out_cost;
  g.out_count = out_count;
  g.ticket = t.teams ? t.ticket : nullptr;
  g.nq = nq;
  g.kmax = kmax;
  g.box_groups = t.box_groups;
  g.team_direct = t.team_direct;
  g.polls = t.polls;
  launch_team<0>(g, t, any_rig, s);
  return hipGetLastError();
}

hipError_t launch_refine(const QueryDesc* qd, BestState* bst, const double* start_direct, int nq, const GNLaunch& t,
                         uint8_t* in_set, double* out_pose, double* out_cost, bool any_rig, bool write_mask,
                         hipStream_t s) {
  if (t.members <= 0) return hipSuccess;
  GNArgs g{};
  g.qd = qd;
  g.bst = bst;
  g.start_direct = start_direct;
  g.box = t.box;
  g.in_set_all = in_set;
  g.out_pose = out_pose;
  g.out_cost = out_cost;
  g.ticket = t.teams ? t.ticket : nullptr;
  g.nq = nq;
  g.kmax = 1;
  g.box_groups = t.box_groups;
  g.team_direct = t.team_direct;
  g.write_mask = write_mask ? 1 : 0;
  g.polls = t.polls;
  launch_team<1>(g, t, any_rig, s);
  return hipGetLastError();
}

}  // namespace imloc
