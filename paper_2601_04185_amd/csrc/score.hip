// score.hip -- hypothesis scoring, the hot loop of LO-RANSAC (ImLoc Sec. 3.3:
// every pose hypothesis is scored against every scored correspondence by a
// confidence-weighted truncated squared reprojection error), and the
// per-query top-k selection of the candidates to refine.
//
// Work decomposition: a work item is (query, tile of CT candidates, chunk of
// 256 * PPL correspondences); persistent workgroups walk a device-side work
// list, so one launch covers any mix of queries.
//
// Layout: one lane per correspondence (PPL correspondences per lane kept in
// registers, coalesced structure-of-arrays loads).  A work item first stages
// its tile's projection rows in LDS; each wave then reads a candidate's rows
// with broadcast LDS loads into vector registers, so that every multiply-add
// of the loop has vector operands only (on gfx950 a multiply-add with a
// scalar-register operand issues about 1.7 times slower, one with a neg or
// abs modifier about 1.5 times).  The rows are K [R | t] with the first two
// divided by tau, and the observations enter divided by tau and negated, so
// per residual:
//   (a', b', w) = P' [X, 1]              9 FMA
//   du' = a' + (-u') w, dv' likewise     2 FMA
//   e' = du'^2 + dv'^2                   MUL + FMA    (= e / tau^2)
//   inlier iff e' - w |w| < 0            FMA + CMP    (one rounding; rejects w <= 0 and NaN)
// The inlier count is a wave ballot + popcount (scalar unit).  The truncated
// cost is MSAC = tau^2 (sum_i w_i - G), G = sum_in w_i (w |w| - e')/(w |w|),
// computed only in point slots whose ballot is not empty (a wave-uniform
// branch), so most candidates pay no reciprocal at all.
//
// Accumulation: each wave's partial G (a float sum over its fixed set of
// 64 * PPL correspondences) is converted once to fixed point (2^-32) and all
// partials are added with integer atomics, as are the counts.  Integer sums
// do not depend on the order, so a candidate's score is the same for any
// tiling, grid size or mix of queries.  The tables in LDS start at zero and
// only a wave block with inliers adds to them; the conversion to fixed point
// happens once per block for all candidates, off the candidate loop.
#include <type_traits>

#include "imloc_device.h"
#include "imloc_kernels.h"
#include "query_device.h"
#include "select_key.h"

namespace imloc {

constexpr int kScoreBlock = 256;
constexpr int kScoreWaves = kScoreBlock / kWave;

// Sum over the 64 lanes of a full wave with DPP lane moves (pairs, quads,
// rows of 16 by shifts, then the row broadcasts 15 and 31); lane 63 ends with
// the total.  Every lane must be active.
template <int CTRL>
__device__ inline float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ inline float wave_scan_dpp(float x) {
  x += dpp_move<0xb1>(x);   // quad_perm [1, 0, 3, 2]
  x += dpp_move<0x4e>(x);   // quad_perm [2, 3, 0, 1]
  x += dpp_move<0x114>(x);  // row_shr:4
  x += dpp_move<0x118>(x);  // row_shr:8
  x += dpp_move<0x142>(x);  // row_bcast:15
  x += dpp_move<0x143>(x);  // row_bcast:31
  return x;  // lane 63 holds the total
}

// Correspondences per work item: `pts` in float32 scoring (a multiple of the
// 512-correspondence wave block), 256 * kScorePPL64 in float64 scoring.
__device__ inline int64_t chunk_pts(const QueryDesc& d, int pts) {
  return d.precision ? (int64_t)kScoreBlock * kScorePPL64 : (int64_t)pts;
}
__device__ inline int64_t chunks_of(const QueryDesc& d, int pts) {
  const int64_t per = chunk_pts(d, pts);
  int64_t c = 0;
  if (d.ncam == 0) {
    c = (d.m + per - 1) / per;
  } else {  // a rig: every camera's segment is chunked on its own
    for (int k = 0; k < d.ncam; ++k) c += (d.segS[k + 1] - d.segS[k] + per - 1) / per;
  }
  return c > 0 ? c : 1;
}

// Points [begin, end) and camera of chunk `chunk` of the scoring set.
struct ChunkRange {
  int64_t begin, end;
  int cam;
};
__device__ inline ChunkRange chunk_range(const QueryDesc& d, int64_t chunk, int pts) {
  const int64_t per = chunk_pts(d, pts);
  if (d.ncam == 0) return ChunkRange{chunk * per, d.m, 0};
  for (int k = 0; k < d.ncam; ++k) {
    const int64_t nch = (d.segS[k + 1] - d.segS[k] + per - 1) / per;
    if (chunk < nch) return ChunkRange{d.segS[k] + chunk * per, d.segS[k + 1], k};
    chunk -= nch;
  }
  return ChunkRange{0, 0, 0};
}


// Work list: items_q = tiles_q * chunks_q for queries sampling this round;
// item_off = exclusive prefix, item_off[nq] = total (one workgroup).  A round of
// one query has no list: its scoring counts its items itself (5 us less).
__global__ __launch_bounds__(1024) void worklist_kernel(const QueryDesc* __restrict__ qd,
                                                        const int32_t* __restrict__ n_cand, int nq, int ct, int pts,
                                                        int64_t* __restrict__ item_off) {
  __shared__ long long s[1024];
  const int seg = (nq + 1023) / 1024;
  const int q0 = threadIdx.x * seg, q1 = min(nq, q0 + seg);
  long long sum = 0;
  for (int q = q0; q < q1; ++q) {
    const QueryDesc& d = qd[q];
    if (d.B > 0) sum += (long long)((n_cand[q] + ct - 1) / ct) * chunks_of(d, pts);
  }
  s[threadIdx.x] = sum;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const long long v = (int)threadIdx.x >= off ? s[threadIdx.x - off] : 0;
    __syncthreads();
    s[threadIdx.x] += v;
    __syncthreads();
  }
  long long run = s[threadIdx.x] - sum;
  for (int q = q0; q < q1; ++q) {
    item_off[q] = run;
    const QueryDesc& d = qd[q];
    if (d.B > 0) run += (long long)((n_cand[q] + ct - 1) / ct) * chunks_of(d, pts);
  }
  if (threadIdx.x == 1023) item_off[nq] = s[1023];
}

hipError_t launch_worklist(const QueryDesc* qd, CandBuf cb, int nq, ScoreTune tune, int64_t* item_off,
                           hipStream_t s) {
  if (nq <= 1) return hipSuccess;
  hipLaunchKernelGGL(worklist_kernel, dim3(1), dim3(1024), 0, s, qd, cb.n, nq, tune.ct, tune.pts, item_off);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The filter of float32 items.  Most candidates are wrong and see hardly any
// correspondence inside the threshold (of the (candidate, 512 correspondences)
// pairs of a round of random P3P samples one in five has one, of the 64-wide
// slots one in 27), so before a wave evaluates a candidate (15 vector
// instructions per residual) the matrix cores rule out the slots that cannot
// hold an inlier.
//
// du', dv' and w are linear in twelve features of a correspondence, X~ = (X, Y,
// Z, 1), p_u X~ and p_v X~ (p = -observation / tau), with the candidate's rows
// as coefficients, so one 32x32x16 product in float16 gives each of them for 32
// correspondences x 32 candidates.  An inlier has |du'| < w and |dv'| < w; a
// slot passes if a correspondence has max(|Du|, |Dv|) < W + E, E bounding the
// error of the float16 values and of the float32 evaluation (it rides on a
// constant feature of W).  Slots that pass are evaluated exactly as without the
// filter, so counts and partial sums do not change in a single bit.
//
// Features are shifted by the middle and divided by the half range of the
// item's correspondences, so that they lie in [-1, 1] and round with an error
// of at most 2^-12 each; a candidate's coefficients are scaled by a power of
// two that brings their sum to 2^13 .. 2^14 (float16 ends at 65504), and what
// their rounding costs is summed as it comes out.  To these two E adds 25 x
// 2^-14 for coefficients that are flushed to zero, and 2^-19 of the terms'
// magnitudes for the 16 additions of a product, the float32 evaluation and the
// shift (about 2^-21 each).  What is not finite passes.
//
// Per 1,024 residuals the three products and the 43 vector instructions on
// their results take 186 cycles of a SIMD (matrix and vector instructions of
// different waves hardly overlap here: 38 cycles a product, 2.5 an
// instruction; four products w +- du', w +- dv' and two bit operations
// instead of the subtraction and the median take 195), the exact evaluation of
// all 640.  256 queries of 5,000 to 80,000 correspondences, 5,570 candidates
// each: 17.7 -> 9.98 ms, of it products 5.8, features and coefficients 1.2,
// exact evaluation 2.8 (with the pairs below 9.6); 50,000 x 13,400: 228 -> 136
// us; 50,000 x 4,096, 6 % of them good: 85 -> 52 us; 10,000 x 1,360: 21 -> 18 us.
// Three waves per SIMD (168 registers); four spill and two leave latency open
// (10.4, 13.5 ms beside the 9.98).
//
// Where most candidates are good (poses given from elsewhere), most slots pass.
// A wave that sees three quarters of its first 32 candidates pass the first slot
// lets the others pass too: from 0.71 on, 186 cycles cost more than they save of
// 640.  And candidates that pass in every slot are evaluated two at a time in
// straight code, since three waves per SIMD do not cover the latency of a single
// one's reciprocals and lane sum.  50,000 x 4,096 poses, all of them good: 211 us
// with neither, 186 with the pairs, 156 with both (130 without a filter at five
// waves per SIMD); half of them good 117 (108), a third 94 (100), none 47 (83).
//
// Rounds in which the filter does not pay (round_tune) take a kernel without it,
// which has registers for four waves per SIMD.
// ---------------------------------------------------------------------------
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
constexpr int kFilterTile = 32;   // candidates, and correspondences, of one product
// candidates of a tile from which the filter pays: its products cost 16 x 186
// cycles per wave block and 32 candidates, the evaluation 320 per candidate
constexpr int kFilterLeast = 12;

// Middle and half range of an item's X, Y, Z, p_u, p_v.
struct FilterRange {
  float mid[5], half[5];
};

__device__ inline float wave_uniform(float x) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

// Minimum / maximum over the wave, in lane 63.
template <bool MAX>
__device__ inline float wave_extreme(float x) {
  auto pick = [&](auto ctrl) {
    const float y = __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, false));
    x = MAX ? fmaxf(x, y) : fminf(x, y);
  };
  pick(std::integral_constant<int, 0xb1>{});
  pick(std::integral_constant<int, 0x4e>{});
  pick(std::integral_constant<int, 0x114>{});
  pick(std::integral_constant<int, 0x118>{});
  pick(std::integral_constant<int, 0x142>{});
  pick(std::integral_constant<int, 0x143>{});
  return x;
}

// Coefficients of one candidate for the three products, 16 each.
__device__ inline void filter_rows(const float4 r0, const float4 r1, const float4 r2, const FilterRange& f,
                                   half8 (&out)[3][2]) {
  const float* c = f.mid;
  const float* s = f.half;
  // the rows of du' and dv' with the middle of the observations folded in
  const float u[4] = {fmaf(c[3], r2.x, r0.x), fmaf(c[3], r2.y, r0.y), fmaf(c[3], r2.z, r0.z), fmaf(c[3], r2.w, r0.w)};
  const float v[4] = {fmaf(c[4], r2.x, r1.x), fmaf(c[4], r2.y, r1.y), fmaf(c[4], r2.z, r1.z), fmaf(c[4], r2.w, r1.w)};
  auto at_mid = [&](float x, float y, float z, float w) { return fmaf(x, c[0], fmaf(y, c[1], fmaf(z, c[2], w))); };
  float cu[4] = {u[0] * s[0], u[1] * s[1], u[2] * s[2], at_mid(u[0], u[1], u[2], u[3])};
  float cv[4] = {v[0] * s[0], v[1] * s[1], v[2] * s[2], at_mid(v[0], v[1], v[2], v[3])};
  float cw[4] = {r2.x * s[0], r2.y * s[1], r2.z * s[2], at_mid(r2.x, r2.y, r2.z, r2.w)};
  const float w3 = fabsf(cw[0]) + fabsf(cw[1]) + fabsf(cw[2]), sw = w3 + fabsf(cw[3]);
  const float u3 = fabsf(cu[0]) + fabsf(cu[1]) + fabsf(cu[2]) + s[3] * sw;
  const float v3 = fabsf(cv[0]) + fabsf(cv[1]) + fabsf(cv[2]) + s[4] * sw;
  const float sum = fmaxf(u3 + fabsf(cu[3]), v3 + fabsf(cv[3])) + sw;
  // magnitudes of the terms before the shift
  const float ax = fabsf(c[0]) + s[0], ay = fabsf(c[1]) + s[1], az = fabsf(c[2]) + s[2];
  const float au = fabsf(c[3]) + s[3], av = fabsf(c[4]) + s[4];
  auto mag = [&](const float4& r) { return fabsf(r.x) * ax + fabsf(r.y) * ay + fabsf(r.z) * az + fabsf(r.w); };
  const float mw = mag(r2);
  const float big = fmaxf(mag(r0) + au * mw, mag(r1) + av * mw) + mw;
  bool fine = big < 1e30f && sum < 1e30f && sum > 1e-30f;  // (false for NaN)
  const int ex = fine ? 14 - __builtin_amdgcn_frexp_expf(sum) : 0;
  float eu = 0.f, ev = 0.f, ew = 0.f;  // what the rounding of the coefficients costs
  auto h = [&](float x, float& err) {
    const float y = ldexpf(x, ex);
    const _Float16 z = (_Float16)y;
    err += fabsf(y - (float)z);
    return z;
  };
  const _Float16 zero = (_Float16)0.f;
  out[0][0] = half8{h(cu[0], eu), h(cu[1], eu), h(cu[2], eu), h(cu[3], eu),
                    h(cw[0] * s[3], eu), h(cw[1] * s[3], eu), h(cw[2] * s[3], eu), h(cw[3] * s[3], eu)};
  out[0][1] = half8{zero, zero, zero, zero, zero, zero, zero, zero};
  out[1][0] = half8{h(cv[0], ev), h(cv[1], ev), h(cv[2], ev), h(cv[3], ev), zero, zero, zero, zero};
  out[1][1] = half8{h(cw[0] * s[4], ev), h(cw[1] * s[4], ev), h(cw[2] * s[4], ev), h(cw[3] * s[4], ev),
                    zero, zero, zero, zero};
  out[2][0] = half8{h(cw[0], ew), h(cw[1], ew), h(cw[2], ew), h(cw[3], ew), zero, zero, zero, zero};
  const float E = fmaxf(eu, ev) + ew + ldexpf((fmaxf(u3, v3) + w3) * (1.01f / 4096.f) + (big + sum) * (1.f / 524288.f), ex) +
                  25.f / 16384.f;
  fine = fine && E < 60000.f;
  // (1.002: the bound itself is rounded)
  out[2][1] = half8{zero, zero, zero, zero, (_Float16)(fine ? E * 1.002f : 1.f), zero, zero, zero};
  if (!fine) {  // W + E = 1, Du = Dv = 0: passes
    const half8 none = {zero, zero, zero, zero, zero, zero, zero, zero};
    out[0][0] = out[1][0] = out[1][1] = out[2][0] = none;
  }
}

// Candidates of a tile: alike over the ceil(n / CT) tiles, in steps of a
// product.  Full tiles and a rest would repeat with the queries, in step with the
// turn in which workgroups go to the parts of the chip, so that some parts get the
// rests alone: 4,096 queries x 350 candidates x 2,000 correspondences (two tiles
// of 256) 1,270 -> 995 us, 1,024 x 348 x 8,000 908 -> 706.
template <int CT>
__device__ inline int tile_candidates(int n) {
  const int tiles = (n + CT - 1) / CT;
  return ((n + tiles - 1) / tiles + kFilterTile - 1) / kFilterTile * kFilterTile;
}

// Tables of a work item in LDS.
template <int CT>
struct ScoreTables {
  float4 rows[CT][3];                         // projections of the tile's candidates
  union {
    half8 coef[CT / kFilterTile][3][2][kFilterTile];  // and their coefficients of the filter
    double rows64[CT][12];                            // float64 items: the projections
  };
  float ext[kScoreWaves][2][5];                 // the waves' ranges
  uint32_t cnt[CT];                             // inliers so far
  unsigned long long gain[CT];                  // G so far (fixed point)
  float part[kScoreWaves][CT];                  // G of the waves' present blocks
  uint32_t item[kScoreWaves];
};

// The item's sums to the candidates, and the tables empty again.
template <int CT>
__device__ __forceinline__ void score_item_end(const QueryDesc& d, uint32_t* __restrict__ ccnt,
                                               unsigned long long* __restrict__ cgain, BestState* st, int c0, int cend,
                                               ScoreTables<CT>& T) {
  __syncthreads();
  const int c = threadIdx.x;
  if (c < cend) {
    const int64_t slot = d.cand_off + c0 + c;
    const uint32_t cnt = T.cnt[c];
    const unsigned long long g = T.gain[c];
    if (cnt) atomicAdd(&ccnt[slot], cnt);
    if (g) atomicAdd(&cgain[slot], g);
    T.cnt[c] = 0;
    T.gain[c] = 0;
  }
  if (c == 0) {  // one add per item to the query's counter (same-address atomics serialise)
    unsigned long long tot = 0;
#pragma unroll
    for (int w = 0; w < kScoreWaves; ++w) tot += T.item[w];
    if (tot) atomicAdd((unsigned long long*)&st->inlier_residuals, tot);
  }
  __syncthreads();
}

// One float32 work item: CT candidates against pts correspondences.  The
// correspondences come in wave blocks of 512 (lane l, slot k: block start +
// 64 k + l); every (candidate, wave block) pair is scored by exactly one wave,
// whose count and gain partial (a float sum over that block, converted once
// to fixed point) are added as integers, so the results do not depend on
// pts.  pts >= 2048: each wave takes blocks w, w + 4, ... for every
// candidate; pts < 2048: the waves split into 2048 / pts candidate groups,
// each of pts / 512 waves.  Between the blocks no wave waits for another.
template <int CT, bool FILTER>
__device__ __forceinline__ void score_item_f32(const QueryDesc& d, const float* __restrict__ proj,
                                               uint32_t* __restrict__ ccnt, unsigned long long* __restrict__ cgain,
                                               BestState* st, int64_t tile, int64_t chunk, int ncand, int pts,
                                               ScoreTables<CT>& T) {
  constexpr int PPL = kScorePPL32;
  // the wave index in a scalar register: the candidate range and the block
  // derived from it are wave-uniform, so the candidate loop stays scalar
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // (addresses derived from it are not kept over the items: registers)
  const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const float inv_tau = (float)(1.0 / d.tau);
  const ChunkRange rg = chunk_range(d, chunk, pts);
  const int per = tile_candidates<CT>(ncand), c0 = (int)tile * per;
  const int cend = min(per, ncand - c0);
  const int wpg = min(kScoreWaves, pts / kScoreWaveBlock);  // waves per candidate group
  const int grp = wave / wpg, gsz = CT * wpg / kScoreWaves;
  const int cg0 = grp * gsz, cg1 = min(cend, cg0 + gsz);
  // correspondences and wave blocks of the item
  const int npt = (int)max((int64_t)0, min(rg.end - rg.begin, (int64_t)pts));
  const int nblk = (npt + kScoreWaveBlock - 1) / kScoreWaveBlock;
  const bool filter = FILTER && gsz >= kFilterTile && cend >= kFilterLeast;
  // the tile's projection rows into LDS: every wave then reads a candidate's
  // 12 values as three broadcast 16-byte LDS loads into vector registers
  // (a multiply-add with a scalar-register operand issues about 1.7 times
  // slower than one with vector operands only on this chip)
  {
    const int rows = rows_per_slot(d);
    const float4* __restrict__ pc =
        reinterpret_cast<const float4*>(proj + d.proj_off + 16 * ((int64_t)rows * c0 + rg.cam));
    for (int e = tid; e < 3 * cend; e += kScoreBlock) {
      const int c = e / 3, r = e - 3 * c;
      T.rows[c][r] = pc[(int64_t)4 * rows * c + r];
    }
  }
  const auto U = gmem(d.S.u) + rg.begin;
  const auto V = gmem(d.S.v) + rg.begin;
  const auto X = gmem(d.S.X) + rg.begin;
  const auto Y = gmem(d.S.Y) + rg.begin;
  const auto Z = gmem(d.S.Z) + rg.begin;
  const auto W = gmem(d.S.w);
  float pu[PPL], pv[PPL], px[PPL], py[PPL], pz[PPL], pw[PPL];
  // the lane's correspondences of a block; past the end the last one again
  // (observations negated, so that du' = a' + pu w is a multiply-add without modifiers)
  auto load = [&](int blk) {
#pragma unroll
    for (int k = 0; k < PPL; ++k) {
      const int i = min(blk * kScoreWaveBlock + k * kWave + lane, npt - 1);
      pu[k] = -(U[i] * inv_tau); pv[k] = -(V[i] * inv_tau); px[k] = X[i]; py[k] = Y[i]; pz[k] = Z[i];
    }
  };
  // past the end a NaN residual, never an inlier
  auto mask_ends = [&](int blk) {
#pragma unroll
    for (int k = 0; k < PPL; ++k)
      if (blk * kScoreWaveBlock + k * kWave + lane >= npt) pu[k] = __builtin_nanf("");
  };
  auto load_weights = [&](int blk) {
#pragma unroll
    for (int k = 0; k < PPL; ++k) {
      const int i = min(blk * kScoreWaveBlock + k * kWave + lane, npt - 1);
      pw[k] = W ? W[rg.begin + i] : 1.0f;
    }
  };
  uint32_t item_cnt = 0;
  // Candidate c on the wave's block, the slots of a mask.
  //   inlier iff e' < w |w|: the sign of e' - w |w| rounded once (rejects w <= 0 and NaN)
  //   G += w_i (w|w| - e') / (w|w|) over the inliers, slots with no inlier skipped
  // (the empty volatile statements keep the wave-uniform branches as branches)
  auto residual = [&](const float4& r0, const float4& r1, const float4& r2, int k, float& w) {
    const float a = fmaf(r0.z, pz[k], fmaf(r0.y, py[k], fmaf(r0.x, px[k], r0.w)));
    const float b = fmaf(r1.z, pz[k], fmaf(r1.y, py[k], fmaf(r1.x, px[k], r1.w)));
    w = fmaf(r2.z, pz[k], fmaf(r2.y, py[k], fmaf(r2.x, px[k], r2.w)));
    const float du = fmaf(pu[k], w, a), dv = fmaf(pv[k], w, b);
    return fmaf(-w, fabsf(w), fmaf(dv, dv, du * du));
  };
  auto add_gain = [&](float dd, float w, int k, float& gain) {
    const float t = w * fabsf(w);
    if (dd < 0.f) gain = fmaf(-pw[k] * dd, __builtin_amdgcn_rcpf(t), gain);
  };
  auto put = [&](int c, uint32_t cnt, uint64_t lanes, float gain) {
    // a lone lane's gain is the sum: no scan
    uint64_t writer = lanes;
    if (lanes & (lanes - 1)) {
      gain = wave_scan_dpp(gain);  // the block's total in lane 63
      writer = 1ull << (kWave - 1);
    }
    if (__builtin_amdgcn_inverse_ballot_w64(writer)) {
      atomicAdd(&T.cnt[c], cnt);
      T.part[wave][c] = gain;
    }
    item_cnt += cnt;
  };
  auto evaluate = [&](int c) {  // all slots
    // (the other waves of the SIMD cover the LDS latency)
    const float4 r0 = T.rows[c][0], r1 = T.rows[c][1], r2 = T.rows[c][2];
    uint32_t cnt = 0;
    uint64_t bal[PPL], lanes = 0;
    float dd[PPL], ww[PPL];
#pragma unroll
    for (int k = 0; k < PPL; ++k) {
      dd[k] = residual(r0, r1, r2, k, ww[k]);
      bal[k] = __ballot(dd[k] < 0.f);
      cnt += (uint32_t)__popcll(bal[k]);
    }
    if (cnt) {
      asm volatile("");
      float gain = 0.f;
#pragma unroll
      for (int k = 0; k < PPL; ++k) {
        if (bal[k]) {
          asm volatile("");
          lanes |= bal[k];
          add_gain(dd[k], ww[k], k, gain);
        }
      }
      put(c, cnt, lanes, gain);
    }
  };
  // Two candidates, all slots, both sums at a time (the same terms in the same
  // order as one by one, so the same bits).
  auto evaluate_pair = [&](int ca, int cb) {
    float da[PPL], wa[PPL], db[PPL], wb[PPL];
    uint32_t na = 0, nb = 0;
    {
      const float4 r0 = T.rows[ca][0], r1 = T.rows[ca][1], r2 = T.rows[ca][2];
#pragma unroll
      for (int k = 0; k < PPL; ++k) {
        da[k] = residual(r0, r1, r2, k, wa[k]);
        na += (uint32_t)__popcll(__ballot(da[k] < 0.f));
      }
    }
    {
      const float4 r0 = T.rows[cb][0], r1 = T.rows[cb][1], r2 = T.rows[cb][2];
#pragma unroll
      for (int k = 0; k < PPL; ++k) {
        db[k] = residual(r0, r1, r2, k, wb[k]);
        nb += (uint32_t)__popcll(__ballot(db[k] < 0.f));
      }
    }
    if (na | nb) {
      float ga = 0.f, gb = 0.f;
#pragma unroll
      for (int k = 0; k < PPL; ++k) {
        asm("" : "+v"(da[k]), "+v"(db[k]));  // (compared again: 32 masks would not fit the scalar registers)
        const float xa = fmaf(-pw[k] * da[k], __builtin_amdgcn_rcpf(wa[k] * fabsf(wa[k])), ga);
        const float xb = fmaf(-pw[k] * db[k], __builtin_amdgcn_rcpf(wb[k] * fabsf(wb[k])), gb);
        ga = da[k] < 0.f ? xa : ga;
        gb = db[k] < 0.f ? xb : gb;
      }
      ga = wave_scan_dpp(ga);
      gb = wave_scan_dpp(gb);
      if (lane == kWave - 1) {
        if (na) {
          atomicAdd(&T.cnt[ca], na);
          T.part[wave][ca] = ga;
        }
        if (nb) {
          atomicAdd(&T.cnt[cb], nb);
          T.part[wave][cb] = gb;
        }
      }
      item_cnt += na + nb;
    }
  };
  auto evaluate_slots = [&](int c, uint32_t slots) {
    const float4 r0 = T.rows[c][0], r1 = T.rows[c][1], r2 = T.rows[c][2];
    uint32_t cnt = 0;
    uint64_t lanes = 0;
    float gain = 0.f;
#pragma unroll
    for (int k = 0; k < PPL; ++k) {
      if (slots & (1u << k)) {
        asm volatile("");
        float w;
        const float dd = residual(r0, r1, r2, k, w);
        const uint64_t bal = __ballot(dd < 0.f);
        if (bal) {
          asm volatile("");
          cnt += (uint32_t)__popcll(bal);
          lanes |= bal;
          add_gain(dd, w, k, gain);
        }
      }
    }
    if (cnt) put(c, cnt, lanes, gain);
  };
  // the block's float partials to fixed point
  auto flush = [&]() {
    for (int c = cg0 + lane; c < cg1; c += kWave) {
      const float p = T.part[wave][c];
      if (p != 0.f) {
        atomicAdd(&T.gain[c], (unsigned long long)((double)p * kGainScale));
        T.part[wave][c] = 0.f;
      }
    }
  };

  int blk = wave % wpg;
  if (blk < nblk) load(blk);
  if (!filter) {
    __syncthreads();  // the rows are staged
    for (; blk < nblk; blk += wpg) {
      if (blk != wave % wpg) load(blk);
      mask_ends(blk);
      load_weights(blk);
      for (int c = cg0; c < cg1; ++c) evaluate(c);
      flush();
    }
  } else {
    // range of the item's correspondences: lane, wave, workgroup
    {
      float lo[5], hi[5];
#pragma unroll
      for (int e = 0; e < 5; ++e) {
        lo[e] = __builtin_inff();
        hi[e] = -__builtin_inff();
      }
      auto widen = [&](int e, float x) {
        lo[e] = fminf(lo[e], x);
        hi[e] = fmaxf(hi[e], x);
      };
      for (int b = blk; b < nblk; b += wpg) {
        if (b != blk) load(b);
#pragma unroll
        for (int k = 0; k < PPL; ++k) {
          widen(0, px[k]);
          widen(1, py[k]);
          widen(2, pz[k]);
          widen(3, pu[k]);
          widen(4, pv[k]);
        }
      }
      if (blk + wpg < nblk) load(blk);
#pragma unroll
      for (int e = 0; e < 5; ++e) {
        const float l = wave_extreme<false>(lo[e]), h = wave_extreme<true>(hi[e]);
        if (lane == kWave - 1) {
          T.ext[wave][0][e] = l;
          T.ext[wave][1][e] = h;
        }
      }
    }
    __syncthreads();  // the rows are staged, the ranges written
    FilterRange f;
    float inv[5];
#pragma unroll
    for (int e = 0; e < 5; ++e) {
      float l = T.ext[0][0][e], h = T.ext[0][1][e];
#pragma unroll
      for (int w = 1; w < kScoreWaves; ++w) {
        l = fminf(l, T.ext[w][0][e]);
        h = fmaxf(h, T.ext[w][1][e]);
      }
      f.mid[e] = wave_uniform(0.5f * (l + h));
      f.half[e] = wave_uniform(fmaxf(h - f.mid[e], f.mid[e] - l) * 1.00001f);
      inv[e] = wave_uniform(f.half[e] > 0.f ? 1.0f / f.half[e] : 0.f);
    }
    if (tid < cend) {
      const int c = tid;
      half8 co[3][2];
      filter_rows(T.rows[c][0], T.rows[c][1], T.rows[c][2], f, co);
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) T.coef[c / kFilterTile][t][h][c % kFilterTile] = co[t][h];
    }
    __syncthreads();  // the coefficients are written
    float inf = __builtin_inff();
    asm("" : "+v"(inf));  // (a known infinity would turn the median below back into fmaxf)
    // max(|a|, |b|) in one instruction (fmaxf adds two that quiet NaNs)
    auto larger = [&](float a, float b) { return __builtin_amdgcn_fmed3f(fabsf(a), fabsf(b), inf); };
    for (; blk < nblk; blk += wpg) {
      if (blk != wave % wpg) load(blk);
      // The products: correspondences are rows, candidates columns, so that a
      // lane holds 16 correspondences of one candidate and their minimum needs
      // no lane moves.  Lane 8 s + k of `passed`: the candidates of step s that
      // may have an inlier in slot k.
      uint32_t passed = 0;
#pragma unroll
      for (int k = 0; k < PPL; ++k) {
        const float x = (px[k] - f.mid[0]) * inv[0], y = (py[k] - f.mid[1]) * inv[1], z = (pz[k] - f.mid[2]) * inv[2];
        const float u = (pu[k] - f.mid[3]) * inv[3], v = (pv[k] - f.mid[4]) * inv[4];
        // (a minimum drops a NaN: a slot that has one passes as a whole)
        const uint32_t odd = __ballot(!(fabsf(x + y + z + u + v) < 6.f)) ? ~0u : 0u;
        // lane l of an operand holds entries 0..7 (l < 32) or 8..15 of row l % 32
        union {
          half8 h;
          unsigned w[4];
        } P, Q;
        P.h = half8{(_Float16)x, (_Float16)y, (_Float16)z, (_Float16)1.f, (_Float16)(u * x), (_Float16)(u * y),
                    (_Float16)(u * z), (_Float16)u};
        Q.h = half8{(_Float16)(v * x), (_Float16)(v * y), (_Float16)(v * z), (_Float16)v, (_Float16)1.f, (_Float16)0.f,
                    (_Float16)0.f, (_Float16)0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const auto sw = __builtin_amdgcn_permlane32_swap(P.w[e], Q.w[e], false, false);
          P.w[e] = sw[0];
          Q.w[e] = sw[1];
        }
        int at = k;
        for (int t0 = cg0; t0 < cg1; t0 += kFilterTile, at += PPL) {
          const auto& co = T.coef[t0 / kFilterTile];
          const half8 au = co[0][lane >> 5][lane & 31], av = co[1][lane >> 5][lane & 31];
          const half8 aw = co[2][lane >> 5][lane & 31];
          const float16v zero{};
          float m = 0.f;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const half8 ft = h ? Q.h : P.h;
            const float16v Du = __builtin_amdgcn_mfma_f32_32x32x16_f16(ft, au, zero, 0, 0, 0);
            const float16v Dv = __builtin_amdgcn_mfma_f32_32x32x16_f16(ft, av, zero, 0, 0, 0);
            const float16v Dw = __builtin_amdgcn_mfma_f32_32x32x16_f16(ft, aw, zero, 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
              const float s0 = larger(Du[e], Dv[e]) - Dw[e], s1 = larger(Du[e + 1], Dv[e + 1]) - Dw[e + 1];
              m = fminf(fminf(s0, s1), m);
            }
          }
          const uint64_t b = __ballot(m < 0.f);
          const uint32_t word = (uint32_t)b | (uint32_t)(b >> 32) | odd;
          passed = lane == at ? word : passed;
        }
        if (k == 0) {  // mostly good candidates: all pass
          const int some = max(0, min(kFilterTile, cg1 - cg0));
          const uint32_t first = some < kFilterTile ? (1u << some) - 1u : ~0u;
          if (4 * __popc((uint32_t)__builtin_amdgcn_readlane((int)passed, 0) & first) >= 3 * some) {
            passed = ~0u;
            break;
          }
        }
      }
      mask_ends(blk);
      load_weights(blk);
      for (int t0 = cg0, at = 0; t0 < cg1; t0 += kFilterTile, at += PPL) {
        uint32_t any = 0, full = ~0u;
#pragma unroll
        for (int k = 0; k < PPL; ++k) {
          const uint32_t word = (uint32_t)__builtin_amdgcn_readlane((int)passed, at + k);
          any |= word;
          full &= word;
        }
        const uint32_t here = cg1 - t0 < kFilterTile ? (1u << (cg1 - t0)) - 1u : ~0u;
        any &= here;
        full &= here;
        while (full & (full - 1)) {  // two left
          const int ca = __builtin_ctz(full);
          full &= full - 1;
          const int cb = __builtin_ctz(full);
          full &= full - 1;
          any &= ~((1u << ca) | (1u << cb));
          evaluate_pair(t0 + ca, t0 + cb);
        }
        for (; any; any &= any - 1) {
          const int c = __builtin_ctz(any);
          evaluate_slots(t0 + c, (uint32_t)(__ballot((passed >> c) & 1u) >> at) & 0xffu);
        }
      }
      flush();
    }
  }
  if (lane == 0) T.item[wave] = item_cnt;
  score_item_end<CT>(d, ccnt, cgain, st, c0, cend, T);
}

// Float64 scoring (every step in double).  A small round gives a CU one item,
// whose waves issue alone, so what counts is the chain of one wave: the
// projection rows are formed from the float64 poses once per item, a candidate
// per thread, where every wave formed each candidate's before its 27
// instructions per residual, and sums go to LDS only where there are inliers.
// 2,000 correspondences x 1,400 candidates: 25.3 -> 14.0 us; 100,000 x 1,000
// (the call) 192 -> 141.
template <int CT>
__device__ __forceinline__ void score_item_f64(const QueryDesc& d, const double* __restrict__ pose,
                                               uint32_t* __restrict__ ccnt, unsigned long long* __restrict__ cgain,
                                               BestState* st, int64_t tile, int64_t chunk, int ncand,
                                               ScoreTables<CT>& T) {
  constexpr int PPL = kScorePPL64;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const ChunkRange rg = chunk_range(d, chunk, 0);
  const int64_t base = rg.begin + wave * (kWave * PPL) + lane;
  const double tau2 = d.tau * d.tau;
  const int per = tile_candidates<CT>(ncand), c0 = (int)tile * per;
  const int cend = min(per, ncand - c0);
  double pu[PPL], pv[PPL], px[PPL], py[PPL], pz[PPL], pw[PPL];
#pragma unroll
  for (int k = 0; k < PPL; ++k) {
    const int64_t i = base + (int64_t)k * kWave;
    if (i < rg.end) {
      pu[k] = gmem(d.S.u)[i]; pv[k] = gmem(d.S.v)[i]; px[k] = gmem(d.S.X)[i]; py[k] = gmem(d.S.Y)[i];
      pz[k] = gmem(d.S.Z)[i];
      pw[k] = d.S.w ? gmem(d.S.w)[i] : 1.0;
    } else {
      pu[k] = __builtin_nan(""); pv[k] = 0.0; px[k] = 0.0; py[k] = 0.0; pz[k] = 0.0; pw[k] = 0.0;
    }
  }
  if (tid < cend) {  // a candidate's projection rows, once for the four waves
    const double* q = pose + 12 * (d.cand_off + c0 + tid);
    Pose Pp, Pc;
    for (int e = 0; e < 9; ++e) Pp.R[e] = q[e];
    for (int e = 0; e < 3; ++e) Pp.t[e] = q[9 + e];
    Cam K;
    camera_pose(d, rg.cam, Pp, Pc, K);
    double M[12];
    projection_rows(Pc, K, M);
#pragma unroll
    for (int e = 0; e < 12; ++e) T.rows64[tid][e] = M[e];
  }
  __syncthreads();
  uint32_t item_cnt = 0;
  for (int c = 0; c < cend; ++c) {
    const double* M = T.rows64[c];
    uint32_t cnt = 0;
    uint64_t lanes = 0;
    double gain = 0.0;
#pragma unroll
    for (int k = 0; k < PPL; ++k) {
      const double a = fma(M[2], pz[k], fma(M[1], py[k], fma(M[0], px[k], M[3])));
      const double b = fma(M[6], pz[k], fma(M[5], py[k], fma(M[4], px[k], M[7])));
      const double w = fma(M[10], pz[k], fma(M[9], py[k], fma(M[8], px[k], M[11])));
      const double du = fma(-pu[k], w, a), dv = fma(-pv[k], w, b);
      const double e = fma(dv, dv, du * du);
      const double t = (tau2 * w) * fabs(w);
      const bool in = e < t;
      const uint64_t bal = __ballot(in);
      if (bal) {
        lanes |= bal;
        cnt += (uint32_t)__popcll(bal);
        if (in) gain += pw[k] * (1.0 - e / t);
      }
    }
    if (cnt) {
      // a lone lane's gain is the sum
      uint64_t writer = lanes;
      if (lanes & (lanes - 1)) {
        gain = wave_sum(gain);
        writer = 1;
      }
      if (__builtin_amdgcn_inverse_ballot_w64(writer)) {
        atomicAdd(&T.cnt[c], cnt);
        atomicAdd(&T.gain[c], (unsigned long long)(gain * kGainScale));
      }
      item_cnt += cnt;
    }
  }
  if (lane == 0) T.item[wave] = item_cnt;
  score_item_end<CT>(d, ccnt, cgain, st, c0, cend, T);
}

// Persistent workgroups over the work list; every workgroup exits once the
// item index passes the device-side total.
template <int CT, bool FILTER>
__global__ __launch_bounds__(kScoreBlock, FILTER ? 3 : 4) void score_kernel(
    const QueryDesc* __restrict__ qd, const float* __restrict__ proj, const double* __restrict__ pose,
    const int32_t* __restrict__ ncand, uint32_t* __restrict__ ccnt, unsigned long long* __restrict__ cgain,
    BestState* __restrict__ st, int nq, int pts, const int64_t* __restrict__ item_off) {
  __shared__ ScoreTables<CT> s_tab;
  // the sums start empty, and every item leaves them empty
  for (int e = threadIdx.x; e < CT * kScoreWaves; e += kScoreBlock) (&s_tab.part[0][0])[e] = 0.f;
  if ((int)threadIdx.x < CT) {
    s_tab.cnt[threadIdx.x] = 0;
    s_tab.gain[threadIdx.x] = 0;
  }
  __syncthreads();
  const int64_t total = nq > 1     ? item_off[nq]
                        : qd[0].B > 0 ? (int64_t)((ncand[0] + CT - 1) / CT) * chunks_of(qd[0], pts)
                                      : 0;
  for (int64_t w = blockIdx.x; w < total; w += gridDim.x) {
    // the query owning item w (the last q with item_off[q] <= w): 64 probes a step
    int lo = 0;
    for (int n = nq; n > 1;) {
      const int step = (n + kWave - 1) / kWave, at = (int)(threadIdx.x & (kWave - 1)) * step;
      const int below = (int)__popcll(__ballot(at < n && item_off[lo + min(at, n - 1)] <= w)) - 1;
      lo += below * step;
      n = min(step, n - below * step);
    }
    const QueryDesc& d = qd[lo];
    const int64_t chunks = chunks_of(d, pts);
    const int64_t local = nq > 1 ? w - item_off[lo] : w;
    const int64_t tile = local / chunks, chunk = local - tile * chunks;
    const int nc = ncand[lo];
    if (d.precision == 0)
      score_item_f32<CT, FILTER>(d, proj, ccnt, cgain, st + lo, tile, chunk, nc, pts, s_tab);
    else
      score_item_f64<CT>(d, pose, ccnt, cgain, st + lo, tile, chunk, nc, s_tab);
  }
}

hipError_t launch_score(const QueryDesc* qd, CandBuf cb, BestState* st, int nq, const int64_t* item_off,
                        ScoreTune tune, int precision, hipStream_t s) {
  (void)precision;
  const dim3 grid(tune.blocks > 0 ? tune.blocks : 2048), block(kScoreBlock);
  unsigned long long* g = reinterpret_cast<unsigned long long*>(cb.gain);
  const int pts = tune.pts;
#define IMLOC_SCORE_LAUNCH(CT, FILTER)                                                                             \
  hipLaunchKernelGGL((score_kernel<CT, FILTER>), grid, block, 0, s, qd, cb.proj, cb.pose, cb.n, cb.cnt, g, st, nq, \
                     pts, item_off)
#define IMLOC_SCORE_TILE(CT)                       \
  do {                                             \
    if (tune.filter) IMLOC_SCORE_LAUNCH(CT, true); \
    else IMLOC_SCORE_LAUNCH(CT, false);            \
  } while (0)
  switch (tune.ct) {
    case 256: IMLOC_SCORE_LAUNCH(256, true); break;
    case 128: IMLOC_SCORE_TILE(128); break;
    case 64: IMLOC_SCORE_TILE(64); break;
    default: IMLOC_SCORE_TILE(32); break;
  }
#undef IMLOC_SCORE_TILE
#undef IMLOC_SCORE_LAUNCH
  return hipGetLastError();
}

// Sum of the weights of query q's scoring set (without weights: its size).
__device__ inline double weight_total(const QueryDesc& d, const CandBuf& cb, int q) {
  if (!d.full.w || d.m == 0) return (double)d.m;
  double p[kWeightParts];
#pragma unroll
  for (int u = 0; u < kWeightParts; ++u) p[u] = cb.wsum[q * kWeightParts + u];
#pragma unroll
  for (int h = kWeightParts / 2; h >= 1; h >>= 1) {
#pragma unroll
    for (int u = 0; u < h; ++u) p[u] += p[u + h];
  }
  return p[0];
}

__device__ inline double cand_msac(const QueryDesc& d, double weights, uint64_t gain) {
  return d.tau * d.tau * (weights - (double)gain * (1.0 / kGainScale));
}

__global__ void candidate_costs_kernel(const QueryDesc* __restrict__ qd, CandBuf cb, int64_t np,
                                       int32_t* __restrict__ count, double* __restrict__ msac) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= np) return;
  const int64_t o = qd[0].cand_off + i;
  count[i] = (int32_t)cb.cnt[o];
  msac[i] = cand_msac(qd[0], weight_total(qd[0], cb, 0), cb.gain[o]);
}

hipError_t launch_candidate_costs(const QueryDesc* qd, CandBuf cb, int64_t np, int32_t* count, double* msac,
                                  hipStream_t s) {
  if (np <= 0) return hipSuccess;
  hipLaunchKernelGGL(candidate_costs_kernel, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s, qd, cb, np, count,
                     msac);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Top-k of a query's batch by (msac asc, count desc, h asc, j asc) among the
// candidates whose truncated cost beats the running best.
// ---------------------------------------------------------------------------
__device__ inline Key key_none() { return Key{__builtin_inf(), 0x7fffffffffffffffll, -1, -1}; }

constexpr int kSelList = 8;      // per-thread list of the fast path (k <= 8)
constexpr int kSelUnroll = 4;    // candidates loaded together per thread
constexpr int kSelThreads = 256;
constexpr int kSelWaves = kSelThreads / kWave;
constexpr int kSelGroups = 8;    // workgroups per query, at most
constexpr int kSelPerThread = 4; // candidates per thread, about: one pass of four
constexpr int kSelWanted = 256;  // workgroups of a launch from which a query gets fewer of its own

__device__ inline Key load_key(const QueryDesc& d, double weights, const CandBuf& cb, int c) {
  const int64_t o = d.cand_off + c;
  return Key{cand_msac(d, weights, cb.gain[o]), hj_order(cb.h[o], cb.j[o]), (int)cb.cnt[o], c};
}

// Order-preserving 64-bit image of a double (total order of the non-NaN
// values): equal images <=> equal values.
__device__ inline unsigned long long ms_order(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// 64-bit unsigned minimum over the wave, received by every lane.  Partners:
// lane ^ 32 and lane ^ 16 (swap instructions), lane ^ 8 (row_ror 8), lane ^ 7
// (row_half_mirror), lane ^ 2 and lane ^ 1 (quad_perm); together they cover
// the 64 lanes.  Every lane of the wave must be active.
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_u64(unsigned long long v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, false);
  return ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
}

__device__ __forceinline__ unsigned long long umin64(unsigned long long a, unsigned long long b) {
  return a < b ? a : b;
}

__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
  {
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(v >> 32), (unsigned)(v >> 32), false, false);
    v = umin64(((unsigned long long)hi[0] << 32) | lo[0], ((unsigned long long)hi[1] << 32) | lo[1]);
  }
  {
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(v >> 32), (unsigned)(v >> 32), false, false);
    v = umin64(((unsigned long long)hi[0] << 32) | lo[0], ((unsigned long long)hi[1] << 32) | lo[1]);
  }
  v = umin64(v, dpp_u64<0x128>(v));
  v = umin64(v, dpp_u64<0x141>(v));
  v = umin64(v, dpp_u64<0x4e>(v));
  v = umin64(v, dpp_u64<0xb1>(v));
  return v;
}

// k rounds of "pop the smallest list head of the wave" over per-lane sorted
// lists; round r writes its key to out[r] (LDS, visible to the wave
// after a wave barrier).  A round takes the wave minimum of the 64-bit image
// of msac; only when several lanes hold that same msac do count and sample
// decide.  Returns the number of keys popped (< k when the lists run dry).
// Every lane of the wave must be active.
__device__ int wave_pop_k(Key (&list)[kSelList], int k, Key* out) {
  const int lane = threadIdx.x & (kWave - 1);
  int r = 0;
  for (; r < k; ++r) {
    const Key head = list[0];
    const bool valid = head.idx >= 0;
    const unsigned long long pr = valid ? ms_order(head.ms) : ~0ull;
    const unsigned long long m = wave_min_u64(pr);
    const unsigned long long tie = __ballot(valid && pr == m);
    if (tie == 0) break;  // uniform: the lists ran dry
    int wl;
    if (__popcll(tie) == 1) {
      wl = __ffsll((long long)tie) - 1;
    } else {
      // several lanes share the smallest msac (candidates without an inlier
      // all do): the most inliers, then the earliest
      const bool in = (tie >> lane) & 1ull;
      const unsigned long long mc = wave_min_u64(in ? (unsigned long long)(0x7fffffffll - head.cnt) : ~0ull);
      const bool in2 = in && (unsigned long long)(0x7fffffffll - head.cnt) == mc;
      const unsigned long long mh = wave_min_u64(in2 ? (unsigned long long)head.hj : ~0ull);
      wl = __ffsll((long long)__ballot(in2 && (unsigned long long)head.hj == mh)) - 1;
    }
    if (lane == wl) {
      out[r] = head;
#pragma unroll
      for (int e = 0; e + 1 < kSelList; ++e) list[e] = list[e + 1];
      list[kSelList - 1] = key_none();
    }
  }
  __syncwarp();
  return r;
}

__device__ __forceinline__ void key_order(Key& a, Key& b) {
  const bool swap = key_less(b, a);
  const Key s = a, t = b;  // member by member: whole selects would go through memory
  a.ms = swap ? t.ms : s.ms;
  a.hj = swap ? t.hj : s.hj;
  a.cnt = swap ? t.cnt : s.cnt;
  a.idx = swap ? t.idx : s.idx;
  b.ms = swap ? s.ms : t.ms;
  b.hj = swap ? s.hj : t.hj;
  b.cnt = swap ? s.cnt : t.cnt;
  b.idx = swap ? s.idx : t.idx;
}

// Four keys into a thread's sorted list (static register indices): sorted by
// 5 exchanges, and that is the list where it was empty; otherwise the 8
// smallest of both are a bitonic sequence, which 12 exchanges put in order.
static_assert(kSelList == 8 && kSelUnroll == 4, "the networks below");
__device__ __forceinline__ void list_merge4(Key (&list)[kSelList], Key (&x)[kSelUnroll], bool first) {
  key_order(x[0], x[1]);
  key_order(x[2], x[3]);
  key_order(x[0], x[2]);
  key_order(x[1], x[3]);
  key_order(x[1], x[2]);
  if (first) {
#pragma unroll
    for (int e = 0; e < kSelUnroll; ++e) list[e] = x[e];
    return;
  }
  if (!__any(key_less(x[0], list[kSelList - 1]))) return;
#pragma unroll
  for (int e = 0; e < kSelUnroll; ++e) key_order(list[4 + e], x[3 - e]);
#pragma unroll
  for (int st = 4; st > 0; st >>= 1)
#pragma unroll
    for (int e = 0; e < kSelList; ++e)
      if (!(e & st)) key_order(list[e], list[e + st]);
}

__host__ __device__ inline int select_groups(int64_t n_cand) {
  const int64_t g = (n_cand + kSelThreads * kSelPerThread - 1) / (kSelThreads * kSelPerThread);
  return g < 1 ? 1 : (g > kSelGroups ? kSelGroups : (int)g);
}

// The k smallest of `n` keys in LDS, to out[] in order, by one wave; returns
// how many are keys at all (at most k).  A lane counts for its key those below
// it, and that is its place: the reads do not wait for one another, where k
// pops are a chain (the launch on 1,400 candidates 6.5 -> 5.8 us).  Every place
// below the number returned is written exactly once, also if keys should tie.
__device__ int wave_rank_k(const Key* keys, int n, int k, Key* out) {
  const int lane = threadIdx.x & (kWave - 1);
  int got = 0;
  for (int e0 = 0; e0 < n; e0 += kWave) {
    const Key mine = e0 + lane < n ? keys[e0 + lane] : key_none();
    int below = 0, same = 0;
#pragma unroll 4
    for (int e = 0; e < n; ++e) {
      const double ms = keys[e].ms;
      below += ms < mine.ms ? 1 : 0;
      same += ms == mine.ms ? 1 : 0;
    }
    const bool valid = mine.idx >= 0;
    if (__ballot(valid && same > 1) && valid)  // candidates without an inlier all cost the same
      below = key_place(keys, n, e0 + lane);
    if (valid && below < k) out[below] = mine;
    got += __popcll(__ballot(valid));
  }
  __syncwarp();
  return got < k ? got : k;
}

// Top k (k <= 8) in one launch: workgroup b of a query scans candidates
// b * 256 + t + j * G * 256, every thread keeps its best kSelList in
// registers, each wave pops its k smallest, wave 0 ranks the waves' lists.  A
// workgroup alone (G == 1) has the query's top k then; of several, each writes
// its k smallest to part[q][b][0..k) (key_none() past the end) and the last to
// finish (counted in cb.sel_done) ranks the G lists.  G follows the candidates
// found, not the slots.  Bound by the chain of compares of one wave per SIMD:
// 13,374 candidates 16.1 -> 12.7 us, 1,400 candidates 7.2 -> 5.9, 256 queries
// 187 -> 30, against one-by-one insertion into lists of 8 in up to 16
// workgroups by slots and pops at every level.
__global__ __launch_bounds__(kSelThreads) void select_kernel(const QueryDesc* __restrict__ qd,
                                                             BestState* __restrict__ st, CandBuf cb,
                                                             Key* __restrict__ part, int32_t* __restrict__ sel,
                                                             int32_t* __restrict__ n_sel) {
  const int q = blockIdx.y, b = blockIdx.x;
  const QueryDesc& d = qd[q];
  if (d.B <= 0) {
    if (b == 0 && threadIdx.x == 0) n_sel[q] = 0;
    return;
  }
  const int nc = cb.n[q];
  const int G = min(select_groups(nc), (int)gridDim.x);
  if (b >= G) return;
  const int k = d.k;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const double gate = st[q].cost, weights = weight_total(d, cb, q);
  Key list[kSelList];
#pragma unroll
  for (int e = 0; e < kSelList; ++e) list[e] = key_none();
  const int stride = G * kSelThreads;
  for (int c0 = b * kSelThreads; c0 < nc; c0 += kSelUnroll * stride) {
    Key xs[kSelUnroll];
#pragma unroll
    for (int u = 0; u < kSelUnroll; ++u) {
      const int c = c0 + (int)threadIdx.x + u * stride;
      xs[u] = c < nc ? load_key(d, weights, cb, c) : key_none();
      if (!(xs[u].ms < gate)) xs[u] = key_none();
    }
    list_merge4(list, xs, c0 == b * kSelThreads);
  }
  __shared__ Key s_all[kSelGroups * kSelList];
  Key* s_wave = s_all;  // [kSelWaves * k]
  __shared__ Key s_out[kSelList];
  const int got = wave_pop_k(list, k, &s_wave[wave * k]);
  if (lane >= got && lane < k) s_wave[wave * k + lane] = key_none();
  __syncthreads();
  if (wave != 0) return;
  // wave 0: the workgroup's k smallest from the waves' lists
  const int got_b = wave_rank_k(s_wave, kSelWaves * k, k, s_out);
  if (G == 1) {
    if (lane < got_b) sel[q * kMaxTopK + lane] = s_out[lane].idx;
    if (lane == 0) {
      n_sel[q] = got_b;
      st[q].candidates += nc;
    }
    return;
  }
  Key* mine = part + ((int64_t)q * kSelGroups + b) * kSelList;
  if (lane < k) mine[lane] = lane < got_b ? s_out[lane] : key_none();
  // publish, then count this workgroup; the last one merges
  __threadfence();
  int last = 0;
  if (lane == 0) last = atomicAdd(&cb.sel_done[q], 1) == G - 1;
  if (!__builtin_amdgcn_readfirstlane(last)) return;
  __threadfence();
  const Key* all = part + (int64_t)q * kSelGroups * kSelList;
  for (int e = lane; e < G * k; e += kWave) s_all[e] = all[(e / k) * kSelList + e % k];
  __syncwarp();
  const int got_q = wave_rank_k(s_all, G * k, k, s_out);
  if (lane < got_q) sel[q * kMaxTopK + lane] = s_out[lane].idx;
  if (lane == 0) {
    n_sel[q] = got_q;
    st[q].candidates += nc;
  }
}

size_t select_scratch_bytes(int nq) {
  return (size_t)(nq > 0 ? nq : 1) * kSelGroups * kSelList * sizeof(Key);
}

// General path (k up to 32): k rounds of a workgroup argmin over all
// candidates not yet taken.
__global__ __launch_bounds__(256) void select_rounds_kernel(const QueryDesc* __restrict__ qd,
                                                            BestState* __restrict__ st, CandBuf cb,
                                                            int32_t* __restrict__ sel, int32_t* __restrict__ n_sel) {
  const int q = blockIdx.x;
  const QueryDesc& d = qd[q];
  if (d.B <= 0) {
    if (threadIdx.x == 0) n_sel[q] = 0;
    return;
  }
  const int nc = cb.n[q];
  const int k = d.k;
  const double gate = st[q].cost, weights = weight_total(d, cb, q);
  __shared__ int s_sel[kMaxTopK];
  __shared__ Key s_red[256];
  int r = 0;
  for (; r < k; ++r) {
    Key bi = key_none();
    for (int c = threadIdx.x; c < nc; c += 256) {
      const Key x = load_key(d, weights, cb, c);
      if (!(x.ms < gate)) continue;
      bool taken = false;
      for (int t = 0; t < r; ++t) taken |= (s_sel[t] == c);
      if (taken) continue;
      if (bi.idx < 0 || key_less(x, bi)) bi = x;
    }
    s_red[threadIdx.x] = bi;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
      if ((int)threadIdx.x < off) {
        const Key a = s_red[threadIdx.x], bb = s_red[threadIdx.x + off];
        if (a.idx < 0 || (bb.idx >= 0 && key_less(bb, a))) s_red[threadIdx.x] = bb;
      }
      __syncthreads();
    }
    const int win = s_red[0].idx;
    __syncthreads();
    if (win < 0) break;
    if (threadIdx.x == 0) { s_sel[r] = win; sel[q * kMaxTopK + r] = win; }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    n_sel[q] = r;
    st[q].candidates += nc;
  }
}

hipError_t launch_select(const QueryDesc* qd, const BestState* st, CandBuf cb, int nq, int kmax, int64_t max_cap,
                         void* scratch, int32_t* sel, int32_t* n_sel, hipStream_t s) {
  BestState* stw = const_cast<BestState*>(st);
  if (kmax <= kSelList) {
    Key* part = reinterpret_cast<Key*>(scratch);
    // One workgroup per query once there are enough of them: each more costs a
    // fence and the merge (256 queries: 30 us with one each, 112 with up to 8),
    // which only a query with few beside it gets back.
    const int most = std::max(1, std::min(select_groups(max_cap), kSelWanted / nq));
    hipLaunchKernelGGL(select_kernel, dim3(most, nq), dim3(kSelThreads), 0, s, qd, stw, cb, part,
                       sel, n_sel);
  } else {
    hipLaunchKernelGGL(select_rounds_kernel, dim3(nq), dim3(256), 0, s, qd, stw, cb, sel, n_sel);
  }
  return hipGetLastError();
}

}  // namespace imloc
