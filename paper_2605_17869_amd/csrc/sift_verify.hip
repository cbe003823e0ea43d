// gfx950 kernels of geometric verification: homography hypotheses from
// minimal samples, scored by the noise-scale-marginalised inlier likelihood,
// the best one refined by reweighted least squares.  Every result is computed in
// fp64 (single precision only passes over terms that are zero beyond doubt), and
// every sum runs in an order fixed by the code (per-lane partial sums in index
// order, then a fixed butterfly and a fixed order over waves), so results are
// bit-identical from run to run.  Built with -ffp-contract=off.
#include <hip/hip_runtime.h>

#include <math.h>

#include "sift_device.h"
#include "sift_verify.h"

namespace sift {

// sqrt(2 ln 100): the 0.99 quantile of the unit Rayleigh distribution
constexpr double kTau = 3.034854258770293;
constexpr double kErfTau = 0.9975934805411772;    // erf(kTau / sqrt 2)
constexpr double kSqrtHalfPi = 1.2533141373155001;
constexpr double kSqrt2 = 1.4142135623730951;
constexpr double kPivotEps = 1e-12;

// Marginal likelihood of residual r (pixels) over sigma uniform on (0, smax]
// of a Rayleigh residual truncated at tau * sigma; 0 at and beyond tau * smax.
__device__ __forceinline__ double marginal_w(double r, double smax) {
  if (!(r < kTau * smax)) return 0.0;
  return kSqrtHalfPi / smax * (kErfTau - erf(r / (kSqrt2 * smax)));
}

__device__ __forceinline__ int verify_count(const VerifyEntry& e) {
  if (!e.n_matches) return e.cap;
  const int c = *e.n_matches;
  return c < 0 ? 0 : (c < e.cap ? c : e.cap);
}

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v = v + __shfl_xor(v, d, 64);
  return v;
}

// wave_sum_d of 16 values: lane l ends with the sum of value l / 4.  Every sum adds
// the same pairs as the butterfly (lanes 32 apart, then 16, 8, 4, 2, 1), but a
// step halves the values a lane carries on with instead of computing every sum in
// every lane: 17 exchanges instead of 96, those over 32 and 16 lanes without LDS.
__device__ __forceinline__ double swap_add(double a, double b, bool by32) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  uint32_t xs[2], ys[2];
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    const uint32_t p = (uint32_t)(x >> (32 * w)), q = (uint32_t)(y >> (32 * w));
    // the upper lanes of the first (odd rows of 16) change places with the lower of the second
    const auto r = by32 ? __builtin_amdgcn_permlane32_swap(p, q, false, false)
                        : __builtin_amdgcn_permlane16_swap(p, q, false, false);
    xs[w] = r[0];
    ys[w] = r[1];
  }
  return __builtin_bit_cast(double, ((uint64_t)xs[1] << 32) | xs[0]) +
         __builtin_bit_cast(double, ((uint64_t)ys[1] << 32) | ys[0]);
}
__device__ __forceinline__ double wave_sum16_d(const double (&v)[16]) {
  const int lane = threadIdx.x & 63;
  double a[8], b[4], c[2];
#pragma unroll
  for (int q = 0; q < 8; ++q) a[q] = swap_add(v[q], v[q + 8], true);
#pragma unroll
  for (int q = 0; q < 4; ++q) b[q] = swap_add(a[q], a[q + 4], false);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const bool up = lane & 8;
    c[q] = (up ? b[q + 2] : b[q]) + __shfl_xor(up ? b[q] : b[q + 2], 8, 64);
  }
  const bool up = lane & 4;
  double d = (up ? c[1] : c[0]) + __shfl_xor(up ? c[0] : c[1], 4, 64);
  d = d + __shfl_xor(d, 2, 64);
  return d + __shfl_xor(d, 1, 64);
}

// Homography x -> H x of a normalised-coordinate solution h (h33 = 1) moved
// back to pixels: H = Tb^-1 Hn Ta, scaled to h33 = 1.  nrm: sa, txa, tya,
// sb, txb, tyb (T = [[s, 0, tx], [0, s, ty], [0, 0, 1]]).
__device__ __forceinline__ bool denormalise(const double* h, const double* nrm, double* H) {
  const double Hn[9] = {h[0], h[1], h[2], h[3], h[4], h[5], h[6], h[7], 1.0};
  const double Ta[9] = {nrm[0], 0.0, nrm[1], 0.0, nrm[0], nrm[2], 0.0, 0.0, 1.0};
  const double ib = 1.0 / nrm[3];
  const double Tbi[9] = {ib, 0.0, -nrm[4] * ib, 0.0, ib, -nrm[5] * ib, 0.0, 0.0, 1.0};
  double M[9], R[9];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      M[3 * i + j] = (Hn[3 * i] * Ta[j] + Hn[3 * i + 1] * Ta[3 + j]) + Hn[3 * i + 2] * Ta[6 + j];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      R[3 * i + j] = (Tbi[3 * i] * M[j] + Tbi[3 * i + 1] * M[3 + j]) + Tbi[3 * i + 2] * M[6 + j];
  bool ok = true;
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    H[q] = R[q] / R[8];
    ok = ok && isfinite(H[q]);
  }
  return ok;
}

// The value lane i (the same for every lane) holds, in scalar registers.
__device__ __forceinline__ double lane_value(double v, int i) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, i);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), i);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Solve an 8 x 8 system by Gaussian elimination with partial pivoting (first
// largest pivot): lane l holds row l % 8 of the augmented 8 x 9 matrix in A.  Rows
// stay where they are; at[i] is the lane of the row at position i.  The pivot row
// goes to the other lanes through scalar registers.  Returns false (on every lane)
// when a pivot falls below kPivotEps of the largest entry of the coefficient block.
// Wave-level.
__device__ __forceinline__ bool solve8_wave(double (&A)[9], double* h) {
  const int row = threadIdx.x & 7;
  double scale = 0.0;
#pragma unroll
  for (int c = 0; c < 8; ++c) scale = fmax(scale, fabs(A[c]));
#pragma unroll
  for (int d = 4; d >= 1; d >>= 1) scale = fmax(scale, __shfl_xor(scale, d, 64));
  bool ok = scale > 0.0;
  int at[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) at[i] = i;
  bool done = false;   // this lane's row has been a pivot
#pragma unroll
  for (int col = 0; col < 8; ++col) {
    // pivot: the first of the largest |A[.][col]| among positions col .. 7
    const double av = fabs(A[col]);
    int piv = col;
    double best = lane_value(av, at[col]);
#pragma unroll
    for (int i = col + 1; i < 8; ++i) {
      const double v = lane_value(av, at[i]);
      const bool up = v > best;
      best = up ? v : best;
      piv = up ? i : piv;
    }
    piv = __builtin_amdgcn_readfirstlane(piv);
    ok = ok && !(best < kPivotEps * scale);
    const int was = at[col];
#pragma unroll
    for (int i = col + 1; i < 8; ++i)
      if (i == piv) {
        at[col] = at[i];
        at[i] = was;
      }
    double pr[9];   // the pivot row
#pragma unroll
    for (int j = col; j < 9; ++j) pr[j] = lane_value(A[j], at[col]);
    done = done || row == at[col];
    if (!done) {
      const double f = A[col] / pr[col];
#pragma unroll
      for (int j = col; j < 9; ++j) A[j] = A[j] - f * pr[j];
    }
  }
#pragma unroll
  for (int r = 7; r >= 0; --r) {
    double acc = lane_value(A[8], at[r]);
#pragma unroll
    for (int j = r + 1; j < 8; ++j) acc = acc - lane_value(A[j], at[r]) * h[j];
    h[r] = acc / lane_value(A[r], at[r]);
  }
  return ok;
}

// Rows of the DLT system of correspondence (x, y) -> (u, v), h33 = 1.
__device__ __forceinline__ void dlt_rows(double x, double y, double u, double v, double* r1,
                                         double* r2) {
  r1[0] = x; r1[1] = y; r1[2] = 1.0; r1[3] = 0.0; r1[4] = 0.0; r1[5] = 0.0;
  r1[6] = -u * x; r1[7] = -u * y; r1[8] = u;
  r2[0] = 0.0; r2[1] = 0.0; r2[2] = 0.0; r2[3] = x; r2[4] = y; r2[5] = 1.0;
  r2[6] = -v * x; r2[7] = -v * y; r2[8] = v;
}

// Weight of correspondence (ax, ay) -> (bx, by) under H: marginal_w of the
// residual r = |(x / w - bx, y / w - by)|, (x, y, w) = H (ax, ay, 1); 0 when
// w <= 0 (the point maps to or behind the line at infinity).  The cut
// r < tau * smax is first tested without divisions, on
// |(x, y) - (bx, by) w|^2 < (tau smax w)^2 relaxed by 1e-9 (far more than the
// rounding that separates the two forms); only where that admits the
// correspondence is r formed, and marginal_w's exact test and weight decide,
// so the filter changes no result.
__device__ __forceinline__ double weight_at(const double* H, double ax, double ay, double bx,
                                            double by, double smax) {
  const double x = (ax * H[0] + ay * H[1]) + H[2];
  const double y = (ax * H[3] + ay * H[4]) + H[5];
  const double w = (ax * H[6] + ay * H[7]) + H[8];
  if (!(w > 0.0)) return 0.0;
  const double ex = x - bx * w, ey = y - by * w, lim = kTau * smax * w;
  if (!(ex * ex + ey * ey < (lim * lim) * (1.0 + 1e-9))) return 0.0;
  const double dx = x / w - bx, dy = y / w - by;
  return marginal_w(sqrt(dx * dx + dy * dy), smax);
}

// Pixel positions of correspondence i (stored as the keypoints' fp32 values).
struct RawPt {
  double ax, ay, bx, by;
};
__device__ __forceinline__ RawPt raw_at(const float4* raw, int i) {
  const float4 v = raw[i];
  return RawPt{(double)v.x, (double)v.y, (double)v.z, (double)v.w};
}

// solve8_wave for one lane: the same steps in the same order on a system in
// this lane's registers (A[r][c], augmented column 8), row swaps by selects.
__device__ __forceinline__ bool solve8_lane(double (&A)[8][9], double* h) {
  double scale = 0.0;
#pragma unroll
  for (int r = 0; r < 8; ++r)
#pragma unroll
    for (int c = 0; c < 8; ++c) scale = fmax(scale, fabs(A[r][c]));
  bool ok = scale > 0.0;
#pragma unroll
  for (int col = 0; col < 8; ++col) {
    // pivot row: the first of the largest |A[r][col]|, r >= col
    int piv = col;
    double best = fabs(A[col][col]);
#pragma unroll
    for (int r = col + 1; r < 8; ++r) {
      const double v = fabs(A[r][col]);
      const bool up = v > best;
      best = up ? v : best;
      piv = up ? r : piv;
    }
    ok = ok && !(best < kPivotEps * scale);
#pragma unroll
    for (int r = col + 1; r < 8; ++r) {
      const bool sw = r == piv;
#pragma unroll
      for (int j = 0; j < 9; ++j) {
        const double t = A[col][j];
        A[col][j] = sw ? A[r][j] : t;
        A[r][j] = sw ? t : A[r][j];
      }
    }
#pragma unroll
    for (int r = col + 1; r < 8; ++r) {
      const double f = A[r][col] / A[col][col];
#pragma unroll
      for (int j = col; j < 9; ++j) A[r][j] = A[r][j] - f * A[col][j];
    }
  }
#pragma unroll
  for (int row = 7; row >= 0; --row) {
    double acc = A[row][8];
#pragma unroll
    for (int j = row + 1; j < 8; ++j) acc = acc - A[row][j] * h[j];
    h[row] = acc / A[row][row];
  }
  return ok;
}

// The model of every minimal sample, one lane per hypothesis: sample k takes
// correspondences floor(u[k][j] n) (at most n - 1), j = 0..3; repeated
// indices give no model, else the DLT rows of the four normalised
// correspondences are solved (solve8_lane) and the solution moved back to
// pixels.  Stored for the scoring and refinement kernels; NaN where a sample
// gives no model.
__global__ __launch_bounds__(kVerifyModelBlock) void k_verify_models(VerifyHdr hd, int n_pairs) {
  const int groups = (hd.n_hyp + kVerifyModelBlock - 1) / kVerifyModelBlock;
  const int p = blockIdx.x / groups;
  const int k = (blockIdx.x - p * groups) * kVerifyModelBlock + threadIdx.x;
  if (k >= hd.n_hyp) return;
  const VerifyEntry e = hd.table[p];
  const int n = verify_count(e);
  SIFT_CHECK_INDEX(k, hd.n_hyp);
  double* out = reinterpret_cast<double*>(hd.ws + e.models) + 9 * (int64_t)k;
  double H[9];
  bool ok = n >= 4;
  if (ok) {
    const double* pts = reinterpret_cast<const double*>(hd.ws + e.pts);
    const double* nrm = reinterpret_cast<const double*>(hd.ws + e.norm);
    int idx[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      SIFT_CHECK_INDEX(4 * k + j, 4 * (int64_t)hd.n_hyp);
      const double u = (double)hd.samples[4 * k + j];
      const int q = (int)floor(u * (double)n);
      idx[j] = q < n - 1 ? q : n - 1;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = i + 1; j < 4; ++j) ok = ok && idx[i] != idx[j];
    if (ok) {
      double A[8][9];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double* q = pts + 4 * (int64_t)idx[i];
        dlt_rows(q[0], q[1], q[2], q[3], A[2 * i], A[2 * i + 1]);
      }
      double h[8];
      ok = solve8_lane(A, h) && denormalise(h, nrm, H);
    }
  }
#pragma unroll
  for (int q = 0; q < 9; ++q) out[q] = ok ? H[q] : NAN;
}

__global__ void k_verify_setup(VerifyHdr hd, VerifySetupChunk c) {
  const int t = threadIdx.x;
  if (t < c.count) const_cast<VerifyEntry*>(hd.table)[c.first + t] = c.e[t];
}

// Per pair, one work-group: the matched points gathered (pixels), the normalising
// similarity of each set (mean to 0, mean distance to sqrt 2) and the normalised points.
// Sums run as 256 partial sums, partial sum v over correspondences v, v + 256, ...,
// whatever the number of threads that gather.  Where the kernel's arguments hold every
// pair (!TABLE), they bring the table entries, which it stores.  Bound: the latency
// of its dependent loads: 7 us for one pair of 211 matches, 11 for 24 of 1300; the table
// in a launch of its own and a preparation by 256 threads took 10 and 16.  More pairs
// have their table written first, 24 a launch, and are prepared together: with a launch
// of this kernel for every 24 pairs 1024 pairs of 50 matches took 313 us here, now 111.
constexpr int kPrepThreads = 1024, kPrepHeld = 4096;   // threads; points kept in LDS

template <bool TABLE>
__global__ __launch_bounds__(kPrepThreads) void k_verify_prep(VerifyHdr hd, VerifySetupChunk c) {
  __shared__ double s4[4];
  __shared__ float4 s_raw[kPrepHeld];
  __shared__ float s_max[kPrepThreads / 64];
  const VerifyEntry e = TABLE ? hd.table[blockIdx.x] : c.e[blockIdx.x];
  const int t = threadIdx.x;
  if (!TABLE && t == 0) const_cast<VerifyEntry*>(hd.table)[c.first + blockIdx.x] = e;
  const int n = verify_count(e);
  float4* raw = reinterpret_cast<float4*>(hd.ws + e.raw);
  double* pts = reinterpret_cast<double*>(hd.ws + e.pts);
  double* nrm = reinterpret_cast<double*>(hd.ws + e.norm);
  float largest = 0.0f;
  for (int i = t; i < n; i += kPrepThreads) {
    SIFT_CHECK_INDEX(i, e.cap);
    const sift_match m = e.matches[i];
    const sift_keypoint ka = e.kp_a[m.query], kb = e.kp_b[m.train];
    const float4 v = make_float4(ka.x, ka.y, kb.x, kb.y);
    raw[i] = v;
    if (i < kPrepHeld) s_raw[i] = v;
    largest = fmaxf(largest, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
  }
  largest = wave_max(largest);
  if ((t & 63) == 0) s_max[t >> 6] = largest;
  __syncthreads();
  auto point = [&](int i) {
    if (i < kPrepHeld) return raw_at(s_raw, i);
    return raw_at(raw, i);
  };
  // sums of the first four waves' partial sums, in wave order
  auto sum = [&](double v) {
    v = wave_sum_d(v);
    __syncthreads();
    if (t < 256 && (t & 63) == 0) s4[t >> 6] = v;
    __syncthreads();
    return ((s4[0] + s4[1]) + s4[2]) + s4[3];
  };
  double sx[4] = {0.0, 0.0, 0.0, 0.0};
  if (t < 256) {
    for (int i = t; i < n; i += 256) {
      SIFT_CHECK_INDEX(i, e.cap);
      const RawPt q = point(i);
      sx[0] += q.ax;
      sx[1] += q.ay;
      sx[2] += q.bx;
      sx[3] += q.by;
    }
  }
  double m[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) m[q] = sum(sx[q]) / (double)(n > 0 ? n : 1);
  double da = 0.0, db = 0.0;
  if (t < 256) {
    for (int i = t; i < n; i += 256) {
      SIFT_CHECK_INDEX(i, e.cap);
      const RawPt q = point(i);
      const double xa = q.ax - m[0], ya = q.ay - m[1], xb = q.bx - m[2], yb = q.by - m[3];
      da += sqrt(xa * xa + ya * ya);
      db += sqrt(xb * xb + yb * yb);
    }
  }
  const double ma = sum(da) / (double)(n > 0 ? n : 1);
  const double mb = sum(db) / (double)(n > 0 ? n : 1);
  const double sa = ma > 0.0 ? kSqrt2 / ma : 1.0, sb = mb > 0.0 ? kSqrt2 / mb : 1.0;
  const double T[6] = {sa, -sa * m[0], -sa * m[1], sb, -sb * m[2], -sb * m[3]};
  if (t < 6) nrm[t] = T[t];
  if (t == 6) {
    for (int w = 1; w < kPrepThreads / 64; ++w) largest = fmaxf(largest, s_max[w]);
    nrm[kNormLargest] = (double)fmaxf(largest, s_max[0]);
  }
  for (int i = t; i < n; i += kPrepThreads) {
    SIFT_CHECK_INDEX(i, e.cap);
    const RawPt q = point(i);
    double* o = pts + 4 * (int64_t)i;
    o[0] = sa * q.ax + T[1];
    o[1] = sa * q.ay + T[2];
    o[2] = sb * q.bx + T[4];
    o[3] = sb * q.by + T[5];
  }
}

// A test in single precision that every correspondence passes that weight_at's
// does (and few others).  With u = 2^-24, C the largest coordinate and X, Y, W the
// largest |x|, |y|, |w| that coordinates up to C can give under H, the computed x, y, w
// (entries of H rounded, two fused steps) are within 4 u X, 4 u Y, 4 u W, and
// ex = x - bx w within 5.1 u (X + C W).  Its test means |(ex, ey)| < L w with
// L = tau smax (1 + 5e-10), so the computed values satisfy |(ex, ey)| < L w + K,
// K = 4 u L W + 5.1 u (X + Y + 2 C W); K is taken with 8 u, the comparison of squares
// with 1e-6 to spare, and K with a floor whose square is a normal number (below those,
// roundings are no longer relative).  The conditions are written so that NaN and
// infinity pass.
struct Admit32 {
  float h[9], L, K;
  __device__ __forceinline__ Admit32(const double* H, double smax, float C) {
#pragma unroll
    for (int q = 0; q < 9; ++q) h[q] = (float)H[q];
    L = (float)(kTau * smax) * 1.000001f;
    const float X = C * (fabsf(h[0]) + fabsf(h[1])) + fabsf(h[2]);
    const float Y = C * (fabsf(h[3]) + fabsf(h[4])) + fabsf(h[5]);
    const float W = C * (fabsf(h[6]) + fabsf(h[7])) + fabsf(h[8]);
    K = 4.76837158e-7f * (L * W + ((X + Y) + 2.0f * (C * W))) + 1e-18f;
  }
  __device__ __forceinline__ bool operator()(const float4& p) const {
    const float x = __fmaf_rn(p.x, h[0], __fmaf_rn(p.y, h[1], h[2]));
    const float y = __fmaf_rn(p.x, h[3], __fmaf_rn(p.y, h[4], h[5]));
    const float w = __fmaf_rn(p.x, h[6], __fmaf_rn(p.y, h[7], h[8]));
    const float ex = __fmaf_rn(-p.z, w, x), ey = __fmaf_rn(-p.w, w, y);
    const float t = __fmaf_rn(L, w, K);
    const float d2 = __fmaf_rn(ex, ex, ey * ey), t2 = (t * t) * 1.000001f;
    return !(t <= 0.0f) & !(d2 > t2);
  }
};

// One wave per hypothesis: its score, the sum over the pair's correspondences
// of the marginal likelihood of the residual under its stored model (lane l adds
// the weights of l, l + 64, ... in that order, then a fixed butterfly).
//
// Most correspondences are far from most hypotheses.  A wave tests kHypChunk of
// them in single precision (Admit32), packs those that pass, computes their weights
// in double precision with every lane busy (the exact test among it), and each lane
// then adds its own.  Testing all in double precision and entering the weight (three
// divisions, root, error function) wherever any of 64 lanes needs it took 187 us
// for 32 pairs of 1300 matches and 1500 hypotheses, this takes 135; packing alone
// did not help, the test was the cost.  Bound: VALU work (1100 instructions a wave,
// 87 us of issue).
constexpr int kHypChunk = 1024;

__global__ __launch_bounds__(64 * kVerifyHypPerGroup) void k_verify_hyp(VerifyHdr hd, int n_pairs) {
  __shared__ double s_w[kVerifyHypPerGroup][kHypChunk];
  __shared__ uint16_t s_at[kVerifyHypPerGroup][kHypChunk];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int p = blockIdx.x / hd.hyp_groups;
  const int k = (blockIdx.x - p * hd.hyp_groups) * kVerifyHypPerGroup + wave;
  if (k >= hd.n_hyp) return;
  const VerifyEntry e = hd.table[p];
  const int n = __builtin_amdgcn_readfirstlane(verify_count(e));
  double* scores = reinterpret_cast<double*>(hd.ws + e.scores);
  SIFT_CHECK_INDEX(k, hd.n_hyp);
  const double* model = reinterpret_cast<const double*>(hd.ws + e.models) + 9 * (int64_t)k;
  double H[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) H[q] = model[q];
  if (isnan(H[0])) {
    if (lane == 0) scores[k] = -INFINITY;
    return;
  }
  const float4* raw = reinterpret_cast<const float4*>(hd.ws + e.raw);
  if (n <= 64) {
    // A weight a lane: nothing to pack.  256 pairs of 64: 170 us, packed 275 (100: 285
    // either way).
    double w = 0.0;
    if (lane < n) {
      SIFT_CHECK_INDEX(lane, e.cap);
      const RawPt q = raw_at(raw, lane);
      w = weight_at(H, q.ax, q.ay, q.bx, q.by, hd.sigma_max);
    }
    w = wave_sum_d(w);
    if (lane == 0) scores[k] = w;
    return;
  }
  const Admit32 near(H, hd.sigma_max,
                     (float)reinterpret_cast<const double*>(hd.ws + e.norm)[kNormLargest]);
  double* const w_of = s_w[wave];
  uint16_t* const at = s_at[wave];
  double acc = 0.0;
  for (int base = 0; base < n; base += kHypChunk) {
    const int m = min(n - base, kHypChunk);
    uint32_t mine = 0;   // bit j: correspondence base + 64 j + lane is near
    int count = 0;       // near ones so far (the same for every lane)
    constexpr int U = 4; // rows of 64 whose points are loaded together
    for (int j0 = 0; 64 * j0 < m; j0 += U) {
      float4 q[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = min(64 * (j0 + u) + lane, m - 1);
        SIFT_CHECK_INDEX(base + i, e.cap);
        q[u] = raw[base + i];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = 64 * (j0 + u) + lane;
        const bool in = (i < m) & near(q[u]);
        const uint64_t b = __ballot(in);
        if (in) {
          mine |= 1u << (j0 + u);
          at[count + __popcll(b & lanemask_lt())] = (uint16_t)i;
        }
        count += __popcll(b);
      }
    }
    wave_lds_sync();
    for (int c = lane; c < count; c += 64) {
      const int i = at[c];
      SIFT_CHECK_INDEX(i, m);
      const RawPt q = raw_at(raw, base + i);
      w_of[i] = weight_at(H, q.ax, q.ay, q.bx, q.by, hd.sigma_max);
    }
    wave_lds_sync();
    // the others add +0 to a sum that is not negative: left out
    while (mine) {
      const int j = __builtin_ctz(mine);
      mine &= mine - 1u;
      acc += w_of[64 * j + lane];
    }
    wave_lds_sync();
  }
  acc = wave_sum_d(acc);
  if (lane == 0) scores[k] = acc;
}

// Per pair: the best hypothesis (largest score, first among equals), then
// reweighted least squares on the normalised DLT rows, each step kept only
// if it raises the score; outputs the model, score, inlier count, weights.
//
// Sums run as 256 partial sums, partial sum v over correspondences v, v + 256,
// ..., then the butterfly of each 64, then the four in order.  The weights under a
// model are computed once, by all threads, and kept in LDS for the score,
// the next step's normal equations and the output; the 35 entries of the normal
// equations that are not zero by construction or equal to another are split over
// the two groups of 256 threads.  Bound: latency (one work-group per pair; at 211
// matches 6.9 us a step, of which 3.8 are the 8 x 8 system's chain of divisions).
// With 256 threads for everything, all 44 entries per thread and lane, weights
// computed for every use and the systems solved in LDS a pair of 211 matches took
// 48 us and 32 pairs of 1300 took 109 us; this takes 27 and 59.  1024 threads spilled
// registers (66 us); a full butterfly for each of 16 sums cost 4.5 us a step.
constexpr int kRefineThreads = 512;
constexpr int kRefineHeld = 4096;   // weights kept in LDS; longer sets go by chunks of as many
constexpr int kRefineSums = 16;     // sums per thread

// Where entry q of the normal equations' upper triangle (rows of 8, 7, .. 1
// entries, then the right side) is summed: group * kRefineSums + sum, -1: zero.
// Rows 3, 4, 5 (x, y, 1 of the second DLT row) repeat rows 0, 1, 2 among themselves.
__device__ const signed char kNormalAt[44] = {
    0, 1, 2, -1, -1, -1, 16, 17,   // (0, 0..7)
    3, 4, -1, -1, -1, 18, 19,      // (1, 1..7)
    5, -1, -1, -1, 20, 21,         // (2, 2..7)
    0, 1, 2, 24, 25,               // (3, 3..7)
    3, 4, 26, 27,                  // (4, 4..7)
    5, 28, 29,                     // (5, 5..7)
    6, 7,                          // (6, 6..7)
    22,                            // (7, 7)
    8, 9, 10, 11, 12, 13, 14, 15}; // right side

__global__ __launch_bounds__(kRefineThreads) void k_verify_refine(VerifyHdr hd, int n_pairs) {
  __shared__ double s_w[2][kRefineHeld];
  __shared__ double s4[4];
  __shared__ double s_red[4][2 * kRefineSums];   // [wave of a group][group, sum]
  __shared__ double s_h[9];
  __shared__ int s_flag, s_cnt;
  __shared__ double s_bv[kRefineThreads / 64];
  __shared__ int s_bi[kRefineThreads / 64];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int group = wave >> 2, v0 = t & 255;   // group of 256 threads; partial sum
  const VerifyEntry e = hd.table[blockIdx.x];
  const int n = verify_count(e);
  const double* scores = reinterpret_cast<const double*>(hd.ws + e.scores);
  const float4* raw = reinterpret_cast<const float4*>(hd.ws + e.raw);
  const double* pts = reinterpret_cast<const double*>(hd.ws + e.pts);
  const double* nrm = reinterpret_cast<const double*>(hd.ws + e.norm);

  // best hypothesis
  double bv = -INFINITY;
  int bi = 0x7fffffff;
  if (n >= 4) {
    for (int k = t; k < hd.n_hyp; k += kRefineThreads) {
      const double v = scores[k];
      if (v > bv || (v == bv && k < bi)) {
        bv = v;
        bi = k;
      }
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const double ov = __shfl_xor(bv, d, 64);
    const int oi = __shfl_xor(bi, d, 64);
    if (ov > bv || (ov == bv && oi < bi)) {
      bv = ov;
      bi = oi;
    }
  }
  if (lane == 0) {
    s_bv[wave] = bv;
    s_bi[wave] = bi;
  }
  if (t == 0) s_cnt = 0;
  __syncthreads();
  bv = s_bv[0];
  bi = s_bi[0];
  for (int w = 1; w < kRefineThreads / 64; ++w)
    if (s_bv[w] > bv || (s_bv[w] == bv && s_bi[w] < bi)) {
      bv = s_bv[w];
      bi = s_bi[w];
    }
  if (!(bv > -INFINITY)) {
    // no hypothesis: NaN model, zero score and inliers
    if (t < 9) e.H[t] = NAN;
    if (t == 0) {
      *e.score = 0.0;
      *e.n_inliers = 0;
      if (e.best) *e.best = -1;
    }
    if (e.weights)
      for (int i = t; i < e.cap; i += kRefineThreads) e.weights[i] = 0.0f;
    return;
  }
  // the best hypothesis' model, as stored
  double H[9];
  {
    SIFT_CHECK_INDEX(bi, hd.n_hyp);
    const double* model = reinterpret_cast<const double*>(hd.ws + e.models) + 9 * (int64_t)bi;
#pragma unroll
    for (int q = 0; q < 9; ++q) H[q] = model[q];
  }
  // weights of correspondences base .. base + kRefineHeld - 1 under G
  auto weigh = [&](const double* G, int base, double* buf) {
    for (int i = base + t; i < min(n, base + kRefineHeld); i += kRefineThreads) {
      SIFT_CHECK_INDEX(i, e.cap);
      const RawPt r = raw_at(raw, i);
      buf[i - base] = weight_at(G, r.ax, r.ay, r.bx, r.by, hd.sigma_max);
    }
  };
  const bool held = n <= kRefineHeld;
  int cur = 0;   // held: the buffer with the weights under H
  if (held) weigh(H, 0, s_w[0]);
  double Q = bv;
  for (int it = 0; it < hd.refine_iters; ++it) {
    // weighted normal equations of the DLT rows (x, y, 1, 0, 0, 0, -u x, -u y; u)
    // and (0, 0, 0, x, y, 1, -v x, -v y; v): this group's sums of a (w b)
    double ne[kRefineSums] = {};
    for (int base = 0; base < n; base += kRefineHeld) {
      if (!held) {
        __syncthreads();
        weigh(H, base, s_w[0]);
      }
      __syncthreads();
      const double* w_of = s_w[held ? cur : 0];
      for (int i = base + v0; i < min(n, base + kRefineHeld); i += 256) {
        SIFT_CHECK_INDEX(i, e.cap);
        const double w = w_of[i - base];
        const double* p = pts + 4 * (int64_t)i;
        const double x = p[0], y = p[1], u = p[2], v = p[3];
        const double ux = -u * x, uy = -u * y, vx = -v * x, vy = -v * y;
        if (group == 0) {
          const double wx = w * x, wy = w * y, wu = w * u, wv = w * v;
          ne[0] = ne[0] + x * wx;
          ne[1] = ne[1] + x * wy;
          ne[2] = ne[2] + x * w;
          ne[3] = ne[3] + y * wy;
          ne[4] = ne[4] + y * w;
          ne[5] = ne[5] + w;
          ne[6] = ne[6] + ux * (w * ux);
          ne[6] = ne[6] + vx * (w * vx);
          ne[7] = ne[7] + ux * (w * uy);
          ne[7] = ne[7] + vx * (w * vy);
          ne[8] = ne[8] + x * wu;
          ne[9] = ne[9] + y * wu;
          ne[10] = ne[10] + wu;
          ne[11] = ne[11] + x * wv;
          ne[12] = ne[12] + y * wv;
          ne[13] = ne[13] + wv;
          ne[14] = ne[14] + ux * wu;
          ne[14] = ne[14] + vx * wv;
          ne[15] = ne[15] + uy * wu;
          ne[15] = ne[15] + vy * wv;
        } else {
          const double wux = w * ux, wuy = w * uy, wvx = w * vx, wvy = w * vy;
          ne[0] = ne[0] + x * wux;
          ne[1] = ne[1] + x * wuy;
          ne[2] = ne[2] + y * wux;
          ne[3] = ne[3] + y * wuy;
          ne[4] = ne[4] + wux;
          ne[5] = ne[5] + wuy;
          ne[6] = ne[6] + uy * wuy;
          ne[6] = ne[6] + vy * wvy;
          ne[8] = ne[8] + x * wvx;
          ne[9] = ne[9] + x * wvy;
          ne[10] = ne[10] + y * wvx;
          ne[11] = ne[11] + y * wvy;
          ne[12] = ne[12] + wvx;
          ne[13] = ne[13] + wvy;
        }
      }
    }
    const double sum = wave_sum16_d(ne);
    if ((lane & 3) == 0) s_red[wave & 3][group * kRefineSums + (lane >> 2)] = sum;
    __syncthreads();
    if (wave == 0) {
      // lane l: row l % 8 of the system
      double A[9];
      const int r = lane & 7;
#pragma unroll
      for (int j = 0; j < 9; ++j) {
        const int a = min(r, j), b = max(r, j);
        const int at = kNormalAt[j == 8 ? 36 + r : 8 * a - a * (a - 1) / 2 + (b - a)];
        const int i = max(at, 0);
        const double v = ((s_red[0][i] + s_red[1][i]) + s_red[2][i]) + s_red[3][i];
        A[j] = at < 0 ? 0.0 : v;
      }
      double h[8], H2[9];
      bool ok = solve8_wave(A, h);
      if (ok) ok = denormalise(h, nrm, H2);
      if (lane == 0) {
        s_flag = ok ? 1 : 0;
        for (int q = 0; q < 9; ++q) s_h[q] = ok ? H2[q] : 0.0;
      }
    }
    __syncthreads();
    if (!s_flag) break;
    double H2[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) H2[q] = s_h[q];
    double acc = 0.0;
    double* const w_new = s_w[held ? cur ^ 1 : 0];
    for (int base = 0; base < n; base += kRefineHeld) {
      if (base > 0) __syncthreads();   // the chunk before has been added
      weigh(H2, base, w_new);
      __syncthreads();
      if (group == 0)
        for (int i = base + v0; i < min(n, base + kRefineHeld); i += 256) acc += w_new[i - base];
    }
    acc = wave_sum_d(acc);
    if (group == 0 && lane == 0) s4[wave] = acc;
    __syncthreads();
    const double Q2 = ((s4[0] + s4[1]) + s4[2]) + s4[3];
    if (!(Q2 > Q)) break;
#pragma unroll
    for (int q = 0; q < 9; ++q) H[q] = H2[q];
    Q = Q2;
    cur ^= 1;
  }
  // outputs
  __syncthreads();
  int cnt = 0;
  for (int base = 0; base < n; base += kRefineHeld) {
    if (!held) weigh(H, base, s_w[0]);   // every thread reads back its own
    for (int i = base + t; i < min(n, base + kRefineHeld); i += kRefineThreads) {
      SIFT_CHECK_INDEX(i, e.cap);
      const double w = s_w[held ? cur : 0][i - base];
      cnt += w > 0.0 ? 1 : 0;
      if (e.weights) e.weights[i] = (float)w;
    }
  }
  if (e.weights)
    for (int i = n + t; i < e.cap; i += kRefineThreads) e.weights[i] = 0.0f;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) cnt += __shfl_xor(cnt, d, 64);
  if (lane == 0) atomicAdd(&s_cnt, cnt);
  __syncthreads();
  if (t < 9) e.H[t] = H[t];
  if (t == 0) {
    *e.score = Q;
    *e.n_inliers = s_cnt;
    if (e.best) *e.best = bi;
  }
}

hipError_t launch_verify_setup(const VerifyHdr& h, const VerifySetupChunk& c, hipStream_t stream) {
  return c.prepare ? launch(k_verify_prep<false>, dim3(c.count), dim3(kPrepThreads), stream, h, c)
                   : launch(k_verify_setup, dim3(1), dim3(64), stream, h, c);
}

hipError_t launch_verify_prep(const VerifyHdr& h, int n, hipStream_t stream) {
  return launch(k_verify_prep<true>, dim3(n), dim3(kPrepThreads), stream, h, VerifySetupChunk{});
}

hipError_t launch_verify_models(const VerifyHdr& h, int n, hipStream_t stream) {
  const int groups = (h.n_hyp + kVerifyModelBlock - 1) / kVerifyModelBlock;
  return launch(k_verify_models, dim3(n * groups), dim3(kVerifyModelBlock), stream, h, n);
}

hipError_t launch_verify_hyp(const VerifyHdr& h, int n, hipStream_t stream) {
  return launch(k_verify_hyp, dim3(n * h.hyp_groups), dim3(64 * kVerifyHypPerGroup), stream, h, n);
}

hipError_t launch_verify_refine(const VerifyHdr& h, int n, hipStream_t stream) {
  return launch(k_verify_refine, dim3(n), dim3(kRefineThreads), stream, h, n);
}

// The bounds-check counter of this file's kernels (see check_index).
hipError_t bounds_count_verify(unsigned long long* count, bool reset) {
#ifdef SIFT_DEBUG_BOUNDS
  hipError_t e = hipMemcpyFromSymbol(count, HIP_SYMBOL(g_bounds_violations), sizeof *count, 0,
                                     hipMemcpyDeviceToHost);
  if (e == hipSuccess && reset) {
    const unsigned long long zero = 0;
    e = hipMemcpyToSymbol(HIP_SYMBOL(g_bounds_violations), &zero, sizeof zero, 0,
                          hipMemcpyHostToDevice);
  }
  return e;
#else
  (void)reset;
  *count = 0;
  return hipErrorNotSupported;
#endif
}

}  // namespace sift
