// gfx950 kernels of the SIFT extraction path.
//
// Every kernel serves a whole batch: work items are decoded from prefix
// tables over the images of the batch, so one image goes through exactly
// the same per-pixel and per-keypoint arithmetic whether it is extracted
// alone or with others.  No two lanes ever add floats into the same memory
// location in one instruction (histograms keep columns that lanes own); every
// sum has an order fixed in this source, which makes the output bit-identical
// from run to run.  The file is built with -ffp-contract=off: every fused
// multiply-add below is written out explicitly.
#include <hip/hip_runtime.h>
#include <math.h>

#include "sift_device.h"
#include "sift_launch.h"

namespace sift {

// ---------------------------------------------------------------------------
// Setup: image-table entries copied from kernel arguments into the workspace, and
// prefix sums over the batch of the blur work items of every (chunk class, octave)
// and of the detection bands.  A wave takes every kSetupWaves-th table, 64 images at
// a time, one lane each.  Where the arguments hold every image one launch does both
// (4.9 us for one image; as two launches, the tables by one wave, 15.6).
constexpr int kSetupWaves = 16;

// Images whose keypoints are counted (k_ori_scan).
__device__ __forceinline__ int* images_done(const HdrPtrs& hp) { return hp.queue + 1; }

// Work counter i of the launch sequence (i < min(n, kQueues)).
__device__ __forceinline__ int* work_counter(const HdrPtrs& hp, const ImgEntry* tab, int i) {
  return i == 0 ? hp.queue : &counters_of(hp.ws, tab[i])[kCntQueue];
}

__device__ __forceinline__ void prefix_tables(const HdrPtrs& hp, const ImgEntry* tab, int n,
                                              const DevParams& p) {
  const LayoutCfg lc = layout_cfg(p);
  const int lane = threadIdx.x & 63;
  const int ntile = kNumTileH * p.n_oct;   // tables 0 .. ntile - 1; the band table last
  for (int t = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); t <= ntile; t += kSetupWaves) {
    // tile prefix for class t / n_oct, octave t % n_oct
    const int cls = t / p.n_oct, k = t - cls * p.n_oct;
    int* out = t < ntile ? hp.tile_prefix + (cls * kMaxOct + k) * (n + 1) : hp.band_prefix;
    int run = 0;
    if (lane == 0) out[0] = 0;
    for (int i0 = 0; i0 < n; i0 += 64) {
      const int i = i0 + lane;
      int v = 0;
      if (i < n) {
        const int h = tab[i].h, w = tab[i].w;
        if (t < ntile) {
          int hk, wk;
          octave_dims(h, w, p.upsample, k, &hk, &wk);
          v = cdiv(wk, kTileW) * cdiv(hk, tile_h_of(cls));
        } else {
          v = region_tail(h, w, lc).total_bands;
        }
      }
      const int incl = wave_incl_scan(v);
      if (i < n) out[i + 1] = run + incl;
      run += __shfl(incl, 63, 64);
    }
  }
  // the counters of this launch sequence
  if (threadIdx.x < min(n, kQueues)) *work_counter(hp, tab, threadIdx.x) = 0;
  if (threadIdx.x == 64) *images_done(hp) = 0;
}

__global__ __launch_bounds__(64 * kSetupWaves) void k_setup(HdrPtrs hp, SetupChunk c) {
  const int t = threadIdx.x;
  if (t < c.count) const_cast<ImgEntry*>(hp.table)[c.first + t] = c.e[t];
  if (c.n > 0) prefix_tables(hp, c.e, c.n, c.p);
}

__global__ __launch_bounds__(64 * kSetupWaves) void k_finalize(HdrPtrs hp, int n, DevParams p) {
  prefix_tables(hp, hp.table, n, p);
}

// ---------------------------------------------------------------------------
// Detection.  One work-group per (image, octave, band of kBand = 8 rows).  Each wave
// walks 64-lane column segments (lanes 1..62 are outputs, lanes 0 and 63 their
// halo) down the band with a 3-row register window of the DoG layers
// D_j = L_{j+1} - L_j.  A pixel of layer i is a candidate when |D| exceeds the
// pre-gate and D is strictly above (below) the maximum (minimum) of its 26
// neighbours.  The per-row result is a 64-bit ballot word per (layer, row, segment),
// stored once per band; per-band counts feed the ordered compaction.
//
// Bound: memory for many images (64 of 768 x 1024, upsampled: 1.50 ms, 8.6 GB read,
// of which 6.5 are the levels, 5.9 TB/s with what is written), for few the latency of
// the rows' loads, kDetAhead of which are on their way: 480 x 640 takes 15.9 us, 17.9
// with one row ahead, 25 with none, and 27.8 with the rows' maxima in plain code (125
// vector instructions a row instead of 75).  Bands of two and four times the rows read
// fewer halo rows but leave fewer waves: 1.52 and 1.64 ms, and 24 and 37 us.

template <int S>
struct DetRow {
  float own[S + 2], mx3[S + 2], mn3[S + 2], lrmx[S + 2], lrmn[S + 2];
};

// Maximum and minimum of three, as one instruction each: fmaxf first makes every
// operand whose origin it cannot see canonical, an instruction each time.
__device__ __forceinline__ float max3(float a, float b, float c) {
  float d;
  __asm__("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
__device__ __forceinline__ float min3(float a, float b, float c) {
  float d;
  __asm__("v_min3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

// The levels at the rows' starts in row plus the lane's byte offset off; the rows
// then move on by step bytes.
template <int S, bool H16>
__device__ __forceinline__ void det_load_row(float (&lv)[S + 3], const char* (&row)[S + 3],
                                             int64_t step, uint32_t off, const Span& rs) {
#pragma unroll
  for (int j = 0; j < S + 3; ++j) {
    using Global = const __attribute__((address_space(1))) char*;
    const Global p = (Global)row[j] + off;
    SIFT_CHECK_IN(rs, row[j] + off, H16 ? 2 : 4);
    lv[j] = H16 ? (float)*(const __attribute__((address_space(1))) _Float16*)p
                : *(const __attribute__((address_space(1))) float*)p;
    row[j] += step;
    __asm__("" : "+s"(row[j]));   // not worked out ahead for all rows: 100 registers
  }
}

// A row's layers and the maxima and minima over left and right neighbours, without
// and with the pixel itself.  The neighbour operands are read across lanes by the
// max and min themselves; lanes 0 and 63, which have only one, are no outputs.  (A
// value just written needs two wait states before it is read across lanes.)
template <int S>
__device__ __forceinline__ void det_row(DetRow<S>& d, const float (&lv)[S + 3]) {
#pragma unroll
  for (int j = 0; j < S + 2; ++j) {
    const float v = lv[j + 1] - lv[j];
    float r;
    d.own[j] = v;
    __asm__("s_nop 1\n\t"
            "v_mov_b32_dpp %2, %5 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
            "v_max_f32_dpp %0, %5, %2 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
            "v_min_f32_dpp %1, %5, %2 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
            "v_max_f32 %3, %0, %5\n\t"
            "v_min_f32 %4, %1, %5"
            : "=&v"(d.lrmx[j]), "=&v"(d.lrmn[j]), "=&v"(r), "=&v"(d.mx3[j]), "=&v"(d.mn3[j])
            : "v"(v));
  }
}

constexpr int kDetAhead = 4;   // rows loaded ahead of the one worked on

// The rows of one band: per-layer candidate counts into cnt.  H16: the
// octave's levels are stored as fp16; W: waves of the work-group.
template <int S, bool H16, int W>
__device__ __forceinline__ void detect_band(const char* const* L, unsigned long long* masks,
                                            int hk, int wk, int pk, int nseg, int b, int r_begin,
                                            int r_end, float thr, int* cnt, const Span& rs) {
  static_assert(kBand * S <= 64, "one lane per row and layer");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t pitch = (int64_t)pk * (H16 ? 2 : 4);
  // lane r S + i keeps the words of row r_begin + r, layer i + 1
  const int word_row = lane / S, word_layer = lane - word_row * S;
  for (int sg = wave; sg < nseg; sg += W) {
    const int c = b + sg * kSeg + lane - 1;
    const uint32_t off = (uint32_t)min(c, wk - 1) * (H16 ? 2 : 4);
    const uint64_t out_cols = __ballot(lane >= 1 && lane <= kSeg && c < wk - b);
    uint32_t lo = 0, hi = 0;
    DetRow<S> w[3];
    float lv[kDetAhead][S + 3];   // rows on their way
    const char* row[S + 3];
#pragma unroll
    for (int j = 0; j < S + 3; ++j) row[j] = L[j] + (r_begin - 1) * pitch;
    // row r_begin - 1 + t; rows beyond r_end repeat it
    auto load = [&](int t) {
      det_load_row<S, H16>(lv[t % kDetAhead], row, r_begin - 1 + t < r_end ? pitch : 0, off, rs);
      __builtin_amdgcn_sched_barrier(0);   // or the loads sink to their uses
    };
#pragma unroll
    for (int t = 0; t < kDetAhead; ++t) load(t);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      det_row<S>(w[t], lv[t % kDetAhead]);
      load(t + kDetAhead);
    }
#pragma unroll
    for (int r = 0; r < kBand; ++r) {
      if (r_begin + r >= r_end) break;
      const DetRow<S>&w0 = w[r % 3], &w1 = w[(r + 1) % 3];
      DetRow<S>& w2 = w[(r + 2) % 3];
      det_row<S>(w2, lv[(r + 2) % kDetAhead]);
      if (r + 2 + kDetAhead < kBand + 2) load(r + 2 + kDetAhead);
      float max9[S + 2], min9[S + 2];
#pragma unroll
      for (int j = 0; j < S + 2; ++j) {
        max9[j] = max3(w0.mx3[j], w1.mx3[j], w2.mx3[j]);
        min9[j] = min3(w0.mn3[j], w1.mn3[j], w2.mn3[j]);
      }
#pragma unroll
      for (int i = 1; i <= S; ++i) {
        const float v = w1.own[i];
        const float max8 = max3(w0.mx3[i], w1.lrmx[i], w2.mx3[i]);
        const float min8 = min3(w0.mn3[i], w1.lrmn[i], w2.mn3[i]);
        const float nb_max = max3(max9[i - 1], max8, max9[i + 1]);
        const float nb_min = min3(min9[i - 1], min8, min9[i + 1]);
        const uint64_t m =
            out_cols & __ballot(fabsf(v) > thr) & (__ballot(v > nb_max) | __ballot(v < nb_min));
        __asm__("v_writelane_b32 %0, %1, %2" : "+v"(lo) : "s"((uint32_t)m), "n"(r * S + i - 1));
        __asm__("v_writelane_b32 %0, %1, %2"
                : "+v"(hi)
                : "s"((uint32_t)(m >> 32)), "n"(r * S + i - 1));
        cnt[i - 1] += __popcll(m);
      }
    }
    if (word_row < r_end - r_begin) {
      unsigned long long* m =
          &masks[((int64_t)word_layer * hk + r_begin + word_row) * nseg + sg];
      SIFT_CHECK_IN(rs, m, 8);
      *m = ((uint64_t)hi << 32) | lo;
    }
  }
}

// H16MODE: fp16 level storage is on (the first octave stays fp32, so each
// work-group picks its octave's path).  W: waves per work-group, which share
// the band's column segments; the counts do not depend on it.
template <int S, bool H16MODE, int W>
__global__ __launch_bounds__(W * 64) void k_detect(char* ws, HdrPtrs hp, int n, DevParams p) {
  __shared__ int s_cnt[W][S];
  const int* bp = hp.band_prefix;
  // bands dealt to the XCDs in contiguous runs (the grid is a multiple of 8):
  // a band's halo rows are its neighbours' rows, read through the same L2
  const int per_xcd = gridDim.x / kXcds;
  const int item = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  if (item >= bp[n]) return;   // a grid sized for larger images than the table's
  const int img = find_owner(bp, n, item);
  const int lb = item - bp[img];
  const ImgEntry e = hp.table[img];
  const LayoutCfg lc = layout_cfg(p);
  int k, band;
  band_owner(e.h, e.w, lc, lb, &k, &band);
  const OctView ov = octave_view(e.h, e.w, lc, k);
  const int hk = ov.h, wk = ov.w, pk = ov.pitch, nseg = ov.nseg;
  const int b = p.border;
  const int r_begin = b + band * kBand;
  const int r_end = min(r_begin + kBand, hk - b);
  const char* L[S + 3];
#pragma unroll
  for (int j = 0; j < S + 3; ++j) L[j] = reinterpret_cast<const char*>(level_ptr(ws, e, ov, j));
  unsigned long long* masks = reinterpret_cast<unsigned long long*>(ws + e.region + ov.masks);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float thr = p.pre_thr;

  int cnt[S];
#pragma unroll
  for (int i = 0; i < S; ++i) cnt[i] = 0;
  if (H16MODE && ov.es == 2)
    detect_band<S, true, W>(L, masks, hk, wk, pk, nseg, b, r_begin, r_end, thr, cnt,
                            SIFT_SPAN_VALUE(region_span(ws, e, lc)));
  else
    detect_band<S, false, W>(L, masks, hk, wk, pk, nseg, b, r_begin, r_end, thr, cnt,
                             SIFT_SPAN_VALUE(region_span(ws, e, lc)));
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < S; ++i) s_cnt[wave][i] = cnt[i];
  }
  __syncthreads();
  if (threadIdx.x < S) {
    const int i = threadIdx.x;
    int tot = 0;
#pragma unroll
    for (int wv = 0; wv < W; ++wv) tot += s_cnt[wv][i];
    int* bc = reinterpret_cast<int*>(ws + e.region + region_tail(e.h, e.w, lc).band_cnt);
    SIFT_CHECK_IN(region_span(ws, e, lc), &bc[ov.band_base * S + i * ov.nband + band], 4);
    bc[ov.band_base * S + i * ov.nband + band] = tot;
  }
}

// Exclusive scan of the band counts of one image in canonical order
// (octave, layer, band); one work-group per image.
__global__ __launch_bounds__(256) void k_band_scan(char* ws, HdrPtrs hp, int n, DevParams p) {
  __shared__ int s_wave[4];
  const ImgEntry e = hp.table[blockIdx.x];
  const RegionTail rt = region_tail(e.h, e.w, layout_cfg(p));
  const int total_bands = rt.total_bands * p.s;
  const int* bc = reinterpret_cast<const int*>(ws + e.region + rt.band_cnt);
  int* bo = reinterpret_cast<int*>(ws + e.region + rt.band_off);
  int base = 0;
  for (int c0 = 0; c0 < total_bands; c0 += 256) {
    const int idx = c0 + threadIdx.x;
    const int v = idx < total_bands ? bc[idx] : 0;
    int tot;
    const int ex = block_excl_scan256(v, s_wave, &tot);
    if (idx < total_bands) bo[idx] = base + ex;
    base += tot;
  }
  if (threadIdx.x == 0) {
    counters_of(ws, e)[kCntCand] = base;
    if (e.n_cand) *e.n_cand = base;
  }
}

// Candidate emission: one wave per (image, octave, band) writes the set bits
// of its mask words, layer by layer, row by row, segment by segment, at the
// offsets of the band scan -- the canonical (octave, layer, row, column) order.
// The first work-group sums the images' candidates for the kernels that follow (as a
// launch of its own 4.6 us).
// SCAN: no band scan has run.  A wave then sums the counts before its band itself, and
// the first work-group every image's, one after the other: worth it while bands and
// images are few (scan_in_emit), where the scan's launch takes longer than the sums.
__device__ __forceinline__ int wave_sum_i(int v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

template <bool SCAN>
__global__ __launch_bounds__(64) void k_emit(char* ws, HdrPtrs hp, int n, DevParams p) {
  if (blockIdx.x == 0) {
    int base = 0;
    if (SCAN) {
      for (int i = 0; i < n; ++i) {
        const ImgEntry e = hp.table[i];
        const RegionTail rt = region_tail(e.h, e.w, layout_cfg(p));
        const int* bc = reinterpret_cast<const int*>(ws + e.region + rt.band_cnt);
        int v = 0;
        for (int q = threadIdx.x; q < rt.total_bands * p.s; q += 64) v += bc[q];
        v = wave_sum_i(v);
        if (threadIdx.x == 0) {
          counters_of(ws, e)[kCntCand] = v;
          if (e.n_cand) *e.n_cand = v;
          hp.cand_prefix[i] = base;
        }
        base += min(v, p.max_cand);
      }
      if (threadIdx.x == 0) hp.cand_prefix[n] = base;
      return;
    }
    for (int i0 = 0; i0 < n; i0 += 64) {
      const int i = i0 + threadIdx.x;
      const int v = i < n ? min(counters_of(ws, hp.table[i])[kCntCand], p.max_cand) : 0;
      const int incl = wave_incl_scan(v);
      if (i < n) hp.cand_prefix[i] = base + incl - v;
      base += __shfl(incl, 63, 64);
    }
    if (threadIdx.x == 0) hp.cand_prefix[n] = base;
    return;
  }
  const int* bp = hp.band_prefix;
  const int item = blockIdx.x - 1;
  if (item >= bp[n]) return;
  const int img = find_owner(bp, n, item);
  const int lb = item - bp[img];
  const ImgEntry e = hp.table[img];
  const LayoutCfg lc = layout_cfg(p);
  int k, band;
  band_owner(e.h, e.w, lc, lb, &k, &band);
  const OctView ov = octave_view(e.h, e.w, lc, k);
  const RegionTail rt = region_tail(e.h, e.w, lc);
  SIFT_SPAN(rspan, region_span(ws, e, lc));
  const int hk = ov.h, nseg = ov.nseg;
  const int b = p.border;
  const int r_begin = b + band * kBand;
  const int r_end = min(r_begin + kBand, hk - b);
  const int nwords = (r_end - r_begin) * nseg;
  const unsigned long long* masks =
      reinterpret_cast<const unsigned long long*>(ws + e.region + ov.masks);
  const int* bo = reinterpret_cast<const int*>(ws + e.region + rt.band_off);
  int4* cands = reinterpret_cast<int4*>(ws + e.region + rt.cands);
  const int lane = threadIdx.x;
  const int slot = ov.band_base * p.s + band;   // of layer 1; a layer's are nband apart
  int before = 0;   // SCAN: lane i, candidates before this band's of layer i + 1
  if (SCAN) {
    int sum[kMaxScales] = {};
    const int* bc = reinterpret_cast<const int*>(ws + e.region + rt.band_cnt);
    for (int q = lane; q < slot + (p.s - 1) * ov.nband; q += 64) {
      const int v = bc[q];
#pragma unroll
      for (int i = 0; i < kMaxScales; ++i) sum[i] += q < slot + i * ov.nband ? v : 0;
    }
#pragma unroll
    for (int i = 0; i < kMaxScales; ++i)
      if (i < p.s) {
        const int all = wave_sum_i(sum[i]);
        before = lane == i ? all : before;
      }
  }
  for (int i = 1; i <= p.s; ++i) {
    int base = SCAN ? __shfl(before, i - 1, 64) : bo[slot + (i - 1) * ov.nband];
    for (int w0 = 0; w0 < nwords; w0 += 64) {
      const int wi = w0 + lane;
      unsigned long long m = 0ull;
      int r = 0, sg = 0;
      if (wi < nwords) {
        r = r_begin + wi / nseg;
        sg = wi - (wi / nseg) * nseg;
        m = masks[((int64_t)(i - 1) * hk + r) * nseg + sg];
      }
      const int pc = __popcll(m);
      const int incl = wave_incl_scan(pc);
      int idx = base + incl - pc;
      while (m) {
        const int bit = __ffsll((long long)m) - 1;
        m &= m - 1ull;
        if (idx < p.max_cand) {
          SIFT_CHECK_IN(rspan, &cands[idx], 16);
          cands[idx] = make_int4(k, i, r, b + sg * kSeg + bit - 1);
        }
        ++idx;
      }
      base += __shfl(incl, 63, 64);
    }
  }
}

// ---------------------------------------------------------------------------
// Refinement: one lane per candidate, in double precision on the fp32 DoG
// samples.  Up to refine_iters Newton steps of the 3-D quadratic fit (the
// 3x3 system solved by Cramer's rule); a step is final when all |x^| <= 0.5,
// otherwise each coordinate with |x^| > 0.5 moves by x^ rounded half away
// from zero.  Then the contrast test on |D(x^)| and the edge test on the 2x2
// spatial Hessian.

__device__ __forceinline__ double det3d(double a00, double a01, double a02, double a10, double a11,
                                        double a12, double a20, double a21, double a22) {
  return a00 * (a11 * a22 - a12 * a21) - a01 * (a10 * a22 - a12 * a20) +
         a02 * (a10 * a21 - a11 * a20);
}

__device__ __forceinline__ double round_half_away(double x) {
  return x >= 0.0 ? floor(x + 0.5) : -floor(-x + 0.5);
}

// The samples of D that the fit reads around (r, c) of layer li: all of the middle
// layer, the centre and its four neighbours of the outer two.  Every load is sent
// before the first is used.
template <bool H16>
__device__ __forceinline__ void dog_samples(double (&d)[3][3][3], char* ws, const ImgEntry& e,
                                            const OctView& ov, int li, int r, int c,
                                            const Span& rs) {
  float l[4][3][3];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const float* L = level_ptr(ws, e, ov, li - 1 + a);
#pragma unroll
    for (int dr = 0; dr < 3; ++dr)
#pragma unroll
      for (int dc = 0; dc < 3; ++dc) {
        if ((a == 0 || a == 3) && dr != 1 && dc != 1) continue;
        const int64_t off = (int64_t)(r - 1 + dr) * ov.pitch + (c - 1 + dc);
        SIFT_CHECK_IN(rs, reinterpret_cast<const char*>(L) + off * (H16 ? 2 : 4), H16 ? 2 : 4);
        l[a][dr][dc] = lv_at<H16>(L, off);
      }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int dr = 0; dr < 3; ++dr)
#pragma unroll
      for (int dc = 0; dc < 3; ++dc)
        if (a == 1 || dr == 1 || dc == 1) d[a][dr][dc] = (double)(l[a + 1][dr][dc] - l[a][dr][dc]);
}

// Candidates are dealt to the waves 8 to 64 at a time, so that about kRefineWaves
// of them (one per SIMD) have work: a load instruction's lanes read as many cache
// lines, one after the other, and waves of one CU share that path.  Bound: the
// latency of up to refine_iters rounds of loads and divisions.  480 x 640: 27 us with
// work-groups of 256 candidates and each sample's loads under a branch of their own,
// 12 now; 64 images of 768 x 1024, upsampled: 70 and 36.5; 512 or 2048 waves, or 4
// candidates at least, make no difference beyond 1 us.
// H16MODE: fp16 level storage is on; each candidate's octave picks the path.
constexpr int kRefineWaves = 1024;

template <bool H16MODE>
__global__ __launch_bounds__(64) void k_refine(char* ws, HdrPtrs hp, int n, DevParams p) {
  const int* cp = hp.cand_prefix;
  const int total = cp[n];
  const ImgEntry* tab = hp.table;
  const LayoutCfg lc = layout_cfg(p);
  const int each = min(max(cdiv(total, kRefineWaves), 8), 64);
  if ((int)threadIdx.x >= each) return;
  for (int g = blockIdx.x * each + threadIdx.x; g < total; g += gridDim.x * each) {
    const int img = find_owner(cp, n, g);
    const int j = g - cp[img];
    const ImgEntry e = tab[img];
    const RegionTail rt = region_tail(e.h, e.w, lc);
    SIFT_SPAN(rspan, region_span(ws, e, lc));
    const int4 cd = reinterpret_cast<const int4*>(ws + e.region + rt.cands)[j];
    const int k = cd.x;
    int li = cd.y, r = cd.z, c = cd.w;
    const OctView ov = octave_view(e.h, e.w, lc, k);
    const int hk = ov.h, wk = ov.w;
    const int b = p.border, s = p.s;
    RefinedKp out;
    out.ok = 0;
    out.k = k;
    out.layer = li;
    out.r = r;
    out.c = c;
    out.dx = out.dy = out.sigma_oct = out.response = out.x = out.y = out.sigma = 0.0f;
    bool converged = false;
    double xs = 0.0, xy = 0.0, xx = 0.0;
    double v = 0.0, gx = 0.0, gy = 0.0, gs = 0.0, dxx = 0.0, dyy = 0.0, dxy = 0.0;
    bool bad = false;
    for (int it = 0; it < p.refine_iters; ++it) {
      // D samples of layers li-1, li, li+1 around (r, c)
      double d[3][3][3];
      if (H16MODE && ov.es == 2)
        dog_samples<true>(d, ws, e, ov, li, r, c, SIFT_SPAN_VALUE(rspan));
      else
        dog_samples<false>(d, ws, e, ov, li, r, c, SIFT_SPAN_VALUE(rspan));
      v = d[1][1][1];
      gx = (d[1][1][2] - d[1][1][0]) * 0.5;
      gy = (d[1][2][1] - d[1][0][1]) * 0.5;
      gs = (d[2][1][1] - d[0][1][1]) * 0.5;
      dxx = d[1][1][2] + d[1][1][0] - 2.0 * v;
      dyy = d[1][2][1] + d[1][0][1] - 2.0 * v;
      const double dss = d[2][1][1] + d[0][1][1] - 2.0 * v;
      dxy = (d[1][2][2] - d[1][2][0] - d[1][0][2] + d[1][0][0]) * 0.25;
      const double dxs = (d[2][1][2] - d[2][1][0] - d[0][1][2] + d[0][1][0]) * 0.25;
      const double dys = (d[2][2][1] - d[2][0][1] - d[0][2][1] + d[0][0][1]) * 0.25;
      const double det = det3d(dxx, dxy, dxs, dxy, dyy, dys, dxs, dys, dss);
      if (det == 0.0) { bad = true; break; }
      const double bx = -gx, by = -gy, bs = -gs;
      xx = det3d(bx, dxy, dxs, by, dyy, dys, bs, dys, dss) / det;
      xy = det3d(dxx, bx, dxs, dxy, by, dys, dxs, bs, dss) / det;
      xs = det3d(dxx, dxy, bx, dxy, dyy, by, dxs, dys, bs) / det;
      if (!isfinite(xx) || !isfinite(xy) || !isfinite(xs)) { bad = true; break; }
      if (fabs(xx) <= 0.5 && fabs(xy) <= 0.5 && fabs(xs) <= 0.5) { converged = true; break; }
      // any move of more than the octave size leaves the frame
      if (fabs(xx) > 1e6 || fabs(xy) > 1e6 || fabs(xs) > 1e6) { bad = true; break; }
      if (fabs(xx) > 0.5) c += (int)round_half_away(xx);
      if (fabs(xy) > 0.5) r += (int)round_half_away(xy);
      if (fabs(xs) > 0.5) li += (int)round_half_away(xs);
      if (li < 1 || li > s || r < b || r >= hk - b || c < b || c >= wk - b) { bad = true; break; }
    }
    if (!bad && converged) {
      const double contrast = v + 0.5 * (gx * xx + gy * xy + gs * xs);
      const double tr = dxx + dyy;
      const double det2 = dxx * dyy - dxy * dxy;
      const double re = (double)p.edge_ratio;
      if (fabs(contrast) >= (double)p.contrast_thr && det2 > 0.0 &&
          tr * tr * re < (re + 1.0) * (re + 1.0) * det2) {
        const int o = p.o0 + k;
        const double sig = (double)p.sigma0 * exp2((li + xs) / s);
        const double sc = ldexp(1.0, o);
        out.ok = 1;
        out.dx = (float)xx;
        out.dy = (float)xy;
        out.sigma_oct = (float)sig;
        out.response = (float)fabs(contrast);
        out.x = (float)((c + xx) * sc);
        out.y = (float)((r + xy) * sc);
        out.sigma = (float)(sig * sc);
      }
    }
    out.layer = li;
    out.r = r;
    out.c = c;
    reinterpret_cast<RefinedKp*>(ws + e.region + rt.refined)[j] = out;
  }
}

// ---------------------------------------------------------------------------
// Orientation: one wave per refined candidate.  Samples of the square window
// are dealt to lanes in a fixed order; each lane accumulates into its own
// LDS column of the 36-bin histogram (layout [bin][lane]: no two lanes share
// an address, so each column is a sequential sum), a sample's weight split
// linearly between the two nearest bins.  Gradient orientations come from
// a polynomial arctangent (error 1.4e-7 rad), weights from the hardware
// exponential.  Bins are then summed over lanes in a fixed order, smoothed
// once with [1/4, 1/2, 1/4], and every strict local maximum >= peak_ratio *
// max gives an orientation refined by a parabola through the bin and its two
// neighbours.
//
// Bound: latency (table, candidate and level loads, then the histogram's turns), so
// as many waves as fit, 8 per SIMD with two samples a lane in flight: 32 photos of
// 1066 x 1600 take 0.265 ms, with 4 waves and four samples 0.31, with 8 and one
// sample 0.29; a division for each sample's row cost registers, not time.

// H16MODE: fp16 level storage is on; each keypoint's octave picks the path.
// Batches of at most this many images keep their candidate (orientation) and
// keypoint (descriptor) prefix tables in LDS.
constexpr int kOriLdsPrefix = 1024;
constexpr int kDescLdsPrefix = 319;
// Descriptor windows of at most this many 8 x 8 tiles form one stream, then two
// (sides up to 69 and 101 pixels).  Each further stream costs a keypoint a
// histogram cleared and summed and half an empty batch: at 49 and 81 tiles the
// 64-image 1024x768 batch took 0.52 ms, at these 0.48 ms, with a single stream for
// every window 0.49 ms; the largest windows then hold a launch of few keypoints
// (one 640x480 image: 31, 35 and 35 us).
constexpr int kDescOneStream = 81;
constexpr int kDescTwoStreams = 169;
// Work items of a wave, out of `total` for the launch.  The items are split
// evenly over up to kQueues counters; a work-group starts at the counter of its
// XCD (work-groups are dealt to the XCDs in turn) and goes on to the others when
// that one has run out.  A run of items is 1 / 4 of what would be the wave's
// share of the items left, so the waves finish together although some items
// cost several times others, and a wave asks for its next run as it starts the
// last item of the one in hand.  Atomics on one address that all XCDs use
// complete every 13 ns: a single counter and one item at a time held a launch
// of 60,000 items at 0.8 ms.  Each item's results go to slots fixed by its
// index, so they do not depend on which wave computed them.
struct WorkRuns {
  HdrPtrs hp;
  int total, nq, waves;    // items; counters; waves per counter
  int each, extra;         // items per counter; the first `extra` have one more
  int q;                   // the counter in use
  int turns = 0;           // counters found empty so far
  int next = 0, end = 0;   // the run in hand
  int run = 0, ticket = 0; // the run asked for (0: none) and the counter's answer
  int left;                // items left at the counter at the last look
  __device__ __forceinline__ WorkRuns(const HdrPtrs& h, int n, int items)
      : hp(h), total(items), nq(min(n, kQueues)) {
    waves = max((int)(gridDim.x * (blockDim.x / 64)) / nq, 1);
    q = blockIdx.x % nq;
    each = total / nq;
    extra = total - each * nq;
    left = each;
  }
  __device__ __forceinline__ void ask() {
    run = min(max(left / (4 * waves), 1), 16);
    if ((threadIdx.x & 63) == 0) ticket = atomicAdd(work_counter(hp, hp.table, q), run);
  }
  // the next item, or total when there is none
  __device__ __forceinline__ int pop() {
    while (next == end && turns < nq) {
      if (run == 0) ask();
      const int v = __builtin_amdgcn_readfirstlane(ticket);
      const int lo = q * each + min(q, extra);
      const int n = each + (q < extra ? 1 : 0);
      left = max(n - v - run, 0);
      next = lo + min(v, n);
      end = lo + min(v + run, n);
      run = 0;
      if (next == end) {
        ++turns;
        q = q + 1 == nq ? 0 : q + 1;
      }
    }
    if (next == end) return total;
    const int item = next++;
    if (next == end && turns < nq) ask();
    return item;
  }
};

template <bool H16MODE>
__global__ __launch_bounds__(256, 8) void k_orient(char* ws, HdrPtrs hp, int n, DevParams p) {
  // OC histogram columns per wave: lanes l, l + OC, ... share column l % OC
  // and add in turn (each group with instructions of its own)
  constexpr int OC = 16, OG = 64 / OC;
  __shared__ float s_hist[4][kOriBins * OC];
  __shared__ float s_bins[4][kOriBins];
  // the candidate prefix over the images, in LDS when it fits: each
  // candidate's image is then found without global-memory round trips
  __shared__ int s_cp[kOriLdsPrefix + 1];
  const int* cp = hp.cand_prefix;
  const bool cp_lds = n <= kOriLdsPrefix;
  if (cp_lds) {
    for (int i = threadIdx.x; i <= n; i += blockDim.x) s_cp[i] = cp[i];
    __syncthreads();
  }
  const int total = cp[n];
  const ImgEntry* tab = hp.table;
  const LayoutCfg lc = layout_cfg(p);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* hist = s_hist[wave];
  float* bins = s_bins[wave];
  const int nwaves = gridDim.x * 4;
  for (int g = blockIdx.x * 4 + wave; g < total; g += nwaves) {
    const int img = __builtin_amdgcn_readfirstlane(cp_lds ? find_owner(s_cp, n, g)
                                                          : find_owner(cp, n, g));
    const int j = g - __builtin_amdgcn_readfirstlane(cp_lds ? s_cp[img] : cp[img]);
    const ImgEntry e = tab[img];
    const RegionTail rt = region_tail(e.h, e.w, lc);
    const RefinedKp kp = reinterpret_cast<const RefinedKp*>(ws + e.region + rt.refined)[j];
    int* n_ori = reinterpret_cast<int*>(ws + e.region + rt.n_ori);
    float* angles = reinterpret_cast<float*>(ws + e.region + rt.angles) + (int64_t)j * kMaxPeaks;
    if (!kp.ok) {
      if (lane == 0) n_ori[j] = 0;
      continue;
    }
    if (p.upright) {
      if (lane == 0) {
        n_ori[j] = 1;
        angles[0] = 0.0f;
      }
      continue;
    }
    const OctView ov = octave_view(e.h, e.w, lc, kp.k);
    const int hk = ov.h, wk = ov.w, pk = ov.pitch;
    const float* L = level_ptr(ws, e, ov, kp.layer);
    SIFT_SPAN(rspan, region_span(ws, e, lc));
    const float sw = p.ori_sigma_factor * kp.sigma_oct;
    const int R = (int)floorf(p.ori_radius_factor * sw + 0.5f);
    const float inv2 = 1.0f / (2.0f * sw * sw);
    const int side = 2 * R + 1;
    // a lane's samples are 64 apart in the window's row order
    const int down = 64 / side, across = 64 - down * side;
    int qy = lane / side, qx = lane - qy * side;
    for (int bn = lane; bn < kOriBins * OC; bn += 64) hist[bn] = 0.0f;
    wave_lds_sync();
    // U samples per lane per pass: their loads are all issued before any is
    // used; the pass count is the same for every lane of the wave
    constexpr int U = 2;
    for (int q0 = 0; q0 < side * side; q0 += 64 * U) {
      float ga[U], gb[U], gc[U], gd[U];
      int ddx[U], ddy[U];
      bool ok[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int dy = qy - R, dx = qx - R;
        const int rr = kp.r + dy, cc = kp.c + dx;
        ok[u] = (qy < side) & (rr >= 1) & (rr <= hk - 2) & (cc >= 1) & (cc <= wk - 2);
        qx += across;
        qy += down;
        if (qx >= side) {
          qx -= side;
          ++qy;
        }
        ddx[u] = dx;
        ddy[u] = dy;
        // samples that do not contribute read the (interior) centre instead
        const int64_t at = (int64_t)(ok[u] ? rr : kp.r) * pk + (ok[u] ? cc : kp.c);
        SIFT_CHECK_IN(rspan, reinterpret_cast<const char*>(L) + (at - pk) * ov.es, ov.es);
        SIFT_CHECK_IN(rspan, reinterpret_cast<const char*>(L) + (at + pk) * ov.es, ov.es);
        if (H16MODE && ov.es == 2) {
          ga[u] = lv_at<true>(L, at + 1);
          gb[u] = lv_at<true>(L, at - 1);
          gc[u] = lv_at<true>(L, at + pk);
          gd[u] = lv_at<true>(L, at - pk);
        } else {
          const float* row = L + at;
          ga[u] = row[1];
          gb[u] = row[-1];
          gc[u] = row[pk];
          gd[u] = row[-pk];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float gx = ga[u] - gb[u];
        const float gy = gc[u] - gd[u];
        const float mag = __builtin_amdgcn_sqrtf(gx * gx + gy * gy);
        float th = atan2_poly(gy, gx);
        if (th < 0.0f) th += kTwoPi;
        const float wgt = exp_fast(-(float)(__mul24(ddx[u], ddx[u]) + __mul24(ddy[u], ddy[u])) * inv2) * mag;
        const float pos = th * ((float)kOriBins / kTwoPi);
        const float fl = floorf(pos);
        const float f = pos - fl;
        int b0 = (int)fl;
        if (b0 >= kOriBins) b0 -= kOriBins;
        int b1 = b0 + 1;
        if (b1 >= kOriBins) b1 -= kOriBins;
        const float w0 = wgt * (1.0f - f), w1 = wgt * f;
        // the two bins differ: read both, then write both
        float* c0 = &hist[b0 * OC + (lane & (OC - 1))];
        float* c1 = &hist[b1 * OC + (lane & (OC - 1))];
        SIFT_CHECK_INDEX(b0 * OC + (lane & (OC - 1)), kOriBins * OC);
        SIFT_CHECK_INDEX(b1 * OC + (lane & (OC - 1)), kOriBins * OC);
#pragma unroll
        for (int grp = 0; grp < OG; ++grp) {
          if (ok[u] && lane / OC == grp) {
            const float h0 = *c0, h1 = *c1;
            *c0 = h0 + w0;
            *c1 = h1 + w1;
          }
          // keeps the groups' updates in separate instructions, in order
          __builtin_amdgcn_wave_barrier();
        }
      }
    }
    wave_lds_sync();
    if (lane < kOriBins) {
      float acc = 0.0f;
      for (int t = 0; t < OC; ++t) acc += hist[lane * OC + ((lane + t) & (OC - 1))];
      bins[lane] = acc;
    }
    wave_lds_sync();
    float hs = -1.0f;
    if (lane < kOriBins) {
      const float l = bins[lane == 0 ? kOriBins - 1 : lane - 1];
      const float m = bins[lane];
      const float rt = bins[lane == kOriBins - 1 ? 0 : lane + 1];
      hs = (0.25f * l + 0.5f * m) + 0.25f * rt;
    }
    wave_lds_sync();
    if (lane < kOriBins) bins[lane] = hs;
    wave_lds_sync();
    const float hmax = wave_max(hs);
    bool peak = false;
    float ang = 0.0f;
    if (lane < kOriBins && hmax > 0.0f) {
      const float l = bins[lane == 0 ? kOriBins - 1 : lane - 1];
      const float rt = bins[lane == kOriBins - 1 ? 0 : lane + 1];
      peak = hs > l && hs > rt && hs >= p.ori_peak_ratio * hmax;
      if (peak) {
        const float delta = 0.5f * (l - rt) / ((l - 2.0f * hs) + rt);
        ang = ((float)lane + delta) * (360.0f / (float)kOriBins);
        if (ang < 0.0f) ang += 360.0f;
        if (ang >= 360.0f) ang -= 360.0f;
      }
    }
    const unsigned long long pm = __ballot(peak);
    if (peak) {
      const int rank = __popcll(pm & ((1ull << lane) - 1ull));
      angles[rank] = ang;
    }
    if (lane == 0) n_ori[j] = __popcll(pm);
    wave_lds_sync();
  }
}

// Exclusive scan of orientation counts in candidate order; one work-group per
// image.  Publishes n_found and count.
__global__ __launch_bounds__(256) void k_ori_scan(char* ws, HdrPtrs hp, int n, DevParams p) {
  __shared__ int s_wave[4];
  __shared__ int s_last;
  const ImgEntry e = hp.table[blockIdx.x];
  const RegionTail rt = region_tail(e.h, e.w, layout_cfg(p));
  int* cnt = counters_of(ws, e);
  const int nc = min(cnt[kCntCand], p.max_cand);
  const int* n_ori = reinterpret_cast<const int*>(ws + e.region + rt.n_ori);
  int* kp_off = reinterpret_cast<int*>(ws + e.region + rt.kp_off);
  int* kp_src = reinterpret_cast<int*>(ws + e.region + rt.kp_src);
  static_assert(kMaxPeaks <= 32, "peak index in five bits");
  int base = 0;
  for (int c0 = 0; c0 < nc; c0 += 256) {
    const int idx = c0 + threadIdx.x;
    const int v = idx < nc ? n_ori[idx] : 0;
    int tot;
    const int ex = block_excl_scan256(v, s_wave, &tot);
    if (idx < nc) kp_off[idx] = base + ex;
    // the inverse: which candidate and peak each keypoint slot describes
    for (int r = 0; r < v && base + ex + r < p.max_kp; ++r) {
      SIFT_CHECK_INDEX(base + ex + r, p.max_kp);
      kp_src[base + ex + r] = idx * 32 + r;
    }
    base += tot;
  }
  if (threadIdx.x == 0) {
    cnt[kCntKp] = base;
    if (e.n_found) *e.n_found = base;
    *e.count = min(min(base, p.max_kp), e.cap);
    if (n > 1) {
      __threadfence();
      s_last = atomicAdd(images_done(hp), 1) == n - 1;
    } else {
      hp.kp_prefix[0] = 0;
      hp.kp_prefix[1] = min(min(base, p.max_kp), e.cap);
      s_last = 0;
    }
  }
  __syncthreads();
  if (!s_last) return;
  __threadfence();
  base = 0;
  for (int c0 = 0; c0 < n; c0 += 256) {
    const int i = c0 + threadIdx.x;
    int v = 0;
    if (i < n) {
      const ImgEntry o = hp.table[i];
      const int kp = __hip_atomic_load(&counters_of(ws, o)[kCntKp], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
      v = min(min(kp, p.max_kp), o.cap);
    }
    int tot;
    const int ex = block_excl_scan256(v, s_wave, &tot);
    if (i < n) hp.kp_prefix[i] = base + ex;
    base += tot;
  }
  if (threadIdx.x == 0) hp.kp_prefix[n] = base;
}

// ---------------------------------------------------------------------------
// Descriptor.  A keypoint's window, the square that holds the rotated 4x4 grid
// of the largest pooled domain size, is cut into tiles of 8 x 8 pixels around
// the centre pixel, numbered ring by ring outwards.  64 tiles at a time, one
// lane each, are tested against the rotated square, and the tiles that touch
// it are scanned one per step, a pixel per lane: no division, one address per
// lane and four loads from it.  The pixels inside the square (about 60 %) are
// packed, with their rotated offsets and gradients, into full 64-lane batches
// by a lane permutation in registers, so the trilinear binning runs with every
// lane busy; each packed pixel is binned for every domain size whose window
// holds it.  Taking the tiles ring by ring puts pixels of about the same
// distance from the centre into one batch, which then leave the loop over the
// sizes together (0.70 of the lanes busy over ten sizes; row by row 0.59).
//
// Streams.  The tiles of a window are dealt to 1, 2 or 4 streams by the window's
// size alone; each stream packs its own pixels into an empty histogram, and the
// streams' sums are added in order.  With many keypoints one wave takes a
// keypoint's streams one after the other; with few (they would leave most of the
// chip idle, and the largest window's wave would run alone for most of the
// launch) each of the four waves of a work-group takes one stream.  The sums
// are the same either way, so an image's descriptors do not depend on the
// batch it is in.
//
// Bound: vector issue (0.85 of it for one size, 64 images of 1024x768) and LDS.
// One instruction of the LDS takes the time of 64 lanes however few are active, so
// the binning keeps all lanes active (see accumulate); with lanes that share a
// column taking turns, four times as many LDS instructions, row-by-row scan order and
// one work counter the launch took 0.84 ms, now 0.48 ms; 64 mixed images with ten
// sizes 2.50 ms, now 1.07 ms; one 97x131 tile 81 us, now 28 us.  Float
// atomics of the LDS were five times slower than reading, adding and writing
// (they take lanes one by one).
//
// Scan, packing and column order are fixed, so the sums are too.  The columns
// are summed in a fixed order, averaged over domain sizes, then L2-normalised,
// clamped, L2-normalised and optionally turned into RootSIFT (L1 normalise,
// square root).

// Tile t of the window in units of tiles from the centre tile: t = 0 is the
// centre, tiles (2r - 1)^2 .. (2r + 1)^2 - 1 run around ring r.
__device__ __forceinline__ void ring_tile(int t, int& ti, int& tj) {
  // r = floor((sqrt(t) + 1) / 2); the root of a square below 2^24 is exact
  const int r = (int)((sqrtf((float)t) + 1.0f) * 0.5f);
  const int k = t - (2 * r - 1) * (2 * r - 1);
  const int q = (k >= 2 * r) + (k >= 4 * r) + (k >= 6 * r);
  const int p = k - 2 * r * q - r;   // -r .. r - 1 along the side
  ti = q == 0 ? p : (q == 1 ? r : (q == 2 ? -p : -r));
  tj = q == 0 ? -r : (q == 1 ? p : (q == 2 ? r : -p));
  if (t == 0) ti = tj = 0;
}

// max(0, 1 - |d|)
__device__ __forceinline__ float hat(float d) {
  return __builtin_amdgcn_fmed3f(1.0f - fabsf(d), 0.0f, 1.0f);
}

constexpr int kDescWaves = 4;

// Histogram of a wave: 16 columns per bin.  Word of column w of orientation slot
// o of cell (r, c): kHistRow2 (r / 2) + kHistCol2 (c / 2) + kHistOri o +
// kHistRow (r % 2) + kHistCol (c % 2) + w.  The parities of the cell select the
// bank, so lanes at cells of different parities never meet in one.  A cell has
// nine slots: orientation 8 is 0 again, so a pixel's two slots are neighbours
// (one instruction reads or writes both).
constexpr int kHistCol = 16, kHistRow = 32, kHistOri = 64;
constexpr int kHistCol2 = 9 * kHistOri, kHistRow2 = 2 * kHistCol2;
constexpr int kHistWords = 2 * kHistRow2;

// ND: the number of domain sizes the code is unrolled for (1, or the most).
// H16MODE: fp16 level storage is on; each keypoint's octave picks the path.
// Four waves per SIMD leave 128 registers: one size takes 99, five 117, ten would take
// a few more and keep 24 bytes a lane in scratch, reloaded in the packing loop; 16
// sizes (156) run three.
template <int ND, bool H16MODE>
__global__ __launch_bounds__(64 * kDescWaves)
__attribute__((amdgpu_waves_per_eu(ND <= 10 ? 4 : 3)))
void k_describe(char* ws, HdrPtrs hp, int n, DevParams p) {
  __shared__ __align__(16) float s_hist[kDescWaves][kHistWords];
  // a stream's sums, when the waves of the work-group share a keypoint
  __shared__ float s_part[kDescWaves][kDescDim];
  // the keypoint prefix over the images, in LDS when it fits (kept small:
  // the LDS is nearly all histograms)
  __shared__ int s_kpp[kDescLdsPrefix + 1];
  const int* kpp = hp.kp_prefix;
  const bool kpp_lds = n <= kDescLdsPrefix;
  if (kpp_lds) {
    for (int i = threadIdx.x; i <= n; i += 64 * kDescWaves) s_kpp[i] = kpp[i];
    __syncthreads();
  }
  const int total = kpp[n];
  const ImgEntry* tab = hp.table;
  const LayoutCfg lc = layout_cfg(p);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* const hist = s_hist[wave];
  WorkRuns runs(hp, n, total);
  const bool shared_kp = total <= desc_share_limit(desc_largest_window(p), p.n_dsp) * (int)gridDim.x;
  int g = shared_kp ? (int)blockIdx.x : runs.pop();
  while (g < total) {
    // the next keypoint, fetched while this one runs
    const int g_next = shared_kp ? g + (int)gridDim.x : runs.pop();
    const int img = __builtin_amdgcn_readfirstlane(kpp_lds ? find_owner(s_kpp, n, g)
                                                           : find_owner(kpp, n, g));
    const int q = __builtin_amdgcn_readfirstlane(g - (kpp_lds ? s_kpp[img] : kpp[img]));
    const ImgEntry e = tab[img];
    const RegionTail rt = region_tail(e.h, e.w, lc);
    // the candidate and peak this keypoint slot describes (written by the
    // orientation scan)
    SIFT_CHECK_INDEX(q, p.max_kp);
    const int src = __builtin_amdgcn_readfirstlane(
        reinterpret_cast<const int*>(ws + e.region + rt.kp_src)[q]);
    const int j = src >> 5;
    const int pk_idx = src & 31;
    const RefinedKp kp = reinterpret_cast<const RefinedKp*>(ws + e.region + rt.refined)[j];
    const int kr = __builtin_amdgcn_readfirstlane(kp.r), kc = __builtin_amdgcn_readfirstlane(kp.c);
    const int k = __builtin_amdgcn_readfirstlane(kp.k);
    const int layer = __builtin_amdgcn_readfirstlane(kp.layer);
    const float angle =
        reinterpret_cast<const float*>(ws + e.region + rt.angles)[(int64_t)j * kMaxPeaks + pk_idx];
    const OctView ov = octave_view(e.h, e.w, lc, k);
    const int hk = ov.h, wk = ov.w;
    const int es = H16MODE ? ov.es : 4;
    SIFT_SPAN(rspan, region_span(ws, e, lc));
    // the four neighbours of a pixel: one byte offset from four uniform bases
    const gchar* gL = uniform_ptr(reinterpret_cast<const gchar*>(as_global(level_ptr(ws, e, ov, layer))));
    const uint32_t pkb = (uint32_t)ov.pitch * (uint32_t)es;
    const gchar* gr = uniform_ptr(gL + es);
    const gchar* gl = uniform_ptr(gL - es);
    const gchar* gd = uniform_ptr(gL + pkb);
    const gchar* gu = uniform_ptr(gL - pkb);
    const float th = angle * (kTwoPi / 360.0f);
    float st, ct;
    sincosf(th, &st, &ct);

    // Domain sizes: a pixel inside the window of one size is inside the
    // window of every larger one (the cell test is monotone in 1 / cell, in
    // fp32 too), so one scan of the largest window finds every contributing
    // pixel; its gradient, magnitude and orientation bin are computed once
    // and its contribution is then added for each size whose window holds it.
    // the sizes come sorted, largest first
    const float smax = p.dsp[0];
    const float wc_max = p.desc_magnif * kp.sigma_oct * smax;
    // A sample contributes only if its rotated cell coordinates fall in
    // (-1, 4), i.e. |u|, |v| < 2.5 wc (|cos| + |sin|) around the sub-pixel
    // centre; one extra ring covers the sub-pixel offset and fp32 rounding.
    const float spread = fabsf(ct) + fabsf(st);
    const int R = __builtin_amdgcn_readfirstlane((int)ceilf(2.5f * wc_max * spread) + 1);
    // tile i covers pixels 8 i - 4 .. 8 i + 3, so tiles -m .. m cover -R .. R
    const int m = (R + 4) >> 3;
    const int ntiles = (2 * m + 1) * (2 * m + 1);
    const int nstreams = ntiles <= kDescOneStream ? 1 : (ntiles <= kDescTwoStreams ? 2 : 4);
    // a tile whose centre lies this far out (in the rotated frame) holds no
    // pixel of the window (3.5 pixels to its outermost ones; rounding margin)
    const float reach = 2.5f * wc_max * 1.0001f + 3.5f * spread + 0.01f;
    // 1 / cell size of every domain size, and the factor that turns a
    // squared pixel distance into the base-2 exponent of the grid's Gaussian
    // weight exp(-(xr^2 + yr^2) / 8) for that size (unused entries 0)
    float inv_ws[ND], gk_ws[ND];
#pragma unroll
    for (int ds = 0; ds < ND; ++ds) {
      inv_ws[ds] = ds < p.n_dsp ? 1.0f / (p.desc_magnif * kp.sigma_oct * p.dsp[ds]) : 0.0f;
      gk_ws[ds] = inv_ws[ds] * inv_ws[ds] * (-0.125f * 1.44269504088896341f);
    }

    // Half the side of every window, in pixels: 2.5 cells.
    float lim_ws[ND];
#pragma unroll
    for (int ds = 0; ds < ND; ++ds)
      lim_ws[ds] = ds < p.n_dsp ? 2.5f * (p.desc_magnif * kp.sigma_oct * p.dsp[ds]) : 0.0f;
    // Trilinear binning of one contributing pixel into this lane's column, once
    // per domain size whose window holds it; every lane of the wave takes part
    // (lanes with valid == false add nothing).  A pixel reaches one even and one
    // odd grid row, one even and one odd grid column: the nearest of each,
    // with weight max(0, 1 - distance) (+0 for one it does not reach; adding
    // +0 to a non-negative sum leaves it unchanged).  In step (a, b) every lane
    // adds to one cell; the four lanes that share a column (lanes l, l + 16,
    // l + 32, l + 48) are then at cells of the four different parities, so no two
    // lanes of a step touch the same word.
    const int par_r = lane >> 5 & 1, par_c = lane >> 4 & 1;   // parities of step (0, 0)
    const float kr0 = par_r ? -0.5f : 0.5f, kc0 = par_c ? -0.5f : 0.5f;
    char* base[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
        base[a][b] = reinterpret_cast<char*>(hist) +
                     4 * (kHistRow * (par_r ^ a) + kHistCol * (par_c ^ b) + (lane & 15));
    auto accumulate = [&](float xr0, float yr0, float gx, float gy, bool valid) {
      const float r2 = xr0 * xr0 + yr0 * yr0;
      const float far = fmaxf(fabsf(xr0), fabsf(yr0));
      const float mag = __builtin_amdgcn_sqrtf(gx * gx + gy * gy);
      // orientation bin: the angle from the keypoint's, in eighths of a turn
      const float ob = __builtin_amdgcn_fractf((atan2_poly(gy, gx) - th) * (1.0f / kTwoPi)) * 8.0f;
      const float o0 = floorf(ob);
      const float fo = ob - o0, fo1 = 1.0f - fo;
      const int at_lo = (int)o0 * (4 * kHistOri), at_hi = at_lo + 4 * kHistCol2;
#pragma unroll
      for (int ds = 0; ds < ND; ++ds) {
        if (ds >= p.n_dsp) break;
        // with one size the scan's window test was this very test
        const bool add = valid && (ND == 1 || far < lim_ws[ds]);
        // sizes run largest first, and a pixel outside one size's window is
        // outside every smaller one's: once no lane adds, none will again
        if (ND > 1 && __ballot(add) == 0ull) break;
        const float wgt = mag * __builtin_amdgcn_exp2f(r2 * gk_ws[ds]);
        // signed distances, in cells, from row 1 (even rows: 0 and 2 are one
        // away from it) or 2 (odd rows), and from column 1 or 2
        const float tr[2] = {__fmaf_rn(yr0, inv_ws[ds], kr0), __fmaf_rn(yr0, inv_ws[ds], -kr0)};
        const float tc[2] = {__fmaf_rn(xr0, inv_ws[ds], kc0), __fmaf_rn(xr0, inv_ws[ds], -kc0)};
        const float wr[2] = {hat(fabsf(tr[0]) - 1.0f), hat(fabsf(tr[1]) - 1.0f)};
        const float wc[2] = {hat(fabsf(tc[0]) - 1.0f), hat(fabsf(tc[1]) - 1.0f)};
        const float wo0 = wgt * fo1, wo1 = wgt * fo;
        if (add) {
#pragma unroll
          for (int a = 0; a < 2; ++a) {
            const float ra0 = wr[a] * wo0, ra1 = wr[a] * wo1;
            const int row = tr[a] < 0.0f ? 0 : 4 * kHistRow2;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
              float* const h = reinterpret_cast<float*>(base[a][b] + (row + (tc[b] < 0.0f ? at_lo : at_hi)));
              SIFT_CHECK_INDEX(h - hist, kHistWords - kHistOri);
              const float s0 = h[0], s1 = h[kHistOri];
              h[0] = s0 + ra0 * wc[b];
              h[kHistOri] = s1 + ra1 * wc[b];
              // keeps the steps' updates in separate instructions, in order
              wave_lds_sync();
            }
          }
        }
      }
    };

    const int lx = (lane & 7) - 4, ly = (lane >> 3) - 4;   // the lane's pixel of tile (0, 0)
    // rows and columns with both neighbours are 1 .. hk - 2 and 1 .. wk - 2
    const int row1 = kr + ly - 1, col1 = kc + lx - 1;   // row - 1 and column - 1 in tile (0, 0)
    const uint32_t centre = (uint32_t)kr * pkb + (uint32_t)(kc * es);
    uint32_t at0 = centre + (uint32_t)(ly * (int)pkb + lx * es);
    // kept as one value: a tile's address is then one addition away
    __asm__("" : "+v"(at0));
    float h0 = 0.0f, h1 = 0.0f;
    for (int stream = shared_kp ? wave : 0; stream < nstreams;
         stream += shared_kp ? kDescWaves : 1) {
#pragma unroll
      for (int i = 0; i < kHistWords / 256; ++i)
        *reinterpret_cast<f32x4*>(&hist[4 * (64 * i + lane)]) = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      wave_lds_sync();
      // the stream's tiles within 64 consecutive ones
      const uint64_t mine = nstreams == 1 ? ~0ull
                            : (nstreams == 2 ? 0x5555555555555555ull : 0x1111111111111111ull)
                                  << stream;
      // Pending contributing pixels sit in lanes [0, fill): rotated offset
      // and gradient.
      int fill = 0;
      float p_x = 0.0f, p_y = 0.0f, p_gx = 0.0f, p_gy = 0.0f;
      for (int t0 = 0; t0 < ntiles; t0 += 64) {
        int ti, tj;
        ring_tile(t0 + lane, ti, tj);
        const float fu = 8.0f * (float)ti - 0.5f - kp.dx, fv = 8.0f * (float)tj - 0.5f - kp.dy;
        const bool touch = t0 + lane < ntiles &&
                           fmaxf(fabsf(ct * fu + st * fv), fabsf(ct * fv - st * fu)) < reach;
        const int tij = (tj << 16) | (ti & 0xffff);
        uint64_t todo = __ballot(touch) & mine;
        while (todo) {
          constexpr int U = 4;   // tiles whose loads are issued together
          float ga[U], gb[U], gc[U], ge[U], xr[U], yr[U];
          uint64_t inside[U];   // the tile's lanes that contribute
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const bool some = todo != 0ull;
            const int bit = some ? __builtin_ctzll(todo) : 0;
            todo &= todo - 1ull;
            const int xy = __builtin_amdgcn_readlane(tij, bit);
            const int tx = 8 * (int)(short)(xy & 0xffff), ty = 8 * (xy >> 16);
            // rotated offset from the sub-pixel centre, in pixels
            const float u0 = (float)(lx + tx) - kp.dx;
            const float v0 = (float)(ly + ty) - kp.dy;
            xr[u] = ct * u0 + st * v0;
            yr[u] = ct * v0 - st * u0;
            const bool ok = ((uint32_t)(row1 + ty) < (uint32_t)(hk - 2)) &
                            ((uint32_t)(col1 + tx) < (uint32_t)(wk - 2)) &
                            (fmaxf(fabsf(xr[u]), fabsf(yr[u])) < lim_ws[0]);
            inside[u] = some ? __ballot(ok) : 0ull;
            // samples that do not contribute read the (interior) centre instead
            const uint32_t at = ok ? at0 + (uint32_t)(ty * (int)pkb + tx * es) : centre;
            SIFT_CHECK_IN(rspan, gu + at, es);
            SIFT_CHECK_IN(rspan, gd + at, es);
            if (H16MODE && es == 2) {
              ga[u] = load_lv<true>(gr, at);
              gb[u] = load_lv<true>(gl, at);
              gc[u] = load_lv<true>(gd, at);
              ge[u] = load_lv<true>(gu, at);
            } else {
              ga[u] = load_at(gr, at);
              gb[u] = load_at(gl, at);
              gc[u] = load_at(gd, at);
              ge[u] = load_at(gu, at);
            }
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int cnt = __popcll(inside[u]);
            // contributing lanes go to [fill, fill + cnt), the others after them
            const int to = (int)__builtin_amdgcn_mbcnt_hi(
                (uint32_t)(inside[u] >> 32),
                __builtin_amdgcn_mbcnt_lo((uint32_t)inside[u], (uint32_t)fill));
            const int dest = __builtin_amdgcn_inverse_ballot_w64(inside[u])
                                 ? to : lane + (2 * fill + cnt) - to;
            const float r_x = lane_send(dest & 63, xr[u]);
            const float r_y = lane_send(dest & 63, yr[u]);
            const float r_gx = lane_send(dest & 63, ga[u] - gb[u]);
            const float r_gy = lane_send(dest & 63, gc[u] - ge[u]);
            const bool fresh = lane >= fill;
            const float n_x = fresh ? r_x : p_x, n_y = fresh ? r_y : p_y;
            const float n_gx = fresh ? r_gx : p_gx, n_gy = fresh ? r_gy : p_gy;
            fill += cnt;
            if (fill >= 64) {
              // a full batch; lanes [0, fill - 64) of what was sent overflow it
              accumulate(n_x, n_y, n_gx, n_gy, true);
              p_x = r_x;
              p_y = r_y;
              p_gx = r_gx;
              p_gy = r_gy;
              fill -= 64;
            } else {
              p_x = n_x;
              p_y = n_y;
              p_gx = n_gx;
              p_gy = n_gy;
            }
          }
        }
      }
      accumulate(p_x, p_y, p_gx, p_gy, lane < fill);
      wave_lds_sync();
      // the stream's sums: bins lane and lane + 64 (two grid rows on), the
      // columns of a bin taken from a start that differs between lanes
      auto bin_sum = [&](const float* h) {
        float v = 0.0f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(&h[4 * ((lane + t) & 3)]);
          v += (x.x + x.y) + (x.z + x.w);
        }
        return v;
      };
      const int cr = lane >> 5, cc = lane >> 3 & 3;   // the bin's cell: row 0 or 1 and column
      const float* const hb = hist + kHistRow * cr + kHistCol2 * (cc >> 1) + kHistCol * (cc & 1) +
                              kHistOri * (lane & 7);
      float a0 = bin_sum(hb), a1 = bin_sum(hb + kHistRow2);
      if ((lane & 7) == 0) {   // the slot past the last orientation is the first one
        a0 += bin_sum(hb + 8 * kHistOri);
        a1 += bin_sum(hb + kHistRow2 + 8 * kHistOri);
      }
      wave_lds_sync();
      if (shared_kp) {
        s_part[wave][lane] = a0;
        s_part[wave][lane + 64] = a1;
      } else {
        h0 = stream == 0 ? a0 : h0 + a0;
        h1 = stream == 0 ? a1 : h1 + a1;
      }
    }
    if (shared_kp) {
      __syncthreads();
      if (wave == 0) {
        h0 = s_part[0][lane];
        h1 = s_part[0][lane + 64];
        for (int s = 1; s < nstreams; ++s) {
          h0 += s_part[s][lane];
          h1 += s_part[s][lane + 64];
        }
      }
      __syncthreads();   // read before the next keypoint's sums are stored
    }
    if (!shared_kp || wave == 0) {
      const float kf = (float)p.n_dsp;
      h0 = h0 / kf;
      h1 = h1 / kf;
      float nrm = sqrtf(wave_sum(h0 * h0 + h1 * h1));
      if (nrm > 0.0f) { h0 = h0 / nrm; h1 = h1 / nrm; } else { h0 = 0.0f; h1 = 0.0f; }
      h0 = fminf(h0, p.desc_clamp);
      h1 = fminf(h1, p.desc_clamp);
      nrm = sqrtf(wave_sum(h0 * h0 + h1 * h1));
      if (nrm > 0.0f) { h0 = h0 / nrm; h1 = h1 / nrm; } else { h0 = 0.0f; h1 = 0.0f; }
      if (p.rootsift) {
        const float l1 = wave_sum(fabsf(h0) + fabsf(h1));
        if (l1 > 0.0f) { h0 = h0 / l1; h1 = h1 / l1; }
        h0 = sqrtf(h0);
        h1 = sqrtf(h1);
      }
      SIFT_CHECK_INDEX(q, e.cap);
      float* dout = e.desc + (int64_t)q * kDescDim;
      dout[lane] = h0;
      dout[lane + 64] = h1;
      if (lane == 0) {
        const int4 cd = reinterpret_cast<const int4*>(ws + e.region + rt.cands)[j];
        sift_keypoint o;
        o.x = kp.x;
        o.y = kp.y;
        o.sigma = kp.sigma;
        o.angle = angle;
        o.response = kp.response;
        o.octave = p.o0 + k;
        o.layer = layer;
        o.ix = kc;
        o.iy = kr;
        o.src_layer = cd.y;
        o.src_iy = cd.z;
        o.src_ix = cd.w;
        e.kp[q] = o;
      }
    }
    g = g_next;
  }
}

// ---------------------------------------------------------------------------
// Launch helpers

hipError_t launch_setup(const HdrPtrs& hp, const SetupChunk& c, hipStream_t stream) {
  return launch(k_setup, dim3(1), dim3(64 * kSetupWaves), stream, hp, c);
}

hipError_t launch_finalize(const HdrPtrs& hp, int n, const DevParams& p, hipStream_t stream) {
  return launch(k_finalize, dim3(1), dim3(64 * kSetupWaves), stream, hp, n, p);
}

hipError_t launch_detect(char* ws, const HdrPtrs& hp, int n, const DevParams& p, int waves,
                         int grid, hipStream_t stream) {
  grid = (grid + kXcds - 1) / kXcds * kXcds;
#define SIFT_DETECT_CASE(SS, WW)                                                          \
  if (p.s == SS && waves == WW)                                                           \
    return p.h16 ? launch(k_detect<SS, true, WW>, dim3(grid), dim3(WW * 64), stream, ws, hp, \
                          n, p)                                                           \
                 : launch(k_detect<SS, false, WW>, dim3(grid), dim3(WW * 64), stream, ws, hp, \
                          n, p);
#define SIFT_DETECT_WAVES(SS) SIFT_DETECT_CASE(SS, 4) SIFT_DETECT_CASE(SS, 8)
  SIFT_DETECT_WAVES(1) SIFT_DETECT_WAVES(2) SIFT_DETECT_WAVES(3)
  SIFT_DETECT_WAVES(4) SIFT_DETECT_WAVES(5) SIFT_DETECT_WAVES(6)
#undef SIFT_DETECT_WAVES
#undef SIFT_DETECT_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_band_scan(char* ws, const HdrPtrs& hp, int n, const DevParams& p,
                         hipStream_t stream) {
  return launch(k_band_scan, dim3(n), dim3(256), stream, ws, hp, n, p);
}

hipError_t launch_emit(char* ws, const HdrPtrs& hp, int n, const DevParams& p, int grid,
                         hipStream_t stream) {
  return scan_in_emit(grid, n)
             ? launch(k_emit<true>, dim3(grid + 1), dim3(64), stream, ws, hp, n, p)
             : launch(k_emit<false>, dim3(grid + 1), dim3(64), stream, ws, hp, n, p);
}

hipError_t launch_refine(char* ws, const HdrPtrs& hp, int n, const DevParams& p, int grid,
                         hipStream_t stream) {
  grid *= 4;   // groups of one wave
  return p.h16 ? launch(k_refine<true>, dim3(grid), dim3(64), stream, ws, hp, n, p)
               : launch(k_refine<false>, dim3(grid), dim3(64), stream, ws, hp, n, p);
}

hipError_t launch_orient(char* ws, const HdrPtrs& hp, int n, const DevParams& p, int grid,
                         hipStream_t stream) {
  grid *= 2;   // 8 waves per SIMD
  return p.h16 ? launch(k_orient<true>, dim3(grid), dim3(256), stream, ws, hp, n, p)
               : launch(k_orient<false>, dim3(grid), dim3(256), stream, ws, hp, n, p);
}

hipError_t launch_ori_scan(char* ws, const HdrPtrs& hp, int n, const DevParams& p,
                         hipStream_t stream) {
  return launch(k_ori_scan, dim3(n), dim3(256), stream, ws, hp, n, p);
}

hipError_t launch_describe(char* ws, const HdrPtrs& hp, int n, const DevParams& p, int grid,
                         hipStream_t stream) {
  // the smallest unrolled size count that covers n_dsp (5: the paper's
  // pooling set, 10: the linearly spaced set of its benchmark)
#define SIFT_DESCRIBE(NDD)                                                         \
  return p.h16 ? launch(k_describe<NDD, true>, dim3(grid), dim3(64 * kDescWaves), stream, ws, hp, n, p) \
               : launch(k_describe<NDD, false>, dim3(grid), dim3(64 * kDescWaves), stream, ws, hp, n, p)
  if (p.n_dsp == 1) SIFT_DESCRIBE(1);
  if (p.n_dsp <= 5) SIFT_DESCRIBE(5);
  if (p.n_dsp <= 10) SIFT_DESCRIBE(10);
  SIFT_DESCRIBE(kMaxDsp);
#undef SIFT_DESCRIBE
}

// The bounds-check counter of this file's kernels (see check_in).
hipError_t bounds_count_kernels(unsigned long long* count, bool reset) {
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
