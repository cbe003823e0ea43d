// gfx950 kernels of descriptor matching (the symmetric ratio test).
//
// Similarities come from the matrix cores: fp16 descriptors, fp32
// accumulation, V_MFMA_F32_16X16X32_F16, with every dot product summed over
// the same fixed sequence of four 32-wide MFMA steps.  Nearest neighbours are
// kept as (value, index) pairs ordered by value, then by smaller index; the
// merge of two such summaries only compares and selects, so the result does
// not depend on the order in which partial summaries meet, and no float
// atomics are used anywhere.  Built with -ffp-contract=off.
#include <hip/hip_runtime.h>

#include <math.h>

#include <type_traits>

#include "sift_device.h"
#include "sift_match.h"

namespace sift {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int kMatchDim = 128;
constexpr int kTileStride = kMatchDim + 8;   // LDS row stride of an fp16 tile (halves)

__device__ __forceinline__ Top2 top2_empty() {
  Top2 t;
  t.v1 = -INFINITY;
  t.i1 = 0x7fffffff;
  t.v2 = -INFINITY;
  t.pad = 0;
  return t;
}

__device__ __forceinline__ bool top2_better(float va, int ia, float vb, int ib) {
  return va > vb || (va == vb && ia < ib);
}

__device__ __forceinline__ Top2 top2_merge(const Top2& a, const Top2& b) {
  Top2 r = top2_empty();
  if (top2_better(a.v1, a.i1, b.v1, b.i1)) {
    r.v1 = a.v1;
    r.i1 = a.i1;
    r.v2 = fmaxf(fmaxf(a.v2, b.v1), b.v2);
  } else {
    r.v1 = b.v1;
    r.i1 = b.i1;
    r.v2 = fmaxf(fmaxf(b.v2, a.v1), a.v2);
  }
  return r;
}

__device__ __forceinline__ Top2 top2_shfl_xor(const Top2& t, int mask) {
  Top2 o;
  o.v1 = __shfl_xor(t.v1, mask, 64);
  o.i1 = __shfl_xor(t.i1, mask, 64);
  o.v2 = __shfl_xor(t.v2, mask, 64);
  o.pad = 0;
  return o;
}

__device__ __forceinline__ int rows_in_use(const int32_t* count, int cap) {
  if (!count) return cap;
  const int c = *count;
  return c < 0 ? 0 : (c < cap ? c : cap);
}

// 8 consecutive descriptor values as fp16 (round to nearest even); rows past
// the set's end read as zeros and never reach a result.
__device__ __forceinline__ half8 load_half8(const float* row, int k, bool valid) {
  half8 h;
  if (valid) {
    const float4 p = *reinterpret_cast<const float4*>(row + k);
    const float4 q = *reinterpret_cast<const float4*>(row + k + 4);
    h[0] = (_Float16)p.x; h[1] = (_Float16)p.y; h[2] = (_Float16)p.z; h[3] = (_Float16)p.w;
    h[4] = (_Float16)q.x; h[5] = (_Float16)q.y; h[6] = (_Float16)q.z; h[7] = (_Float16)q.w;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = (_Float16)0.0f;
  }
  return h;
}

// Calls of more pairs than the kernels carry in their arguments.
__global__ void k_match_setup(MatchEntry* table, int* row_prefix, int* col_prefix,
                              MatchSetupChunk c, int n) {
  const int t = threadIdx.x;
  if (t < c.count) table[c.first + t] = c.e[t];
  if (t <= c.count && c.first + t <= n) {
    row_prefix[c.first + t] = c.row_prefix[t];
    col_prefix[c.first + t] = c.col_prefix[t];
  }
}

// Where the results of set `b_side` (0: a, 1: b) of a pair lie.
__device__ __forceinline__ Top2* best_of(const MatchHdr& h, const MatchEntry& e, int b_side) {
  return reinterpret_cast<Top2*>(h.ws + e.best) + (b_side ? e.cap_a : 0);
}
// Parts of the walks of that set's rows over the other set.
__device__ __forceinline__ int parts_of(const MatchEntry& e, int b_side) {
  return b_side ? e.parts_b : e.parts_a;
}
// v / parts for 0 <= v < 2^13, the same for every lane: v + 1/2 over at most 8 is 1 / 16 or
// more from a whole number, far more than the error of its product.
static_assert(kMatchMaxParts <= 8 && 2 * SIFT_MATCH_MAX_ROWS / kMatchTile * kMatchMaxParts <= 8192, "");
__device__ __forceinline__ int parts_quotient(int v, int parts) {
  return __builtin_amdgcn_readfirstlane(
      (int)(((float)v + 0.5f) * __builtin_amdgcn_rcpf((float)parts)));
}
__device__ __forceinline__ Top2* part_of(const MatchHdr& h, const MatchEntry& e, int b_side,
                                         int part) {
  const int64_t after_a = e.parts_a > 1 ? (int64_t)e.parts_a * e.cap_a : 0;
  return reinterpret_cast<Top2*>(h.ws + e.part) +
         (b_side ? after_a + (int64_t)part * e.cap_b : (int64_t)part * e.cap_a);
}
__device__ __forceinline__ _Float16* half_of(const MatchHdr& h, const MatchEntry& e, int b_side) {
  return reinterpret_cast<_Float16*>(h.ws + e.half) + (b_side ? (int64_t)e.cap_a * kMatchDim : 0);
}

// Entry of pair p.
__device__ __forceinline__ MatchEntry entry_of(const MatchHdr& h, int p) {
  if (h.carried) return h.e[p];
  return h.table[p];
}

// Pair of a work item and the item's number within it.  Pairs of equally many need
// no search: its dependent loads were a third of a work-group's time before its
// first product.
__device__ __forceinline__ int pair_of_item(const MatchHdr& h, int n, int item, int* local) {
  if (h.same_items) {
    const int p = item / h.same_items;
    *local = item - p * h.same_items;
    return p;
  }
  if (h.carried) {
    int p = 0;
    for (int step = kMatchOwnPairs / 2; step >= 1; step /= 2)
      if (p + step < n && h.rows[p + step] <= item) p += step;
    *local = item - h.rows[p];
    return p;
  }
  const int p = __builtin_amdgcn_readfirstlane(find_owner(h.row_prefix, n, item));
  *local = item - __builtin_amdgcn_readfirstlane(h.row_prefix[p]);
  return p;
}

// Pair of a block of kMatchMergeBlock rows of its two sets, a's and then b's, and the
// block's number within it.
__device__ __forceinline__ int pair_of_rows(const MatchHdr& h, int n, int block, int* local) {
  int p = 0;
  if (h.carried) {
    for (int step = kMatchOwnPairs / 2; step >= 1; step /= 2)
      if (p + step < n && h.cols[p + step] <= block) p += step;
    *local = block - h.cols[p];
  } else {
    p = find_owner(h.col_prefix, n, block);
    *local = block - h.col_prefix[p];
  }
  return p;
}

// The sets as fp16 (round to nearest even), kMatchMergeBlock rows a work-group.
__global__ __launch_bounds__(256) void k_match_half(MatchHdr h, int n) {
  int local;
  const int p = pair_of_rows(h, n, blockIdx.x, &local);
  const MatchEntry e = entry_of(h, p);
  const int first = local * kMatchMergeBlock;
  for (int b_side = 0; b_side < 2; ++b_side) {
    // the block's rows of this set
    const int off = b_side ? e.cap_a : 0, cap = b_side ? e.cap_b : e.cap_a;
    const int row0 = max(first - off, 0);
    if (row0 >= cap || first + kMatchMergeBlock <= off) continue;
    const int end = min(first + kMatchMergeBlock - off, rows_in_use(b_side ? e.count_b : e.count_a, cap));
    const float* src = b_side ? e.desc_b : e.desc_a;
    _Float16* dst = half_of(h, e, b_side);
#pragma unroll
    for (int i = 0; i < kMatchMergeBlock * (kMatchDim / 8) / 256; ++i) {
      const int piece = i * 256 + threadIdx.x;
      const int row = row0 + piece / (kMatchDim / 8), k = piece % (kMatchDim / 8) * 8;
      if (row < end) {
        SIFT_CHECK_INDEX(row, cap);
        *reinterpret_cast<half8*>(dst + (int64_t)row * kMatchDim + k) =
            load_half8(src + (int64_t)row * kMatchDim, k, true);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Nearest neighbours.  One work-group (4 waves) per (pair, set, tile of 32 OB
// rows of that set, its own rows, part of the other set); it walks the part's
// tiles of 128 rows.  Waves 2 h and 2 h + 1 hold half h of the own rows as
// MFMA B operands in registers for the whole walk and take the two halves of
// each tile, which is staged in LDS as fp16 (two buffers: the next tile is on
// its way while the current one is computed).  Lane l supplies other row
// 16 ta + l % 16 and own row 16 tb + l % 16, 8 values each at k = 32 kk + 8
// (l / 16), and receives s for other rows 16 ta + 4 (l / 16) + r, own row
// 16 tb + l % 16: every value a lane receives belongs to one of OB own rows,
// whose nearest and second nearest it keeps.  Both directions are walked this
// way: the products are computed twice, on matrix cores that would idle
// otherwise, and no summary leaves the lane before the end of the walk.
//
// Bound: matrix products and vector issue in turn (four operations per
// similarity: comparison, second largest as a median, two selects), with what is
// read from LDS on top; of 83 us for 32 pairs of 2000 x 2000 the products take 30,
// the comparisons 18.  Keeping both directions' summaries from one product took 20
// states per lane, merges between lanes per tile, and tiles converted between
// two barriers: 236 us, and 398 us for one pair of 8192 x 7900 (now 50), whose 64
// row tiles left three quarters of the chip idle.
// HALF: the sets have been copied to fp16.  OB: blocks of 16 own rows per wave.
// Eight read half of LDS and memory per product that four do (83 against 96
// us), four make twice the work-groups of a small call.
template <bool HALF, int OB>
__global__ __launch_bounds__(256, 2) void k_match_best(MatchHdr h, int n, int items) {
  // HALF: a tile is copied to LDS by the load unit, rows unpadded, the 16-byte
  // pieces of row r at places p ^ (r % 16) (the 16 rows a wave reads together
  // then lie in different banks)
  constexpr int kStride = HALF ? kMatchDim : kTileStride;
  __shared__ __align__(256) _Float16 s_t0[kMatchTile * kStride], s_t1[kMatchTile * kStride];
  constexpr int kOwn = 32 * OB;   // own rows of the work-group
  __shared__ Top2 s_part[2][kOwn];
  // neighbouring items (one pair's tiles) to one XCD, whose L2 then holds the pair
  const int per_xcd = gridDim.x / kXcds;
  const int item = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  if (item >= items) return;
  int local;
  const int p = pair_of_item(h, n, item, &local);
  const MatchEntry e = entry_of(h, p);
  const int a_items = (e.cap_a + kOwn - 1) / kOwn * e.parts_a;
  const int b_side = local >= a_items;   // own rows are b's
  const int parts = parts_of(e, b_side);
  if (b_side) local -= a_items;
  // a tile's parts follow each other
  const int tile = parts_quotient(local, parts), part = local - tile * parts;
  const int row0 = tile * kOwn;
  const int na = __builtin_amdgcn_readfirstlane(rows_in_use(e.count_a, e.cap_a));
  const int nb = __builtin_amdgcn_readfirstlane(rows_in_use(e.count_b, e.cap_b));
  const int n_own = b_side ? nb : na, n_oth = b_side ? na : nb;
  if (row0 >= n_own) return;
  const int cap_own = b_side ? e.cap_b : e.cap_a, cap_oth = b_side ? e.cap_a : e.cap_b;
  const float* f_own = b_side ? e.desc_b : e.desc_a;
  const float* f_oth = b_side ? e.desc_a : e.desc_b;
  const _Float16* h_own = HALF ? half_of(h, e, b_side) : nullptr;
  const _Float16* h_oth = HALF ? half_of(h, e, !b_side) : nullptr;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int li = lane & 15, gq = lane >> 4;
  const int own_half = wv >> 1, oth_half = wv & 1;
  // 8 values of a row as fp16
  auto piece_of = [&](const _Float16* hs, const float* fs, int64_t at) {
    if (HALF) return *reinterpret_cast<const half8*>(hs + at);
    return load_half8(fs + at, 0, true);
  };
  // own fragments: row row0 + 16 OB own_half + 16 tb + li, k = 32 kk + 8 gq (rows past
  // the set's end repeat the last one; nothing of theirs is stored)
  half8 fb[OB][4];
#pragma unroll
  for (int tb = 0; tb < OB; ++tb) {
    const int i = min(row0 + 16 * OB * own_half + 16 * tb + li, n_own - 1);
    SIFT_CHECK_INDEX(i, cap_own);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      fb[tb][kk] = piece_of(h_own, f_own, (int64_t)i * kMatchDim + 32 * kk + 8 * gq);
  }
  float v1[OB], v2[OB];
  int i1[OB];
#pragma unroll
  for (int tb = 0; tb < OB; ++tb) {
    v1[tb] = v2[tb] = -INFINITY;
    i1[tb] = 0x7fffffff;
  }
  // pieces of 8 values of a tile: 8 per thread, piece i of thread t in row
  // 16 i + t / 16 (rows past the set's end repeat the last one: the walk leaves
  // them out)
  constexpr int kPieces = kMatchTile * kMatchDim / 8 / 256, kPieceRows = kMatchTile / kPieces;
  static_assert(kPieceRows * (kMatchDim / 8) == 256, "a piece of every thread is whole rows");
  const int prow = t / (kMatchDim / 8), pk = t % (kMatchDim / 8) * 8;
  auto stage = [&](int ct, _Float16* buf) {
    const int r0 = ct * kMatchTile;
    if constexpr (HALF) {
#pragma unroll
      for (int i = 0; i < kPieces; ++i) {
        const int row = min(r0 + kPieceRows * i + prow, n_oth - 1);
        SIFT_CHECK_INDEX(row, cap_oth);
        const _Float16* from = h_oth + (int64_t)row * kMatchDim + (pk ^ (prow * 8));
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void*)from,
            (__attribute__((address_space(3))) void*)(buf + (256 * i + 64 * wv) * 8), 16, 0, 0);
      }
    } else {
      half8 st[kPieces];
#pragma unroll
      for (int i = 0; i < kPieces; ++i) {
        const int row = min(r0 + kPieceRows * i + prow, n_oth - 1);
        SIFT_CHECK_INDEX(row, cap_oth);
        st[i] = load_half8(f_oth + (int64_t)row * kMatchDim, pk, true);
      }
#pragma unroll
      for (int i = 0; i < kPieces; ++i)
        *reinterpret_cast<half8*>(&buf[(kPieceRows * i + prow) * kStride + pk]) = st[i];
    }
  };
  // the part's tiles of the other set, from the rows in use
  const int used = (n_oth + kMatchTile - 1) / kMatchTile;
  const int c0 = parts_quotient(used * part, parts), c1 = parts_quotient(used * (part + 1), parts);
  // one tile: TAIL, the last one, has rows past the set's end
  auto walk = [&](auto tail, const _Float16* buf, int ct) {
    constexpr bool TAIL = decltype(tail)::value;
    const int o0 = ct * kMatchTile + 64 * oth_half + 4 * gq;   // the lane's other row at ta = r = 0
    int code[OB];   // 4 ta + r of the new nearest
#pragma unroll
    for (int tb = 0; tb < OB; ++tb) code[tb] = -1;
    auto products = [&](int ta, float4v* acc) {
#pragma unroll
      for (int tb = 0; tb < OB; ++tb) acc[tb] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const half8 fa = *reinterpret_cast<const half8*>(
            &buf[(64 * oth_half + 16 * ta + li) * kStride +
                 (HALF ? (32 * kk + 8 * gq) ^ (8 * li) : 32 * kk + 8 * gq)]);
#pragma unroll
        for (int tb = 0; tb < OB; ++tb)
          acc[tb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa, fb[tb][kk], acc[tb], 0, 0, 0);
      }
    };
    float4v acc[OB];
#pragma unroll
    for (int ta = 0; ta < 4; ++ta) {
      products(ta, acc);
      // A lane meets its other rows in increasing order, so a tie keeps the
      // earlier one: "nearer" is a strict comparison.  v2 <= v1: the second
      // largest of the three is their median.
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int tb = 0; tb < OB; ++tb) {
          float s = acc[tb][r];
          if (TAIL) s = o0 + 16 * ta + r < n_oth ? s : -INFINITY;
          const bool up = s > v1[tb];
          code[tb] = up ? 4 * ta + r : code[tb];
          v2[tb] = __builtin_amdgcn_fmed3f(v1[tb], v2[tb], s);
          v1[tb] = up ? s : v1[tb];
        }
      // One block's comparisons end here and one block's products are in flight,
      // no more: left alone, the compiler keeps all 64 values and takes 256
      // registers.
#pragma unroll
      for (int tb = 0; tb < OB; ++tb)
        __asm__ volatile("" : "+v"(v1[tb]), "+v"(v2[tb]), "+v"(code[tb]));
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int tb = 0; tb < OB; ++tb)
      i1[tb] = code[tb] >= 0 ? o0 + 16 * (code[tb] >> 2) + (code[tb] & 3) : i1[tb];
  };
  auto step = [&](int ct, const _Float16* buf, _Float16* next) {
    if (ct + 1 < c1) stage(ct + 1, next);
    if ((ct + 1) * kMatchTile > n_oth)
      walk(std::true_type(), buf, ct);
    else
      walk(std::false_type(), buf, ct);
    __syncthreads();
  };
  if (c0 < c1) stage(c0, s_t0);
  __syncthreads();
  for (int ct = c0; ct < c1; ct += 2) {
    step(ct, s_t0, s_t1);
    if (ct + 1 < c1) step(ct + 1, s_t1, s_t0);
  }
  // merge the four lanes of an own row, then the two halves of the tiles
#pragma unroll
  for (int tb = 0; tb < OB; ++tb) {
    Top2 v;
    v.v1 = v1[tb];
    v.i1 = i1[tb];
    v.v2 = v2[tb];
    v.pad = 0;
    v = top2_merge(v, top2_shfl_xor(v, 16));
    v = top2_merge(v, top2_shfl_xor(v, 32));
    if (gq == 0) s_part[oth_half][16 * OB * own_half + 16 * tb + li] = v;
  }
  __syncthreads();
  if (t < kOwn && row0 + t < n_own) {
    SIFT_CHECK_INDEX(row0 + t, cap_own);
    Top2* out = parts == 1 ? best_of(h, e, b_side) : part_of(h, e, b_side, part);
    out[row0 + t] = top2_merge(s_part[0][t], s_part[1][t]);
  }
}

// The nearest over all parts of row i of one set.
__device__ __forceinline__ Top2 best_at(const MatchHdr& h, const MatchEntry& e, int b_side, int i) {
  const int parts = parts_of(e, b_side);
  if (parts == 1 || h.merged) return best_of(h, e, b_side)[i];
  Top2 c = part_of(h, e, b_side, 0)[i];
  for (int q = 1; q < parts; ++q) c = top2_merge(c, part_of(h, e, b_side, q)[i]);
  return c;
}

// Merge of the parts, one thread per row of either set.
__global__ __launch_bounds__(kMatchMergeBlock) void k_match_merge(MatchHdr h, int n) {
  int local;
  const int p = pair_of_rows(h, n, blockIdx.x, &local);
  const MatchEntry e = entry_of(h, p);
  int i = local * kMatchMergeBlock + threadIdx.x;
  const int b_side = i >= e.cap_a;
  if (b_side) i -= e.cap_a;
  if (i >= (b_side ? rows_in_use(e.count_b, e.cap_b) : rows_in_use(e.count_a, e.cap_a))) return;
  if (parts_of(e, b_side) == 1) return;   // one part is the whole walk
  SIFT_CHECK_INDEX(i, b_side ? e.cap_b : e.cap_a);
  best_of(h, e, b_side)[i] = best_at(h, e, b_side, i);
}

// Squared distance of unit vectors from a similarity, in fp32.
__device__ __forceinline__ float sq_dist(float s) { return fmaxf(2.0f - 2.0f * s, 0.0f); }

__device__ __forceinline__ bool ratio_pass(const Top2& t, float ratio_sq) {
  const float d1 = sq_dist(t.v1);
  const float d2 = t.v2 == -INFINITY ? 4.0f : sq_dist(t.v2);
  return d1 < ratio_sq * d2;
}

// Mutual nearest neighbours passing both ratio tests, written in ascending
// query order (one work-group per pair).  Up to kEmitRows x 1024 rows are taken
// together: their loads are all in flight at once, and one scan of the waves'
// counts places them (a scan per 256 rows took 36 us for 8192 rows).
constexpr int kEmitThreads = 1024, kEmitRows = 8;

__global__ __launch_bounds__(kEmitThreads) void k_match_emit(MatchHdr h, int n, float ratio_sq) {
  constexpr int kCounts = kEmitRows * kEmitThreads / 64;   // one per 64 rows
  __shared__ int s_cnt[kCounts], s_wave[4];
  const MatchEntry e = entry_of(h, blockIdx.x);
  const int na = rows_in_use(e.count_a, e.cap_a);
  const int nb = rows_in_use(e.count_b, e.cap_b);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int base = 0;
  const int rows = nb > 0 ? na : 0;
  for (int i0 = 0; i0 < rows; i0 += kEmitRows * kEmitThreads) {
    Top2 rb[kEmitRows];
    unsigned long long kept[kEmitRows];
#pragma unroll
    for (int u = 0; u < kEmitRows; ++u) {
      const int i = i0 + u * kEmitThreads + t;
      rb[u] = top2_empty();
      if (i < rows) {
        SIFT_CHECK_INDEX(i, e.cap_a);
        rb[u] = best_at(h, e, 0, i);
      }
    }
#pragma unroll
    for (int u = 0; u < kEmitRows; ++u) {
      const int i = i0 + u * kEmitThreads + t, j = rb[u].i1;
      bool keep = false;
      if (i < rows && j >= 0 && j < nb) {
        SIFT_CHECK_INDEX(j, e.cap_b);
        const Top2 cb = best_at(h, e, 1, j);
        keep = cb.i1 == i && ratio_pass(rb[u], ratio_sq) && ratio_pass(cb, ratio_sq);
      }
      kept[u] = __ballot(keep);
      if (lane == 0) s_cnt[u * (kEmitThreads / 64) + wave] = __popcll(kept[u]);
    }
    __syncthreads();
    // exclusive prefix of the counts (in row order), by the first two waves
    int c = t < kCounts ? s_cnt[t] : 0;
    const int incl = wave_incl_scan(c);
    if (t < kCounts && lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int before = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < kCounts / 64; ++w) {
      if (w < wave) before += s_wave[w];
      sum += s_wave[w];
    }
    if (t < kCounts) s_cnt[t] = before + incl - c;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kEmitRows; ++u) {
      const int at = base + s_cnt[u * (kEmitThreads / 64) + wave] +
                     __popcll(kept[u] & lanemask_lt());
      if ((kept[u] >> lane & 1ull) && at < e.capacity) {
        sift_match m;
        m.query = i0 + u * kEmitThreads + t;
        m.train = rb[u].i1;
        m.similarity = rb[u].v1;
        m.distance = sqrtf(sq_dist(rb[u].v1));
        SIFT_CHECK_INDEX(at, e.capacity);
        e.matches[at] = m;
      }
    }
    base += sum;
    __syncthreads();   // the counts are read before the next rows' are written
  }
  if (t == 0) {
    *e.n_matches = base < e.capacity ? base : e.capacity;
    if (e.n_found) *e.n_found = base;
  }
}

hipError_t launch_match_setup(const MatchHdr& h, const MatchSetupChunk& c, int n,
                              hipStream_t stream) {
  return launch(k_match_setup, dim3(1), dim3(64), stream, const_cast<MatchEntry*>(h.table),
                h.row_prefix, h.col_prefix, c, n);
}

hipError_t launch_match_rows(const MatchHdr& h, int n, int grid, hipStream_t stream) {
  if (h.half) {
    const hipError_t e = launch(k_match_half, dim3(h.half), dim3(256), stream, h, n);
    if (e != hipSuccess) return e;
  }
  const int items = (grid + kXcds - 1) / kXcds * kXcds;
  return launch(h.half ? k_match_best<true, kMatchOwnHalf / 32> : k_match_best<false, kMatchTile / 32>,
                dim3(items), dim3(256), stream, h, n, grid);
}

hipError_t launch_match_cols(const MatchHdr& h, int n, int grid, hipStream_t stream) {
  return launch(k_match_merge, dim3(grid), dim3(kMatchMergeBlock), stream, h, n);
}

hipError_t launch_match_emit(const MatchHdr& h, int n, float ratio_sq, hipStream_t stream) {
  return launch(k_match_emit, dim3(n), dim3(kEmitThreads), stream, h, n, ratio_sq);
}

// The bounds-check counter of this file's kernels (see check_index).
hipError_t bounds_count_match(unsigned long long* count, bool reset) {
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
