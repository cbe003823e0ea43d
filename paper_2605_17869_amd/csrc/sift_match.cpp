// Host runtime of descriptor matching: argument checks, workspace layout and
// the launch sequence (setup, nearest neighbours, merge of parts, emission).
// Like extraction, it never allocates device memory, copies or synchronises.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/sift.h"
#include "sift_match.h"

namespace sift {
void set_last_error(const std::string& msg);
}

using namespace sift;

namespace {

sift_status fail(sift_status st, const std::string& msg) {
  set_last_error(msg);
  return st;
}

int64_t align256(int64_t v) { return (v + 255) / 256 * 256; }
int cdiv_i(int a, int b) { return (a + b - 1) / b; }

struct MatchLayout {
  int64_t table, row_prefix, col_prefix;
  std::vector<int64_t> best, part, half;
  std::vector<int> parts_a, parts_b;   // parts of the walks over the other set
  int own_rows = kMatchTile;
  bool half_copies = false, merge = false;
  int64_t bytes;
};

sift_status check_pairs(int32_t n, const sift_match_pair* pairs) {
  if (n < 1) return fail(SIFT_ERR_INVALID_ARG, "at least one pair");
  if (n > SIFT_MATCH_MAX_PAIRS)
    return fail(SIFT_ERR_TOO_LARGE, "at most " + std::to_string(SIFT_MATCH_MAX_PAIRS) + " pairs");
  if (!pairs) return fail(SIFT_ERR_INVALID_ARG, "null pairs");
  for (int i = 0; i < n; ++i) {
    const sift_match_pair& q = pairs[i];
    const std::string at = "pair " + std::to_string(i) + ": ";
    if (q.cap_a < 0 || q.cap_a > SIFT_MATCH_MAX_ROWS || q.cap_b < 0 || q.cap_b > SIFT_MATCH_MAX_ROWS)
      return fail(SIFT_ERR_INVALID_ARG, at + "caps must be in 0.." + std::to_string(SIFT_MATCH_MAX_ROWS));
    if ((q.cap_a > 0 && !q.desc_a) || (q.cap_b > 0 && !q.desc_b))
      return fail(SIFT_ERR_INVALID_ARG, at + "null descriptors");
    if (q.capacity < 0) return fail(SIFT_ERR_INVALID_ARG, at + "negative capacity");
    if ((q.capacity > 0 && !q.matches) || !q.n_matches)
      return fail(SIFT_ERR_INVALID_ARG, at + "null output");
    if ((reinterpret_cast<uintptr_t>(q.desc_a) | reinterpret_cast<uintptr_t>(q.desc_b)) % 16)
      return fail(SIFT_ERR_INVALID_ARG, at + "descriptors must be 16-byte aligned");
  }
  return SIFT_OK;
}

// Work-groups of the nearest-neighbour kernel that fill the chip: two on each
// of 256 CUs (32 pairs of 2000 x 2000: 512 row tiles, 0.114 ms; in two parts each 0.123).
constexpr int64_t kMatchTargetGroups = 512;
// Similarity tiles from which the sets are first copied to fp16: below, a tile
// is staged so few times that a launch of its own costs more than converting
// it again (one pair of 2000 x 2000: 256 tiles; 8192 x 7900: 3968).
constexpr int64_t kMatchHalfTiles = 1024;
// ... and only where a tile of the sets is staged that often on average: a copy moves
// 6 bytes per value to save 2 of 4 each time the value is read.  With and without
// copies, us: 1000 pairs of 500 x 500 (4 stagings) 485 and 468, 100 of 640 x 640 (5) 85
// and 73, 100 of 700 x 700 (6) 93 and 91, one of 65536 x 500 (8) 256 and 266.
constexpr int64_t kMatchHalfStagings = 7;
// Rows of a pair's sets up to which the emission merges the parts itself.
constexpr int64_t kMatchEmitMergeRows = 2048;

// The plan of a call and its workspace.  `half`: the sets are copied to fp16 first where
// that pays; `most`: parts that a walk may be cut into.  Without copies and in one part a
// call runs in the least memory.
MatchLayout layout_of(int32_t n, const sift_match_pair* pairs, bool half, int most) {
  MatchLayout L;
  int64_t off = 0;
  L.table = off;
  off = align256(off + (int64_t)n * (int64_t)sizeof(MatchEntry));
  L.row_prefix = off;
  off = align256(off + (int64_t)(n + 1) * 4);
  L.col_prefix = off;
  off = align256(off + (int64_t)(n + 1) * 4);
  int64_t row_tiles = 0, tiles = 0;
  int most_rows = 0;
  for (int i = 0; i < n; ++i) {
    const int ta = cdiv_i(pairs[i].cap_a, kMatchTile), tb = cdiv_i(pairs[i].cap_b, kMatchTile);
    row_tiles += ta + tb;
    tiles += (int64_t)ta * tb;
    most_rows = std::max(most_rows, pairs[i].cap_a + pairs[i].cap_b);
  }
  L.half_copies =
      half && tiles >= kMatchHalfTiles && 2 * tiles >= kMatchHalfStagings * row_tiles;
  if (L.half_copies) L.own_rows = kMatchOwnHalf;
  // A walk is cut where it is longer than every group's share of all tiles, be it that
  // the call has few groups (8192 x 7900 without parts: 63 of them) or that one set is
  // much longer than the other (65536 x 100: 512 walks of one tile and one of 512, 1264
  // us while only the number of groups was looked at, 252 now; 32 pairs of 4096 x 128
  // 128 and 56).
  int64_t steps = 0;
  for (int i = 0; i < n; ++i) {
    const int ca = pairs[i].cap_a, cb = pairs[i].cap_b;
    steps += (int64_t)cdiv_i(ca, L.own_rows) * cdiv_i(cb, kMatchTile) +
             (int64_t)cdiv_i(cb, L.own_rows) * cdiv_i(ca, kMatchTile);
  }
  const int walk = (int)std::min<int64_t>(std::max<int64_t>(steps / kMatchTargetGroups, 1),
                                          SIFT_MATCH_MAX_ROWS);   // tiles of a part
  for (int i = 0; i < n; ++i) {
    const int64_t rows = (int64_t)pairs[i].cap_a + pairs[i].cap_b;
    L.best.push_back(off);
    off = align256(off + rows * (int64_t)sizeof(Top2));
    L.part.push_back(off);
    const int pa = match_parts(walk, pairs[i].cap_b, most);
    const int pb = match_parts(walk, pairs[i].cap_a, most);
    L.parts_a.push_back(pa);
    L.parts_b.push_back(pb);
    L.merge = L.merge || ((pa > 1 || pb > 1) && most_rows > kMatchEmitMergeRows);
    const int64_t kept = (pa > 1 ? (int64_t)pa * pairs[i].cap_a : 0) +
                         (pb > 1 ? (int64_t)pb * pairs[i].cap_b : 0);
    off = align256(off + kept * (int64_t)sizeof(Top2));
    L.half.push_back(off);
    if (L.half_copies) off = align256(off + rows * 128 * 2);
  }
  L.bytes = off;
  return L;
}

// The best plan that fits: the one sift_match_workspace_size reports, then without
// copies, then in fewer parts.
MatchLayout layout_within(int32_t n, const sift_match_pair* pairs, int64_t bytes) {
  MatchLayout L = layout_of(n, pairs, true, kMatchMaxParts);
  for (int most = kMatchMaxParts; L.bytes > bytes && most >= 1; most /= 2)
    L = layout_of(n, pairs, false, most);
  return L;
}

}  // namespace

extern "C" {

sift_status sift_match_workspace_size(int32_t n, const sift_match_pair* pairs, size_t* bytes) {
  if (!bytes) return fail(SIFT_ERR_INVALID_ARG, "null bytes");
  sift_status st = check_pairs(n, pairs);
  if (st != SIFT_OK) return st;
  *bytes = (size_t)layout_of(n, pairs, true, kMatchMaxParts).bytes;
  return SIFT_OK;
}

sift_status sift_match_batch(int32_t n, const sift_match_pair* pairs, float ratio,
                             void* d_workspace, size_t workspace_bytes, void* stream_v) {
  sift_status st = check_pairs(n, pairs);
  if (st != SIFT_OK) return st;
  if (!(ratio > 0.0f && ratio <= 1.0f)) return fail(SIFT_ERR_INVALID_ARG, "ratio must be in (0, 1]");
  if (!d_workspace) return fail(SIFT_ERR_INVALID_ARG, "null workspace");
  if (reinterpret_cast<uintptr_t>(d_workspace) % 256)
    return fail(SIFT_ERR_INVALID_ARG, "workspace must be 256-byte aligned");
  const MatchLayout L = layout_within(n, pairs, (int64_t)workspace_bytes);
  if ((int64_t)workspace_bytes < L.bytes)
    return fail(SIFT_ERR_WORKSPACE_TOO_SMALL, "workspace " + std::to_string(workspace_bytes) +
                                                  " bytes, need " + std::to_string(L.bytes));
  hipStream_t stream = reinterpret_cast<hipStream_t>(stream_v);
  char* ws = static_cast<char*>(d_workspace);
  MatchHdr h;
  std::memset(&h, 0, sizeof h);
  h.ws = ws;
  h.table = reinterpret_cast<const MatchEntry*>(ws + L.table);
  h.row_prefix = reinterpret_cast<int*>(ws + L.row_prefix);
  h.col_prefix = reinterpret_cast<int*>(ws + L.col_prefix);
  h.merged = 0;
  h.own_rows = L.own_rows;

  std::vector<int> rp(n + 1, 0), cp(n + 1, 0);
  for (int i = 0; i < n; ++i) {
    rp[i + 1] = rp[i] + cdiv_i(pairs[i].cap_a, L.own_rows) * L.parts_a[i] +
                cdiv_i(pairs[i].cap_b, L.own_rows) * L.parts_b[i];
    cp[i + 1] = cp[i] + cdiv_i(pairs[i].cap_a + pairs[i].cap_b, kMatchMergeBlock);
  }
  h.half = L.half_copies ? cp[n] : 0;
  h.same_items = rp[1];
  for (int i = 1; i < n; ++i)
    if (rp[i + 1] - rp[i] != rp[1]) h.same_items = 0;
  auto hip_fail = [](hipError_t e, const char* what) {
    return fail(SIFT_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
  };
  hipError_t e;
  auto entry = [&](int i) {
    const sift_match_pair& q = pairs[i];
    MatchEntry m;
    std::memset(&m, 0, sizeof m);
    m.desc_a = q.desc_a;
    m.count_a = q.count_a;
    m.desc_b = q.desc_b;
    m.count_b = q.count_b;
    m.matches = q.matches;
    m.n_matches = q.n_matches;
    m.n_found = q.n_found;
    m.cap_a = q.cap_a;
    m.cap_b = q.cap_b;
    m.capacity = q.capacity;
    m.parts_a = (int16_t)L.parts_a[i];
    m.parts_b = (int16_t)L.parts_b[i];
    m.best = L.best[i];
    m.part = L.part[i];
    m.half = L.half[i];
    return m;
  };
  h.carried = n <= kMatchOwnPairs ? 1 : 0;
  for (int i = 0; h.carried && i <= n; ++i) {
    h.rows[i] = rp[i];
    h.cols[i] = cp[i];
    if (i < n) h.e[i] = entry(i);
  }
  for (int first = 0; !h.carried && first < n; first += kMatchSetupChunk) {
    MatchSetupChunk c;
    std::memset(&c, 0, sizeof c);
    c.first = first;
    c.count = std::min(kMatchSetupChunk, n - first);
    for (int t = 0; t < c.count; ++t) c.e[t] = entry(first + t);
    for (int t = 0; t <= c.count; ++t) {
      c.row_prefix[t] = rp[first + t];
      c.col_prefix[t] = cp[first + t];
    }
    if ((e = launch_match_setup(h, c, n, stream)) != hipSuccess) return hip_fail(e, "match setup");
  }
  if (rp[n] > 0 && (e = launch_match_rows(h, n, rp[n], stream)) != hipSuccess)
    return hip_fail(e, "match similarity");
  if (L.merge && cp[n] > 0) {
    if ((e = launch_match_cols(h, n, cp[n], stream)) != hipSuccess) return hip_fail(e, "match merge");
    h.merged = 1;
  }
  const float ratio_sq = (float)((double)ratio * (double)ratio);
  if ((e = launch_match_emit(h, n, ratio_sq, stream)) != hipSuccess) return hip_fail(e, "match emit");
  return SIFT_OK;
}

}  // extern "C"
