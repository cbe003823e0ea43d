// Internal definitions of descriptor matching shared by the host runtime and
// the gfx950 kernels: the on-device pair table, workspace layout and launch
// helpers.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <hip/hip_runtime.h>

#include "../../include/sift.h"

namespace sift {

constexpr int kMatchTile = 128;      // rows of either set per similarity tile
constexpr int kMatchOwnHalf = 256;    // own rows of a work-group where the sets are copied to fp16
constexpr int kMatchMergeBlock = 256; // rows per block of the merge and of the copies
constexpr int kMatchSetupChunk = 24; // pair-table entries per setup launch
// Pairs whose entries every kernel carries in its arguments (3.3 KiB of the 4 they may
// take) instead of reading a table that launches of their own write first: one pair of
// 300 x 263 rows 17.0 -> 15.1 us, 32 pairs of 2000 x 2000 (two such launches) 103 -> 99.
constexpr int kMatchOwnPairs = 32;
constexpr int kMatchMaxParts = 8;    // most parts of a walk over the other set

// Parts that a walk over a set of `cap` rows is cut into, of about `walk` tiles each, at
// most `most`.
inline int match_parts(int walk, int cap, int most) {
  const int tiles = (cap + kMatchTile - 1) / kMatchTile;
  const int parts = (tiles + walk - 1) / walk;
  return parts < 1 ? 1 : (parts < most ? parts : most);
}

// Running nearest / second-nearest of one row or column: the best candidate
// (largest value, smallest index among equals) and the largest value among
// the others.  An empty set holds (-inf, INT32_MAX, -inf).
struct Top2 {
  float v1;
  int32_t i1;
  float v2;
  int32_t pad;
};

// One pair as the kernels see it (written by the setup kernel).
struct MatchEntry {
  const float* desc_a;
  const int32_t* count_a;
  const float* desc_b;
  const int32_t* count_b;
  sift_match* matches;
  int32_t* n_matches;
  int32_t* n_found;
  int32_t cap_a, cap_b, capacity;
  int16_t parts_a, parts_b;   // parts of the walks of a's and of b's rows over the other set
  int64_t best;            // Top2 [cap_a], then Top2 [cap_b]: a_i's nearest in b, b_j's in a
  int64_t part;            // the same per part, of a set whose walk is cut: Top2 [parts][cap_a], then [parts][cap_b]
  int64_t half;            // fp16 copies of the sets: [cap_a][128], then [cap_b][128]
};

// Device addresses of the header arrays (computed on the host).
struct MatchHdr {
  char* ws;
  const MatchEntry* table;   // [n]
  int* row_prefix;           // [n + 1] walks' parts (of both sets' row tiles) before each pair
  int* col_prefix;           // [n + 1] merge blocks (of both sets) before each pair
  int half;                  // > 0: the sets are copied to fp16 first, by so many work-groups
  int merged;                // 1: the parts' results have been merged into `best`
  int own_rows;              // rows per row tile: kMatchTile or kMatchOwnHalf
  int same_items;            // what row_prefix counts of every pair when all have as many, else 0
  int carried;               // 1: the arrays are those below, not the header's
  int rows[kMatchOwnPairs + 1], cols[kMatchOwnPairs + 1];   // the prefixes
  MatchEntry e[kMatchOwnPairs];
};
static_assert(sizeof(MatchHdr) <= 4000, "kernel arguments");

struct MatchSetupChunk {
  int first;
  int count;
  MatchEntry e[kMatchSetupChunk];
  int row_prefix[kMatchSetupChunk + 1];
  int col_prefix[kMatchSetupChunk + 1];
};

hipError_t launch_match_setup(const MatchHdr& h, const MatchSetupChunk& c, int n,
                              hipStream_t stream);
// grid: walks' parts of all pairs (row_prefix[n])
hipError_t launch_match_rows(const MatchHdr& h, int n, int grid, hipStream_t stream);
// merge of the parts; grid: merge blocks of all pairs (col_prefix[n])
hipError_t launch_match_cols(const MatchHdr& h, int n, int grid, hipStream_t stream);
hipError_t launch_match_emit(const MatchHdr& h, int n, float ratio_sq, hipStream_t stream);

}  // namespace sift
