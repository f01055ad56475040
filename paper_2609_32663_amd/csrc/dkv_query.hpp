// Launch interface of query-block attention (argument checks live in the
// C-ABI layer; the launcher assumes validated arguments).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace dkv {

constexpr int kQueryRowsPerWG = 256;     // query rows (tokens x heads of a group) per workgroup
constexpr int kQueryTargetItems = 512;   // workgroups a split call aims at: two per compute unit
constexpr int kQueryMinTiles = 8;        // 64-key tiles per key range at least
constexpr int kQueryUnknownTiles = 512;  // key tiles per segment assumed when the caller gives no hint
constexpr int kQueryPlanHead = 4;        // plan words before the first-item table

struct QueryParams {
  const void* q;           // [B][n_q][Hq][d] bf16
  const void* k;           // packed K rows (bf16)
  const void* v;
  const int64_t* seg_off;  // [B*Hkv]
  const int32_t* seg_len;  // [B*Hkv]
  int32_t n_tail;          // tokens appended before the block
  int32_t n_q;             // tokens in the block (already appended after them)
  int32_t nseg, Hkv, Hq, G;
  int32_t rows;            // query rows per segment: n_q * G
  int32_t qtiles;          // ceil(rows / kQueryRowsPerWG)
  int32_t tiles_per_range; // C before the plan kernel's check against max_items
  int32_t max_items;       // items the records hold
  float scale_log2;        // sm_scale * log2(e)
  float* out;              // [B][n_q][Hq][d] fp32
  // Split calls only (nullptr otherwise): plan words [0] items, [1] tiles per
  // range, then [kQueryPlanHead + s] first item of segment s (s <= nseg); and
  // the records [max_items][kQueryRowsPerWG][d + 2] (max, sum, output).
  int32_t* plan;
  float* rec;
  // Short blocks (rows <= kShortRows) only: workgroups of the split (0: no
  // split, one workgroup per segment), rows of a record (a multiple of 4;
  // record slot x holds rec_rows maxima, sums and then outputs of d floats),
  // and per segment the first record slot and the piece count.
  int32_t P, rec_rows;
  int32_t stream_once;     // load K and V past the caches
  int32_t* seg_meta;
};

// How a call is split, from the shapes and the caller's hint of the total
// rows (0 = unknown) only, so the workspace size is known before the call.
struct QueryPlanShape {
  int32_t qtiles;
  int64_t tiles_per_range;
  int64_t max_items;   // attention workgroups launched
  size_t plan_bytes;   // 0: no split, one workgroup per (segment, query tile)
  size_t rec_bytes;
};

QueryPlanShape query_plan_shape(int32_t nseg, int32_t rows, int32_t head_dim, int64_t rows_hint);
// Short blocks: most query rows per segment, and most segments of a call (the
// workgroups' prefix over them shares the LDS with the tiles).
constexpr int kShortRows = 256;
constexpr int kShortSegments = 512;
// Whether the short kernels take a call, where they are level or ahead; long /
// short, us, attention and combine.
//   * Up to 64 rows: always.
//   * Up to 128 rows: but for many segments of few keys, where a piece is little
//     more than its start and its record and the long kernel's items fit one
//     round of workgroups or, with more than 96 rows, nearly fill two (128 rows
//     of 64 dimensions: 128 segments of 960 keys 36 / 55, 80 of 1,400 33 / 41, 160
//     of 1,400 58 / 69; a started second round turns it: 160 of 1,000 66 / 59, 96
//     of 1,250 57 / 46; 65 rows, 256 unequal segments of 1,700 141 / 86).
//   * More rows leave one key wave and up to 133 KB of record per piece, so the
//     segments have to be long (240 rows: 128 segments of 1,050 keys 85.8 /
//     110.9, 8 of 11,500 54.7 / 41.2) and few; with 128 dimensions the long
//     kernel's overlapped products win again once all the keys are many (192
//     rows: 8 segments of 120,000 199 / 180, 16 of 45,000 151 / 147, of 120,000
//     341 / 371, 32 of 9,000 83 / 81, of 45,000 256 / 280, 128 of 9,000 214 /
//     261; of 64 dimensions 32 of 45,000 203 / 196).
constexpr int64_t kShortLongKeys = 8192;  // keys per segment on average
constexpr int kShortManySegments = 48;
constexpr int64_t kShortFewKeys = 2048;
inline bool query_takes_short(int32_t nseg, int32_t rows, int32_t head_dim, int64_t rows_hint,
                              const QueryPlanShape& sh) {
  if (rows > kShortRows || nseg > kShortSegments) return false;
  if (rows <= kShortRows / 4) return true;
  if (rows <= kShortRows / 2) {
    if (sh.plan_bytes == 0 || nseg < kShortManySegments || rows_hint <= 0 || rows_hint / kShortFewKeys >= nseg)
      return true;
    const int64_t tiles = (rows_hint / nseg + 63) / 64;  // of a segment, on average
    const int64_t items = nseg * ((tiles + sh.tiles_per_range / 2) / sh.tiles_per_range);
    return items > kQueryTargetItems / 2 && (items < 400 || rows <= 96);
  }
  return sh.plan_bytes > 0 && rows_hint / kShortLongKeys >= nseg && nseg <= 32 &&
         (head_dim == 64 || rows_hint <= (int64_t(1) << 24) / nseg);
}
// K and V of a call up to this size may still be in the 256 MB last-level
// cache from the call before (the block's append, the last step), so they are
// loaded normally; larger ones are streamed past the caches.
constexpr int64_t kShortCachedBytes = 96 << 20;
hipError_t launch_query_short(const QueryParams& p, int head_dim, hipStream_t stream);
hipError_t launch_query_attn(const QueryParams& p, int head_dim, int64_t grid, hipStream_t stream);

}  // namespace dkv
