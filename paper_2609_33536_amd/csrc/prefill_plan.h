// Parts of the prefill launch that also compile for the host (internal
// header): which kernel a launch uses, and which work a workgroup takes.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ekv {

// Whether a launch that would have `workgroups` workgroups of 32 columns uses
// prefill_split_kernel (`columns`: the longest chunk's; max_len: the context
// bound, stated by the caller or the table's width).  Measured (us, bf16, half
// BASE, 128-column / split kernel):
//  - contexts of one unit and at most 64 columns: never (three waves would have
//    no unit).  4 prompts of up to 32 rows, 16 / 16 heads 6.0 / 6.7, 8-bit 6.1 / 7.0;
//    12 of up to 16 rows, 32 / 8 heads 6.6 / 7.0 (but 32 rows 8.6 / 6.7 for one);
//  - else up to 256 workgroups (one a CU): always.  128 workgroups of 8 rows over
//    16-215 keys 12.9 / 10.1, over 4096 112 / 57;
//  - up to 512 over contexts of at least 512 keys, where a quarter of the chain
//    saves more than the second round's start and merge cost: 384 and 512
//    workgroups with one context of 4096 among short ones 112 / 53 and 113 / 54,
//    three chunks of 130 rows over 2000 keys 68 / 59; all contexts alike 384
//    x 1100 42 / 43, 512 x 1100 43 / 48; short ones 512 x 16-215 16.1 / 19.1;
//  - chunks of one 32-column tile leave three of prefill_kernel's waves without
//    columns whatever the number of workgroups: up to 2048 over contexts of at
//    least 1024 keys.  One context of 4096 among short ones at 528 / 1024 / 2048
//    workgroups 114 / 55, 115 / 56, 116 / 68; all of 2000 keys 127 / 106, 152 /
//    157, 298 / 300.  Beyond, the split kernel's single workgroup a CU costs
//    more: one long context at 4096 and 8192 workgroups 119 / 135, 209 / 266
//    (all of 4096 keys 1126 / 1088, 2230 / 2154).  And only if the caller states
//    the bound: the table's width says nothing about the lengths, and all-short
//    batches lose (16-215 keys at 528 / 1024 / 2048 workgroups 20.4 / 22.7, 28.5 /
//    33.9, 49 / 64).
inline bool divide_units(int64_t workgroups, int64_t columns, int max_len, bool stated) {
  constexpr int64_t kCus = 256;
  if (stated && max_len <= 32 && columns <= 64) return false;
  return workgroups <= kCus || (workgroups <= 2 * kCus && max_len >= 512) ||
         (workgroups <= 8 * kCus && columns <= 32 && stated && max_len >= 1024);
}

// Whether the tiles of a (sequence, KV head) are spread over the XCDs where the
// number of KV heads is not a multiple of 8 (groups: batch * num_kv_heads; rows:
// of all chunks; most_rows: if every chunk were as long as the longest).  Ids go
// round robin over the 8 XCDs, so with groups a multiple of 8 every tile of a
// (sequence, KV head) lands on one XCD: its K and V stay in one L2, but sequences
// of unlike lengths load the XCDs unevenly.  So they are spread if the chunks
// are ragged, or if an XCD would have fewer than 4 of them (an odd number of
// groups spreads by itself).  Measured (us, one XCD / spread): 16 x (2048 + 512)
// ragged, 16 / 1 heads 181 / 122, 32 / 4 heads 258 / 211; 16 x 0-1024, 16 / 2 heads 111
// / 63; 64 chunks of up to 300 rows, 16 / 1 heads 73 / 52; alike, 16 x (2048 + 512),
// 32 / 4 heads 460 / 489, 16 / 1 heads 231 / 238.
inline bool spread_tiles(int64_t groups, int64_t rows, int64_t most_rows) {
  return groups % 2 == 0 && (groups < 32 || 8 * rows < 7 * most_rows);
}

struct PrefillPlace {
  int seq, kv_head, tile;
};

// Workgroup (bx, by) of a grid of gx = tiles * num_kv_heads by gy = batch ->
// (sequence, KV head), query tile; the last tiles (most keys) first.  Ids go
// round robin over the 8 XCDs: with a multiple of 8 KV heads all tiles of one
// (sequence, KV head) go to one XCD and share its L2, and every XCD gets a KV
// head of every sequence; otherwise see spread_tiles.
// (Two grid dimensions only for the launch's size limits.  A grid of 2^31
// workgroups or more has no 32-bit id and takes the dimensions as they are: a
// batch of tens of thousands of sequences with one very long chunk, nearly all
// of whose workgroups have nothing to do.)
__host__ __device__ inline PrefillPlace place_workgroup(uint32_t bx, uint32_t by, uint32_t gx, uint32_t gy, int tiles,
                                                        int num_kv_heads, int batch, bool spread) {
  if ((uint64_t)gx * gy >> 31)
    return {(int)by, (int)(bx % (uint32_t)num_kv_heads), tiles - 1 - (int)(bx / (uint32_t)num_kv_heads)};
  const int id = (int)(by * gx + bx);
  int group, tile;   // group: sequence * num_kv_heads + KV head
  if (num_kv_heads % 8 == 0) {
    const int i = id >> 3;
    group = 8 * (i / tiles) + (id & 7);
    tile = i % tiles;
  } else {
    const int groups = batch * num_kv_heads;
    tile = id / groups;
    group = (id % groups + (spread ? tile : 0)) % groups;
  }
  return {group / num_kv_heads, group % num_kv_heads, tiles - 1 - tile};
}

}  // namespace ekv
