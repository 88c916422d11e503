// Parts of the prefill launch that also compile for the host (internal
// header): which work a workgroup of the grid takes.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ekv {

struct PrefillPlace {
  int seq, kv_head, tile;
};

// Workgroup (bx, by) of a grid of gx = tiles * num_kv_heads by gy = batch ->
// (sequence, KV head), query tile; the last tiles (most keys) first.  Ids go
// round robin over the 8 XCDs: with a multiple of 8 KV heads all tiles of one
// (sequence, KV head) go to one XCD and share its L2, and every XCD gets a KV
// head of every sequence; otherwise whole (sequence, KV head)s would load the
// XCDs unevenly (12 of them: 1.4x the time), and the tiles are spread instead.
// (Two grid dimensions only for the launch's size limits.  A grid of 2^31
// workgroups or more has no 32-bit id and takes the dimensions as they are: a
// batch of tens of thousands of sequences with one very long chunk, nearly all
// of whose workgroups have nothing to do.)
__host__ __device__ inline PrefillPlace place_workgroup(uint32_t bx, uint32_t by, uint32_t gx, uint32_t gy, int tiles,
                                                        int num_kv_heads, int batch) {
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
    group = id % groups;
    tile = id / groups;
  }
  return {group / num_kv_heads, group % num_kv_heads, tiles - 1 - tile};
}

}  // namespace ekv
