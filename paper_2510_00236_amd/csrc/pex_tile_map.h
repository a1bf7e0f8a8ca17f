// pex_tile_map.h -- workgroup id -> tile of S, shared by the MFMA contraction kernels.  Device code only.
#pragma once

#include <hip/hip_runtime.h>

namespace pex {
namespace {

// Workgroup id -> (split, tile_m, tile_n): undo the round-robin assignment of consecutive ids to the 8 XCDs,
// then walk tiles in groups of GROUP_M tile rows so the workgroups resident on one XCD form a compact patch
// that shares X and G panels in that XCD's L2.
// `id` of the `n` workgroups of a layer; they may be a part of a launch (any eight consecutive ids are on eight XCDs)
__device__ __forceinline__ void map_workgroup(int n, int id, int tiles_m, int tiles_n, int& split, int& tm, int& tn)
{
    const int xcd = id % 8, local = id / 8;
    const int base = n / 8, rem = n % 8;
    const int nid = xcd * base + (xcd < rem ? xcd : rem) + local;
    const int tiles = tiles_m * tiles_n;
    split = nid / tiles;
    const int q = nid - split * tiles;
    constexpr int GROUP_M = 4;
    const int per_group = GROUP_M * tiles_n;
    const int group = q / per_group;
    const int first_m = group * GROUP_M;
    const int gm = (tiles_m - first_m) < GROUP_M ? (tiles_m - first_m) : GROUP_M;
    const int r = q - group * per_group;
    tm = first_m + r % gm;
    tn = r / gm;
}
__device__ __forceinline__ void map_workgroup(int tiles_m, int tiles_n, int& split, int& tm, int& tn)
{
    map_workgroup((int)gridDim.x, (int)blockIdx.x, tiles_m, tiles_n, split, tm, tn);
}

}  // namespace
}  // namespace pex
