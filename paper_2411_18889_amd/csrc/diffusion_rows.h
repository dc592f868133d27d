// How the diffusion step deals a grid's rows to lanes and workgroups (host
// and device side of diffusion_rows_kernel).
//
// A grid has up to 2^31 - 1 points, so a row length or an offset may be any
// int: sums that can pass it are formed in 64 bits or as differences.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace nb {

constexpr int kDiffLanes = 256;   // threads per workgroup
constexpr int kPacedLanes = 1024;  // of the paced one

struct DiffRows {
    int ci;              // planes per slab
    int row_lanes;       // lanes per row, 4 points each
    int lanes;           // lanes per plane, R rows each
    int chunks, blocks;  // workgroups per slab, in all
};

// Rows of nz >= 4 points, R per lane, in slabs of ci planes, `wg` lanes per
// workgroup.
inline DiffRows diff_rows(int64_t nx, int64_t ny, int64_t nz, int R, int64_t ci,
                          int wg = kDiffLanes) {
    DiffRows d;
    d.ci = (int)ci;
    const int64_t row_lanes = (nz + 3) / 4, lanes = row_lanes * ((ny + R - 1) / R);
    const int64_t chunks = (lanes + wg - 1) / wg;
    d.row_lanes = (int)row_lanes;
    d.lanes = (int)lanes;
    d.chunks = (int)chunks;
    d.blocks = (int)(chunks * ((nx + ci - 1) / ci));
    return d;
}

// Planes per slab of the paced workgroups, of which a CU holds one: the fewest
// planes marched in all rounds of the chip's 256 CUs, a slab's start counted as
// four (the two planes that it reads again and the way of the first loads).
// 1000^3: slabs of 64 1573 us, of 8 1666; 100 x 3000 x 3000: of 16 1530, of 64
// 1661; 64 x 1500 x 1500: of 8 251, of 32 302.
inline int64_t paced_planes(int64_t nx, int64_t ny, int64_t nz, int R) {
    int64_t best = 8, least = INT64_MAX;
    for (int64_t ci : {8, 16, 32, 64}) {
        const int64_t blocks = diff_rows(nx, ny, nz, R, ci, kPacedLanes).blocks;
        const int64_t planes = (blocks + 255) / 256 * (std::min(ci, nx) + 4);
        if (planes < least) {
            least = planes;
            best = ci;
        }
    }
    return best;
}

// The 4 points of lane l of a row: the first of them, whether the row starts
// and ends with them, and whether the point before and after them is not at
// the end of the adjacent lane's 4, so that it has to be loaded (wave_lane:
// the lane's number in its wave).
struct DiffLane {
    int k0;
    bool first, last, left, right;
};
__host__ __device__ inline DiffLane diff_lane(int l, int nz, int wave_lane) {
    DiffLane d;
    d.k0 = 4 * l < nz - 4 ? 4 * l : nz - 4;
    d.first = d.k0 == 0;
    d.last = d.k0 == nz - 4;
    d.left = !d.first && (wave_lane == 0 || d.k0 != 4 * l);
    d.right = !d.last && (wave_lane == 63 || nz - d.k0 < 8);
    return d;
}

}  // namespace nb
