// Host-side check of how the diffusion step deals rows to lanes
// (csrc/diffusion_rows.h): for row lengths from 4 to the largest the library
// takes (2^31 - 1 points in one row), with the kernel's own functions,
//   * the lanes of a row are ceil(nz / 4), their 4 points lie inside it, meet
//     without a gap and end at its end;
//   * a point before or after a lane's 4 is loaded exactly where it is not the
//     end of the adjacent lane's 4 in the same wave, and then lies inside the
//     row;
//   * lanes, workgroups per slab and workgroups cover the plane and the grid.
// No device is touched. Prints "ok" and exits 0, or names the failure.
#include <cstdio>
#include <cstdlib>

#include "diffusion_rows.h"

using namespace nb;

static int fail(const char* what, long long a, long long b) {
    std::printf("FAIL: %s (%lld, %lld)\n", what, a, b);
    std::exit(1);
}

static void check_row(int64_t nz) {
    const DiffRows g = diff_rows(1, 1, nz, 1, 1);
    if (g.row_lanes != (nz + 3) / 4) fail("lanes of the row", nz, g.row_lanes);
    const int64_t n = g.row_lanes;
    auto lane = [&](int64_t l, int wl) {
        if (l < 0 || l >= n) return;
        const DiffLane d = diff_lane((int)l, (int)nz, wl);
        const int64_t k = d.k0;
        if (k < 0 || k + 4 > nz || k > 4 * l) fail("points outside the row", nz, l);
        if (d.first != (k == 0) || d.last != (k + 4 == nz)) fail("ends of the row", nz, l);
        if (l == 0 && k != 0) fail("start of the row", nz, l);
        if (l == n - 1 && !d.last) fail("end of the row", nz, l);
        // the point before: the previous lane's last, in the lane below of the wave
        if (l > 0) {
            const int64_t prev = diff_lane((int)l - 1, (int)nz, 0).k0;
            if (prev + 4 < k) fail("gap before a lane", nz, l);
            if (!d.first && !d.left && (wl == 0 || prev + 4 != k)) fail("left neighbour", nz, l);
        }
        if (l < n - 1) {
            const int64_t next = diff_lane((int)l + 1, (int)nz, 0).k0;
            if (!d.last && !d.right && (wl == 63 || next != k + 4)) fail("right neighbour", nz, l);
        }
        if (d.left && k < 1) fail("left load outside the row", nz, l);
        if (d.right && k + 4 >= nz) fail("right load outside the row", nz, l);
    };
    for (int wl : {0, 1, 31, 62, 63}) {
        for (int64_t l = 0; l < 70; ++l) lane(l, wl);
        for (int64_t l = n - 70; l < n; ++l) lane(l, wl);
        lane(n / 2, wl);
    }
}

static void check_grid(int64_t nx, int64_t ny, int64_t nz, int R, int64_t ci, int wg) {
    const DiffRows g = diff_rows(nx, ny, nz, R, ci, wg);
    const int64_t lanes = (nz + 3) / 4 * ((ny + R - 1) / R), slabs = (nx + ci - 1) / ci;
    if (g.lanes != lanes) fail("lanes of a plane", g.lanes, lanes);
    if (g.chunks < 1 || (int64_t)g.chunks * wg < lanes ||
        (int64_t)(g.chunks - 1) * wg >= lanes)
        fail("workgroups of a slab", g.chunks, lanes);
    if (g.blocks != g.chunks * slabs) fail("workgroups", g.blocks, slabs);
    if (((int64_t)g.blocks + 7) / 8 * 8 * wg >= (int64_t(1) << 32)) fail("threads", g.blocks, 0);
}

int main() {
    const int64_t top = (int64_t(1) << 31) - 1;  // points of the largest grid
    for (int64_t nz = 4; nz < 1200; ++nz) check_row(nz);
    for (int64_t d = 0; d < 300; ++d) check_row(top - d);
    for (int R : {1, 4})
        for (int64_t ci : {1, 8, 64})
            for (int64_t nz : {int64_t(4), int64_t(5), int64_t(1000), int64_t(46341), top / 3, top - 2, top})
                for (int64_t ny : {int64_t(1), int64_t(2), int64_t(3), int64_t(524280)})
                    for (int64_t nx : {int64_t(1), int64_t(7), int64_t(1) << 21})
                        if (nx * ny <= (int64_t(1) << 31) && nz <= top / (nx * ny))
                            for (int wg : {kDiffLanes, kPacedLanes})
                                check_grid(nx, ny, nz, R, ci, wg);
    std::printf("ok\n");
    return 0;
}
