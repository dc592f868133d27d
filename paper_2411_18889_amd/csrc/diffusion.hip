// One explicit step of the 3-D diffusion equation (section "3D diffusion
// equation"): every point of an nx x ny x nz FP32 grid (k fastest) becomes
//   cc f + ce f(i+1) + cw f(i-1) + cn f(j+1) + cs f(j-1) + ct f(k+1) + cb f(k-1)
// with neighbours outside the grid replaced by the nearest point inside, in
// the listing's order (left to right, contracted into one multiply and six
// FMAs).
//
// The step moves 8 bytes per point at best (one read, one write) against 13
// flops, so it is bound by memory: HBM where f and fn exceed the 256 MB
// last-level cache, that cache (and, for small grids, latency) below.
//
// A lane owns 4 consecutive k points of R rows and marches along i over a
// slab of CI planes; planes i - 1, i, i + 1 of its points stay in registers,
// plane i + 2 and the two outer rows (j - 1, j + R) of plane i + 1 are already
// loading while plane i is computed. There is no LDS, and a barrier only for
// pace (PACED, large planes): rows above and below come from L1 / L2, where the
// neighbouring lanes' own loads put them, and the k neighbours of a lane's 4
// points from the adjacent lanes (DPP wave shifts).
//
// 16-byte accesses need only 4-byte alignment here, so every nz >= 4 and every
// array alignment takes them: the last lane of a row is shifted back to end at
// the row's end (where nz is no multiple of 4 it repeats, with the same
// values, points its neighbour also writes).
#include "common.h"
#include "diffusion_rows.h"

namespace nb {

namespace {

struct Coef {
    float cc, ce, cw, cn, cs, ct, cb;
};

typedef float v4f __attribute__((ext_vector_type(4), aligned(4)));

struct DiffArgs {
    int nx, ny, nz;
    Coef c;
    const float* f;
    float* fn;
    DiffRows g;
};

__device__ __forceinline__ v4f load4(const float* p) { return *reinterpret_cast<const v4f*>(p); }

// PACED: the workgroup's waves keep to the same plane by a barrier per plane.
template <int R, int TPB, bool PACED>
__global__ __launch_bounds__(TPB) void diffusion_rows_kernel(DiffArgs a) {
    // workgroups are dealt to the 8 XCDs round-robin: give each XCD one
    // contiguous run of the grid, so that rows and planes which neighbouring
    // workgroups share are read into one L2 (256^3: 25.4 -> 22.7 us, 512^3
    // 218 -> 203 us)
    const int per = (a.g.blocks + 7) / 8;
    const int b = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (b >= a.g.blocks) return;
    const int slab = b / a.g.chunks;
    int t = (b - slab * a.g.chunks) * TPB + threadIdx.x;
    const bool in = t < a.g.lanes;
    if (!PACED && !in) return;
    if (PACED) t = min(t, a.g.lanes - 1);  // (every wave comes to the barriers)

    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const Coef c = a.c;
    const int jb = t / a.g.row_lanes;
    const int j0 = jb * R;
    const DiffLane d = diff_lane(t - jb * a.g.row_lanes, nz, threadIdx.x & 63);
    const int k0 = d.k0;
    const int64_t plane = (int64_t)ny * nz;
    const int i0 = slab * a.g.ci, i1 = min(i0 + a.g.ci, nx);
    int off[R + 2];  // rows j0 - 1 .. j0 + R, clamped into the grid
#pragma unroll
    for (int r = 0; r < R + 2; ++r) off[r] = min(max(j0 - 1 + r, 0), ny - 1) * nz + k0;

    v4f prev[R], cur[R], next[R];
    float el[R], er[R];
    const float* p = a.f + (int64_t)i0 * plane;
    const float* pm = a.f + (int64_t)max(i0 - 1, 0) * plane;
    const float* pn = a.f + (int64_t)min(i0 + 1, nx - 1) * plane;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        prev[r] = load4(pm + off[r + 1]);
        cur[r] = load4(p + off[r + 1]);
        next[r] = load4(pn + off[r + 1]);
        el[r] = d.left ? p[off[r + 1] - 1] : 0.f;
        er[r] = d.right ? p[off[r + 1] + 4] : 0.f;
    }
    v4f jm = load4(p + off[0]), jp = load4(p + off[R + 1]);
    for (int i = i0; i < i1; ++i) {
        const float* p1 = a.f + (int64_t)min(i + 1, nx - 1) * plane;
        const float* p2 = a.f + (int64_t)min(i + 2, nx - 1) * plane;
        v4f after[R];
        float eln[R], ern[R];
#pragma unroll
        for (int r = 0; r < R; ++r) after[r] = load4(p2 + off[r + 1]);
        const v4f jmn = load4(p1 + off[0]), jpn = load4(p1 + off[R + 1]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            eln[r] = d.left ? p1[off[r + 1] - 1] : 0.f;
            ern[r] = d.right ? p1[off[r + 1] + 4] : 0.f;
        }
        if (PACED) __builtin_amdgcn_s_barrier();
        float* o = a.fn + (int64_t)i * plane;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float km = __int_as_float(__builtin_amdgcn_update_dpp(
                0, __float_as_int(cur[r].w), 0x138, 0xF, 0xF, false));  // lane - 1
            float kp = __int_as_float(__builtin_amdgcn_update_dpp(
                0, __float_as_int(cur[r].x), 0x130, 0xF, 0xF, false));  // lane + 1
            // the ends of the grid have themselves as neighbours
            km = d.first ? cur[r].x : (d.left ? el[r] : km);
            kp = d.last ? cur[r].w : (d.right ? er[r] : kp);
            const v4f up = r < R - 1 ? cur[r < R - 1 ? r + 1 : r] : jp;
            const v4f dn = r > 0 ? cur[r > 0 ? r - 1 : 0] : jm;
            v4f q;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float kpe = e < 3 ? cur[r][e < 3 ? e + 1 : 3] : kp;
                const float kme = e > 0 ? cur[r][e > 0 ? e - 1 : 0] : km;
                float s = c.cc * cur[r][e];
                s = __builtin_fmaf(c.ce, next[r][e], s);
                s = __builtin_fmaf(c.cw, prev[r][e], s);
                s = __builtin_fmaf(c.cn, up[e], s);
                s = __builtin_fmaf(c.cs, dn[e], s);
                s = __builtin_fmaf(c.ct, kpe, s);
                q[e] = __builtin_fmaf(c.cb, kme, s);
            }
            // streaming store: fn is not read again by this step
            if ((!PACED || in) && j0 + r < ny)
                __builtin_nontemporal_store(q, reinterpret_cast<v4f*>(o + off[r + 1]));
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            prev[r] = cur[r];
            cur[r] = next[r];
            next[r] = after[r];
            el[r] = eln[r];
            er[r] = ern[r];
        }
        jm = jmn;
        jp = jpn;
    }
}

// Rows shorter than one 16-byte access (nz < 4): a thread per point.
constexpr int TPB = kDiffLanes;
__global__ __launch_bounds__(TPB) void diffusion_point_kernel(int nx, int ny, int nz, Coef c,
                                                              const float* __restrict__ f,
                                                              float* __restrict__ fn) {
    const int64_t t = blockIdx.x * (int64_t)TPB + threadIdx.x;
    const int64_t row = t / nz;
    const int k = (int)(t - row * nz);
    const int i = (int)(row / ny), j = (int)(row - (int64_t)i * ny);
    if (i >= nx) return;
    const int64_t plane = (int64_t)ny * nz;
    float s = c.cc * f[t];
    s = __builtin_fmaf(c.ce, f[i + 1 < nx ? t + plane : t], s);
    s = __builtin_fmaf(c.cw, f[i > 0 ? t - plane : t], s);
    s = __builtin_fmaf(c.cn, f[j + 1 < ny ? t + nz : t], s);
    s = __builtin_fmaf(c.cs, f[j > 0 ? t - nz : t], s);
    s = __builtin_fmaf(c.ct, f[k + 1 < nz ? t + 1 : t], s);
    fn[t] = __builtin_fmaf(c.cb, f[k > 0 ? t - 1 : t], s);
}

template <int R, int WG, bool PACED>
hipError_t launch_rows(DiffArgs a, int64_t ci, hipStream_t stream) {
    a.g = diff_rows(a.nx, a.ny, a.nz, R, ci, WG);
    hipLaunchKernelGGL((diffusion_rows_kernel<R, WG, PACED>),
                       dim3((unsigned)((a.g.blocks + 7) / 8 * 8)), dim3(WG), 0, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_diffusion3d(int64_t nx, int64_t ny, int64_t nz, double dx, double dy, double dz,
                              double dt, double kappa, const float* f, float* fn, hipStream_t stream) {
    Coef c;
    const double ce = kappa * dt / (dx * dx), cn = kappa * dt / (dy * dy), ct = kappa * dt / (dz * dz);
    c.ce = c.cw = float(ce);
    c.cn = c.cs = float(cn);
    c.ct = c.cb = float(ct);
    c.cc = float(1.0 - 2.0 * (ce + cn + ct));
    if (nz < 4) {
        hipLaunchKernelGGL(diffusion_point_kernel, dim3((unsigned)((nx * ny * nz + TPB - 1) / TPB)),
                           dim3(TPB), 0, stream, (int)nx, (int)ny, (int)nz, c, f, fn);
        return hipGetLastError();
    }
    DiffArgs a{};
    a.nx = (int)nx;
    a.ny = (int)ny;
    a.nz = (int)nz;
    a.c = c;
    a.f = f;
    a.fn = fn;
    // Rows per lane and planes per slab, measured on MI355X (us per step):
    //  * beyond the last-level cache (f and fn together over 256 MB) four rows
    //    per lane, which asks the L2 for 1.5 rows per row computed instead of
    //    3, in slabs of 8 planes: 384^3 93.5 against 98.8 with one row, 512^3
    //    201.9 against 245, 700 x 430 x 444 242.9 against 269 (slabs of 64:
    //    126, 203, 289). The former 256 x 16 LDS tile with a barrier per plane
    //    and slabs of 64: 148, 204, 318;
    //  * of those, planes of which three do not fit an XCD's 4 MB L2: 16 waves a
    //    workgroup that keep to the same plane, so that the rows its waves share
    //    are read once (unpaced, with 256 lanes, and the former kernel: 700^3
    //    574, 606, 606; 1000^3 1573, 1773, 1671; 1200^3 2714, 3213, 2800;
    //    300 x 640 x 640 180, 195, 250; but 512^3 200, 196, 196);
    //  * within it one row per lane (52 VGPRs against 126: more loads in
    //    flight), 256^3 21.8 against 23.0, 150 x 175 x 201 9.9 against 12.9;
    //    slabs of 16 planes, thinner where that would leave the chip short of
    //    lanes: about 3 waves per SIMD are enough (150 x 175 x 201: 8 planes
    //    9.9, 16 12.6; 128^3: 2 planes 5.0, 4 5.3, 16 13.4; 64^3: one plane
    //    2.8, 16 10.2; former kernel: 79, 42, 67, 63).
    const int64_t points = nx * ny * nz;
    if (2 * points * (int64_t)sizeof(float) > (int64_t(256) << 20)) {
        if (3 * ny * nz * (int64_t)sizeof(float) > (int64_t(4) << 20))
            return launch_rows<4, kPacedLanes, true>(a, paced_planes(nx, ny, nz, 4), stream);
        return launch_rows<4, kDiffLanes, false>(a, 8, stream);
    }
    const int64_t work = (nz + 3) / 4 * ny * nx;  // lanes times planes
    return launch_rows<1, kDiffLanes, false>(a, std::min<int64_t>(16, std::max<int64_t>(1, work / 196608)), stream);
}

}  // namespace nb
