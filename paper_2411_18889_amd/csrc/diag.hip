// FP64 diagnostics: kinetic, potential and total energy, linear and angular
// momentum, centre of mass and total mass of a state.
//
// Potential energy PE = -G sum_{i<j} m_i m_j / sqrt(|r_j - r_i|^2 + eps^2):
// only the pairs i < j are visited. Sinks are cut into tiles of T = 256 PK
// (PK per lane, in registers), sources into groups of PG = 16; tile I meets
// the groups from its own start on, and these (tile, group) units, tile by
// tile, are cut into equal runs, one per workgroup, so that the chip is
// evenly loaded from a thousand particles on (one workgroup per pair of
// 1024-particle tiles left most of it idle: a call at
// 16384 particles 191 -> 71 us, at 1024 188 -> 15). Groups inside the tile keep j > i only.
// Every workgroup adds its pairs into one FP64 partial; the partials and the
// per-particle terms of KE, P, L and the centre of mass (the first workgroups
// of the same launch) are reduced in a fixed order (fixed runs, fixed trees),
// so the result is bitwise reproducible.
//
// Reciprocal square root: y = v_rsq_f64(s) (about 24 correct bits) and one
// Newton-Raphson step, r = y (3 - s y^2) / 2, which leaves a relative error of
// a few 1e-15 per term. The sum is of 2 m_j r = (m_j y) (3 - s y^2), halved
// once at the end: 10 FP64 operations and the quarter-rate v_rsq_f64 per pair,
// about 60 cycles per 64 pairs and SIMD, which is what bounds the pass.
#include "common.h"

namespace nb {

namespace {

constexpr int TPB = 256;
constexpr int NW = TPB / 64;
constexpr int PG = 16;              // sources per unit
constexpr int CH = 128;             // sources per LDS chunk
constexpr int PE_GRID = 16384;      // room for partials of the potential pass
constexpr int NV = 13;              // output slots; slot 1 (PE) and 2 (E) formed at the end

inline int diag_blocks(int64_t n) {
    int64_t b = (n + TPB - 1) / TPB;
    return (int)(b > 1024 ? 1024 : b);
}

// The lane's value summed over the wave (every lane gets the sum; fixed order).
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int mask = 32; mask >= 1; mask >>= 1) v += __shfl_xor(v, mask, 64);
    return v;
}

struct PePlan {
    int64_t ng;     // groups of PG sources
    int64_t units;  // (tile, group) pairs
    int64_t per;    // units per workgroup
    int wgs;
};

inline PePlan pe_plan(int64_t n, int tile, int64_t target) {
    PePlan p;
    const int64_t gpt = tile / PG, nt = (n + tile - 1) / tile;
    p.ng = (n + PG - 1) / PG;
    p.units = nt * p.ng - gpt * (nt * (nt - 1) / 2);
    p.per = (p.units + target - 1) / target;
    p.wgs = (int)((p.units + p.per - 1) / p.per);
    return p;
}

template <typename P, typename M>
struct DiagArgs {
    const P *x, *v;
    const M* m;
    int64_t n;
    double eps2;
    PePlan pe;
    int nblocks;      // workgroups of the per-particle sums, then pe.wgs of the pairs
    double *pe_part, *blocks;
};

template <typename P, typename M>
__device__ __forceinline__ void particle_sums(const DiagArgs<P, M>& a, double (*lds)[NV]) {
    const P *x = a.x, *v = a.v;
    const int64_t n = a.n;
    double acc[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) acc[q] = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)TPB + threadIdx.x; i < n; i += (int64_t)a.nblocks * TPB) {
        const double mi = double(a.m[i]);
        const double rx = double(x[i]), ry = double(x[n + i]), rz = double(x[2 * n + i]);
        const double vx = double(v[i]), vy = double(v[n + i]), vz = double(v[2 * n + i]);
        acc[0] += 0.5 * mi * (vx * vx + vy * vy + vz * vz);
        acc[3] += mi * vx;
        acc[4] += mi * vy;
        acc[5] += mi * vz;
        acc[6] += mi * (ry * vz - rz * vy);
        acc[7] += mi * (rz * vx - rx * vz);
        acc[8] += mi * (rx * vy - ry * vx);
        acc[9] += mi * rx;
        acc[10] += mi * ry;
        acc[11] += mi * rz;
        acc[12] += mi;
    }
#pragma unroll
    for (int q = 0; q < NV; ++q) acc[q] = wave_sum(acc[q]);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int q = 0; q < NV; ++q) lds[w][q] = acc[q];
    __syncthreads();
    if (threadIdx.x < NV) {
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < NW; ++u) s += lds[u][threadIdx.x];
        a.blocks[(size_t)blockIdx.x * NV + threadIdx.x] = s;
    }
}

template <typename P, typename M, int PK>
__global__ __launch_bounds__(TPB) void diag_kernel(DiagArgs<P, M> a) {
    __shared__ double4 src[CH];
    __shared__ double lds[NW][NV];
    if ((int)blockIdx.x < a.nblocks) {
        particle_sums(a, lds);
        return;
    }
    constexpr int T = TPB * PK;
    constexpr int64_t GPT = T / PG;
    const P *x = a.x, *y = a.x + a.n, *z = a.x + 2 * a.n;
    const int64_t n = a.n, ng = a.pe.ng;
    const int64_t wg = blockIdx.x - a.nblocks;
    int64_t u = wg * a.pe.per;
    const int64_t uend = min(u + a.pe.per, a.pe.units);
    // unit u -> tile I: the units before tile I number before(I)
    auto before = [&](int64_t I) { return I * ng - GPT * (I * (I - 1) / 2); };
    const double half = double(ng) / double(GPT) + 0.5;
    int64_t I = (int64_t)(half - sqrt(max(half * half - 2.0 * double(u) / double(GPT), 0.0)));
    I = max(int64_t(0), min(I, (n - 1) / T));
    while (I > 0 && before(I) > u) --I;
    while (I < (n - 1) / T && before(I + 1) <= u) ++I;

    double total = 0.0;
    for (; u < uend; ++I) {
        const int64_t g0 = I * GPT + (u - before(I));
        const int64_t g1 = min(ng, g0 + (uend - u));
        u += g1 - g0;
        const int i0 = threadIdx.x;
        double xi[PK], yi[PK], zi[PK], acc[PK];
#pragma unroll
        for (int k = 0; k < PK; ++k) {
            const int64_t i = I * T + k * TPB + i0;
            const bool ok = i < n;
            xi[k] = ok ? double(x[i]) : 0.0;
            yi[k] = ok ? double(y[i]) : 0.0;
            zi[k] = ok ? double(z[i]) : 0.0;
            acc[k] = 0.0;
        }
        for (int64_t j0 = g0 * PG; j0 < g1 * PG; j0 += CH) {
            const int cnt = (int)min((int64_t)CH, g1 * PG - j0);  // a multiple of PG
            __syncthreads();  // the previous chunk has been read
            if ((int)threadIdx.x < cnt) {
                const int64_t j = j0 + threadIdx.x;
                double4 r;
                r.x = r.y = r.z = r.w = 0.0;  // zero mass past the end: adds exactly 0
                if (j < n) {
                    r.x = double(x[j]);
                    r.y = double(y[j]);
                    r.z = double(z[j]);
                    r.w = double(a.m[j]);
                }
                src[threadIdx.x] = r;
            }
            __syncthreads();
            if (j0 >= (I + 1) * T) {
#pragma unroll 4
                for (int q = 0; q < cnt; ++q) {
                    const double4 r = src[q];
#pragma unroll
                    for (int k = 0; k < PK; ++k) {
                        const double dx = r.x - xi[k], dy = r.y - yi[k], dz = r.z - zi[k];
                        const double s = fmat(dz, dz, fmat(dy, dy, fmat(dx, dx, a.eps2)));
                        const double t = __builtin_amdgcn_rsq(s);
                        acc[k] = fmat(r.w * t, fmat(-(s * t), t, 3.0), acc[k]);
                    }
                }
            } else {  // sources of the tile itself: only j > i
                const int d = (int)(j0 - I * T);
                for (int q = 0; q < cnt; ++q) {
                    const double4 r = src[q];
#pragma unroll
                    for (int k = 0; k < PK; ++k) {
                        const double dx = r.x - xi[k], dy = r.y - yi[k], dz = r.z - zi[k];
                        const double s = fmat(dz, dz, fmat(dy, dy, fmat(dx, dx, a.eps2)));
                        const double t = __builtin_amdgcn_rsq(s);
                        const double term = (r.w * t) * fmat(-(s * t), t, 3.0);
                        acc[k] += (d + q > k * TPB + i0) ? term : 0.0;
                    }
                }
            }
        }
#pragma unroll
        for (int k = 0; k < PK; ++k) {
            const int64_t i = I * T + k * TPB + i0;
            if (i < n) total = fmat(double(a.m[i]), acc[k], total);
        }
    }
    total = wave_sum(total);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6][0] = total;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += lds[w][0];
        a.pe_part[wg] = 0.5 * s;
    }
}

// One workgroup of 16 waves: wave q adds the blocks' sums of slot q (lane l
// takes blocks l, l + 64, ...); the waves without a slot (1, 2, 13, 14, 15)
// share the potential's partials. Thirteen tree sums in LDS, ten barriers
// each, took 10 us here.
constexpr int FW = 16;
__global__ __launch_bounds__(FW * 64) void diag_final_kernel(const double* __restrict__ blocks,
                                                             int nblocks,
                                                             const double* __restrict__ pe_part,
                                                             int npe, double G,
                                                             double* __restrict__ out) {
    __shared__ double sums[FW];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const bool slot = w == 0 || (w >= 3 && w < NV);
    double acc = 0.0;
    if (slot) {
#pragma unroll 4
        for (int b = lane; b < nblocks; b += 64) acc += blocks[(size_t)b * NV + w];
    } else {
        const int share = w < 3 ? w - 1 : w - 11;  // 0 .. 4
#pragma unroll 8
        for (int b = share * 64 + lane; b < npe; b += 5 * 64) acc += pe_part[b];
    }
    acc = wave_sum(acc);
    if (lane == 0) sums[w] = acc;
    __syncthreads();
    const int q = threadIdx.x;
    if (q >= NV) return;
    const double pe = -G * (sums[1] + sums[2] + sums[13] + sums[14] + sums[15]);
    double r = sums[q];
    if (q == 1) r = pe;
    if (q == 2) r = sums[0] + pe;
    if (q >= 9 && q < 12) r = sums[q] / sums[12];
    out[q] = r;
}

template <typename P, typename M>
hipError_t run_diag(int64_t n, const void* x, const void* v, const void* m, double eps, double G,
                    double* out, void* ws, hipStream_t stream) {
    DiagArgs<P, M> a;
    a.x = static_cast<const P*>(x);
    a.v = static_cast<const P*>(v);
    a.m = static_cast<const M*>(m);
    a.n = n;
    a.eps2 = eps * eps;
    a.nblocks = diag_blocks(n);
    a.pe_part = static_cast<double*>(ws);
    a.blocks = a.pe_part + PE_GRID;
    // Sinks per lane and workgroups of the pair pass, measured on MI355X (us
    // per call): few sinks a lane while the pairs inside a tile (half of them
    // masked) still count -- 32768: 238 with two, 242 with four; 157847: 4881
    // with four, 4964 with two. 4096 runs are short enough to even out the
    // CUs at small n (10007: 33.6, with 16384 runs 39.0; 16384: 71.2, 74.4),
    // more runs balance better above (32768: 244 against 238, 157847: 4950
    // against 4881).
    const bool small = n < 40000;
    a.pe = pe_plan(n, TPB * (small ? 2 : 4), n < 24576 ? 4096 : PE_GRID);
    const dim3 grid((unsigned)(a.nblocks + a.pe.wgs));
    if (small)
        hipLaunchKernelGGL((diag_kernel<P, M, 2>), grid, dim3(TPB), 0, stream, a);
    else
        hipLaunchKernelGGL((diag_kernel<P, M, 4>), grid, dim3(TPB), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(diag_final_kernel, dim3(1), dim3(FW * 64), 0, stream, a.blocks, a.nblocks,
                       a.pe_part, a.pe.wgs, G, out);
    return hipGetLastError();
}

}  // namespace

size_t diag_workspace_bytes(int64_t n) {
    return ((size_t)PE_GRID + (size_t)diag_blocks(n) * NV) * sizeof(double);
}

hipError_t launch_diag(int prec, int64_t n, const void* x, const void* v, const void* m, double eps,
                       double G, double* out, void* ws, hipStream_t stream) {
    if (prec == NB_F32) return run_diag<float, float>(n, x, v, m, eps, G, out, ws, stream);
    if (prec == NB_F64) return run_diag<double, double>(n, x, v, m, eps, G, out, ws, stream);
    return run_diag<double, float>(n, x, v, m, eps, G, out, ws, stream);
}

}  // namespace nb
