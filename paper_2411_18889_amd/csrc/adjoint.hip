// Fused adjoint pair kernel for the reverse KDK walk on gfx950.
//
// For sinks k at positions x (all particles are both sinks and sources) and
// an adjoint vector lam (the velocity adjoint), one pass over all pairs
// computes, with d = r_j - r_k, s = |d|^2 + eps^2, T(d) = s^-3/2 I
// - 3 s^-5/2 d d^T (the derivative of d s^-3/2, symmetric and even in d):
//   a_k        = G sum_j m_j d s^-3/2                      (Eq. (1))
//   (J^T lam)_k = G sum_j T(d) (m_k lam_j - m_j lam_k)      (position adjoint)
//   (G^T lam)_k = -G sum_j (lam_j . d) s^-3/2               (mass adjoint)
// The j = k term is zero in all three (d = 0 and m_k lam_k - m_k lam_k = 0).
// The first is needed to walk the state back one step and comes almost
// free: it shares d, s and the reciprocal square root. A pass that does not
// walk the state back (the entry pass, a state reloaded from a checkpoint)
// leaves it out: 6 % (FP64) to 20 % (mixed, FP64 sums) faster at 262144.
//
// Per pair, with u = m_k lam_j - m_j lam_k and e = -3 s^-1 (d . u):
//   T(d) u = s^-3/2 (u + e d)
// i.e. 6 operations for u, 3 for d.u, 2 for e, 3 FMAs for u + e d and 3 for
// the sum; plus 4 for the mass adjoint and the 12 + rsqrt of the force:
// 34 VALU + 1 rsqrt.
//
// Tiling, j-split, the origin of the pair arithmetic in the mixed policies
// and the fixed-order split reduction are as in the force kernel, and so is
// the kernel with the sources on the lanes for the smallest sets
// (adjoint_lanes_kernel); the LDS record of a source is (x, y, z, m) and
// (lam_x, lam_y, lam_z, 0).
#include <algorithm>

#include "common.h"

namespace nb {

namespace {

constexpr int NQ = 7;  // partials per sink: a (3), J^T lam (3), G^T lam (1)

template <class Pol>
struct AdjArgs {
    using pos_t = typename Pol::pos_t;
    using mass_t = typename Pol::mass_t;
    using calc_t = typename Pol::calc_t;
    const pos_t *x, *y, *z;
    const mass_t* m;
    const pos_t *lx, *ly, *lz;  // lam_v (read only)
    int n;
    int jspan;
    calc_t eps2;
    double G;
    double c;      // weight of the position / mass adjoint update
    double h;      // half step, for the velocity walk-back
    int update_state;
    pos_t *ax, *ay, *az;   // acceleration out (update_state)
    pos_t *vx, *vy, *vz;   // velocity in/out (update_state)
    pos_t *gx, *gy, *gz;   // lam_x in/out
    double* gm;            // lam_m in/out
    WalkArgs<pos_t> next;  // next.x == nullptr: nothing
    double* part;          // [nsplit][NQ][n] or nullptr
};

// NEXT: also enter the walk's next step (the reduction; the pair kernel would
// pay for it in registers).
template <class Pol, bool NEXT>
__device__ __forceinline__ void finish_adj(const AdjArgs<Pol>& a, int i, const double q[NQ]) {
    using pos_t = typename Pol::pos_t;
    const double G = a.G, c = a.c;
    const pos_t gx = pos_t(double(a.gx[i]) + c * (G * q[3]));
    const pos_t gy = pos_t(double(a.gy[i]) + c * (G * q[4]));
    const pos_t gz = pos_t(double(a.gz[i]) + c * (G * q[5]));
    a.gx[i] = gx;
    a.gy[i] = gy;
    a.gz[i] = gz;
    a.gm[i] = a.gm[i] + c * (-G * q[6]);
    if (a.update_state) {
        const pos_t ax = pos_t(G * q[0]), ay = pos_t(G * q[1]), az = pos_t(G * q[2]);
        const pos_t h = pos_t(a.h);
        a.ax[i] = ax;
        a.ay[i] = ay;
        a.az[i] = az;
        a.vx[i] = fmat(-h, ax, a.vx[i]);
        a.vy[i] = fmat(-h, ay, a.vy[i]);
        a.vz[i] = fmat(-h, az, a.vz[i]);
    }
    if (NEXT && a.next.x) {
        const size_t n = a.n, n3 = 3 * n;
        const pos_t h = pos_t(a.h);
        a.next.apply(i, n3, h, gx, a.vx, a.ax);
        a.next.apply(n + i, n3, h, gy, a.vx, a.ax);
        a.next.apply(2 * n + i, n3, h, gz, a.vx, a.ax);
    }
}

// F: also sum the force a (quantities 0..2, for a pass that walks the state
// back); without it they stay 0 and the pair body is 4 operations shorter.
// FEW: built for few waves in flight (kFewWaves): tile-compensated entry pass
// 36.5 -> 25.3 us at 2500 particles, 38.4 -> 33.0 at 5003 (at 10000 88 against
// 85, so not there); with Kahan sums from half as many waves down, and with the
// force sums too up to one wave per SIMD (walked-back step 87 -> 70 at 5003,
// but 91 -> 99 at 6000, 128 -> 146 at 9377).
template <class Pol, int BS, int K, bool F, bool FEW>
__global__ __launch_bounds__(BS) NB_WAVES_PER_EU(FEW) void adjoint_kernel(AdjArgs<Pol> a) {
    using calc_t = typename Pol::calc_t;
    using sum_t = typename Pol::sum_t;
    using V4 = typename Vec4<calc_t>::type;
    __shared__ V4 tp[BS];
    __shared__ V4 tl[BS];

    const int tid = threadIdx.x;
    const int b0 = blockIdx.x * (BS * K);
    const int i0 = b0 + tid;
    // origin of the pair arithmetic (mixed policies): the centroid of this
    // workgroup's sinks
    double ox = 0.0, oy = 0.0, oz = 0.0;
    if constexpr (Pol::origin) {
        __shared__ double org[BS / 64][3];
        double cx = 0.0, cy = 0.0, cz = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int i = i0 + k * BS;
            if (i < a.n) {
                cx += a.x[i];
                cy += a.y[i];
                cz += a.z[i];
            }
        }
        sink_block_origin<BS / 64>(cx, cy, cz, min(a.n - b0, BS * K), org, ox, oy, oz);
    }
    calc_t xi[K], yi[K], zi[K], mi[K], lxi[K], lyi[K], lzi[K];
    sum_t s[K][NQ];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = i0 + k * BS;
        const bool ok = i < a.n;
        xi[k] = ok ? pair_coord<Pol>(a.x[i], ox) : calc_t(0);
        yi[k] = ok ? pair_coord<Pol>(a.y[i], oy) : calc_t(0);
        zi[k] = ok ? pair_coord<Pol>(a.z[i], oz) : calc_t(0);
        mi[k] = ok ? calc_t(a.m[i]) : calc_t(0);
        lxi[k] = ok ? calc_t(a.lx[i]) : calc_t(0);
        lyi[k] = ok ? calc_t(a.ly[i]) : calc_t(0);
        lzi[k] = ok ? calc_t(a.lz[i]) : calc_t(0);
#pragma unroll
        for (int q = 0; q < NQ; ++q) s[k][q].init();
    }
    const calc_t eps2 = a.eps2;
    const int jbeg = blockIdx.y * a.jspan;
    const int jend = min(a.n, jbeg + a.jspan);

    for (int jt = jbeg; jt < jend; jt += BS) {
        const int j = jt + tid;
        V4 p, l;
        if (j < jend) {
            p.x = pair_coord<Pol>(a.x[j], ox);
            p.y = pair_coord<Pol>(a.y[j], oy);
            p.z = pair_coord<Pol>(a.z[j], oz);
            p.w = calc_t(a.m[j]);
            l.x = calc_t(a.lx[j]); l.y = calc_t(a.ly[j]); l.z = calc_t(a.lz[j]); l.w = calc_t(0);
        } else {  // zero mass and zero adjoint: contributes exactly 0
            p.x = p.y = p.z = p.w = calc_t(0);
            l.x = l.y = l.z = l.w = calc_t(0);
        }
        __syncthreads();
        tp[tid] = p;
        tl[tid] = l;
        __syncthreads();
#pragma unroll 4
        for (int jj = 0; jj < BS; ++jj) {
            const V4 q = tp[jj];
            const V4 lj = tl[jj];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const calc_t dx = q.x - xi[k];
                const calc_t dy = q.y - yi[k];
                const calc_t dz = q.z - zi[k];
                const calc_t ss = fmat(dz, dz, fmat(dy, dy, fmat(dx, dx, eps2)));
                const calc_t r = rsqrt_pair(ss);
                const calc_t r2 = r * r;
                const calc_t r3 = r2 * r;
                if (F) {  // force
                    const calc_t w = r3 * q.w;
                    s[k][0].add_fma(dx, w);
                    s[k][1].add_fma(dy, w);
                    s[k][2].add_fma(dz, w);
                }
                // position adjoint: T(d) u = r3 (u + e d), e = -3 r2 (d . u)
                const calc_t ux = fmat(mi[k], lj.x, -(q.w * lxi[k]));
                const calc_t uy = fmat(mi[k], lj.y, -(q.w * lyi[k]));
                const calc_t uz = fmat(mi[k], lj.z, -(q.w * lzi[k]));
                const calc_t du = fmat(dz, uz, fmat(dy, uy, dx * ux));
                const calc_t e = (calc_t(-3) * r2) * du;
                s[k][3].add_fma(r3, fmat(e, dx, ux));
                s[k][4].add_fma(r3, fmat(e, dy, uy));
                s[k][5].add_fma(r3, fmat(e, dz, uz));
                // mass adjoint (sign applied at the end)
                const calc_t dl = fmat(dz, lj.z, fmat(dy, lj.y, dx * lj.x));
                s[k][6].add_fma(r3, dl);
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int q = 0; q < NQ; ++q) s[k][q].tile_end();
    }

#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = i0 + k * BS;
        if (i >= a.n) continue;
        if (a.part) {
            double* out = a.part + (size_t)blockIdx.y * NQ * a.n;
#pragma unroll
            for (int q = F ? 0 : 3; q < NQ; ++q) out[(size_t)q * a.n + i] = s[k][q].total();
        } else {
            double t[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) t[q] = s[k][q].total();
            finish_adj<Pol, false>(a, i, t);
        }
    }
}

// Sources on the lanes, as the force pass's force_lanes_kernel (which has the
// reasons): LB lanes, LS sinks per workgroup, every lane with every LB-th
// source; the lanes' sums meet in LDS and the workgroup finishes its sinks. The
// walk's next step is entered by a kernel of its own, since other workgroups
// still read x and lam_v. org_block: sinks per origin block (the one-sided
// kernel's workgroups). Four sinks, two for FP32 with the force sums (4001
// particles, us: FP64 25 with four, 31 with two; FP32 with the force sums 23
// and 21).
constexpr int LB = 256;
template <class Pol, bool F>
constexpr int lane_sinks = std::is_same<Pol, PolF32>::value && F ? 2 : 4;

template <class Pol, bool F>
__global__ __launch_bounds__(LB) void adjoint_lanes_kernel(AdjArgs<Pol> a, int org_block) {
    using calc_t = typename Pol::calc_t;
    using sum_t = typename Pol::sum_t;
    constexpr int LS = lane_sinks<Pol, F>;
    constexpr int Q0 = F ? 0 : 3, N = NQ - Q0, V = LS * N;
    __shared__ double lsum[V][LB + 1];
    __shared__ double tot[LS][N];
    const int tid = threadIdx.x;
    const int i0 = blockIdx.x * LS;
    double ox = 0.0, oy = 0.0, oz = 0.0;
    if constexpr (Pol::origin) {
        __shared__ double org[LB / 64][3];
        const int b0 = i0 / org_block * org_block, i = b0 + tid;
        const bool ok = tid < org_block && i < a.n;
        sink_block_origin<LB / 64>(ok ? a.x[i] : 0.0, ok ? a.y[i] : 0.0, ok ? a.z[i] : 0.0,
                                   min(a.n - b0, org_block), org, ox, oy, oz);
    }
    calc_t xi[LS], yi[LS], zi[LS], mi[LS], lxi[LS], lyi[LS], lzi[LS];
    sum_t s[LS][NQ];
#pragma unroll
    for (int k = 0; k < LS; ++k) {
        const int i = min(i0 + k, a.n - 1);
        xi[k] = pair_coord<Pol>(a.x[i], ox);
        yi[k] = pair_coord<Pol>(a.y[i], oy);
        zi[k] = pair_coord<Pol>(a.z[i], oz);
        mi[k] = calc_t(a.m[i]);
        lxi[k] = calc_t(a.lx[i]);
        lyi[k] = calc_t(a.ly[i]);
        lzi[k] = calc_t(a.lz[i]);
#pragma unroll
        for (int q = 0; q < NQ; ++q) s[k][q].init();
    }
#pragma unroll 2
    for (int j = tid; j < a.n; j += LB) {
        const calc_t x = pair_coord<Pol>(a.x[j], ox), y = pair_coord<Pol>(a.y[j], oy),
                     z = pair_coord<Pol>(a.z[j], oz), m = calc_t(a.m[j]);
        const calc_t lx = calc_t(a.lx[j]), ly = calc_t(a.ly[j]), lz = calc_t(a.lz[j]);
#pragma unroll
        for (int k = 0; k < LS; ++k) {
            const calc_t dx = x - xi[k], dy = y - yi[k], dz = z - zi[k];
            const calc_t ss = fmat(dz, dz, fmat(dy, dy, fmat(dx, dx, a.eps2)));
            const calc_t r = rsqrt_pair(ss);
            const calc_t r2 = r * r;
            const calc_t r3 = r2 * r;
            if (F) {
                const calc_t w = r3 * m;
                s[k][0].add_fma(dx, w);
                s[k][1].add_fma(dy, w);
                s[k][2].add_fma(dz, w);
            }
            const calc_t ux = fmat(mi[k], lx, -(m * lxi[k]));
            const calc_t uy = fmat(mi[k], ly, -(m * lyi[k]));
            const calc_t uz = fmat(mi[k], lz, -(m * lzi[k]));
            const calc_t e = (calc_t(-3) * r2) * fmat(dz, uz, fmat(dy, uy, dx * ux));
            s[k][3].add_fma(r3, fmat(e, dx, ux));
            s[k][4].add_fma(r3, fmat(e, dy, uy));
            s[k][5].add_fma(r3, fmat(e, dz, uz));
            s[k][6].add_fma(r3, fmat(dz, lz, fmat(dy, ly, dx * lx)));
        }
    }
#pragma unroll
    for (int k = 0; k < LS; ++k)
#pragma unroll
        for (int q = 0; q < N; ++q) lsum[k * N + q][tid] = s[k][Q0 + q].total();
    __syncthreads();
    const int l = tid & 15;
    for (int v = tid >> 4; v < V; v += LB / 16) {  // 16 lanes add sum v
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < LB / 16; ++q) t += lsum[v][q * 16 + l];
#pragma unroll
        for (int mask = 8; mask >= 1; mask >>= 1) t += __shfl_xor(t, mask, 64);
        if (l == 0) tot[v / N][v % N] = t;
    }
    __syncthreads();
    if (tid < LS && i0 + tid < a.n) {
        double t[NQ] = {0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < N; ++q) t[Q0 + q] = tot[tid][q];
        finish_adj<Pol, false>(a, i0 + tid, t);
    }
}

// The partial sums in the fixed order of the force pass's reduction: wave g of
// a workgroup takes ranges g, g + 4, ... of 64 sinks, the first wave adds the
// four sums and finishes. F as the pair kernel's.
template <class Pol, bool F>
__global__ __launch_bounds__(256) void adjoint_reduce_kernel(AdjArgs<Pol> a, int nsplit) {
    constexpr int Q0 = F ? 0 : 3;
    __shared__ double other[3][NQ][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int i = reduce_first_sink() + lane;
    double t[NQ] = {0, 0, 0, 0, 0, 0, 0};
    if (i < a.n) {
        for (int r0 = g; r0 < nsplit; r0 += 4 * 4) {  // four ranges' loads in flight
            double p[4][NQ];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int r = r0 + 4 * u;
                const double* q = a.part + (size_t)r * NQ * a.n + i;
#pragma unroll
                for (int c = Q0; c < NQ; ++c) p[u][c] = r < nsplit ? q[(size_t)c * a.n] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int c = Q0; c < NQ; ++c) t[c] += p[u][c];
        }
    }
    if (g)
#pragma unroll
        for (int c = Q0; c < NQ; ++c) other[g - 1][c][lane] = t[c];
    __syncthreads();
    if (g || i >= a.n) return;
#pragma unroll
    for (int v = 0; v < 3; ++v)
#pragma unroll
        for (int c = Q0; c < NQ; ++c) t[c] += other[v][c][lane];
    finish_adj<Pol, true>(a, i, t);
}

template <class Pol, int BS, int K>
hipError_t launch_shape(AdjArgs<Pol> a, int nsplit, hipStream_t stream) {
    dim3 grid((a.n + BS * K - 1) / (BS * K), nsplit);
    auto launch = [&](auto few) {
        constexpr bool FEW = decltype(few)::value;
        if (a.update_state)
            hipLaunchKernelGGL((adjoint_kernel<Pol, BS, K, true, FEW>), grid, dim3(BS), 0, stream, a);
        else
            hipLaunchKernelGGL((adjoint_kernel<Pol, BS, K, false, FEW>), grid, dim3(BS), 0, stream, a);
        return hipGetLastError();
    };
    constexpr bool kahan = std::is_same<typename Pol::sum_t, SumKahan>::value;
    if constexpr (K == 1 && (kahan || std::is_same<typename Pol::sum_t, SumTile>::value)) {
        const int64_t waves = (int64_t)grid.x * nsplit * (BS / 64);
        const int64_t most = !kahan ? kFewWaves : a.update_state ? kFewWaves / 4 + 1 : kFewWaves / 2;
        if (waves < most) return launch(std::true_type{});
    }
    return launch(std::false_type{});
}

template <class Pol>
hipError_t launch_any(const Shape& sh, AdjArgs<Pol> a, int nsplit, hipStream_t stream) {
#define NB_ADJ_CASE(BSV, KV) \
    if (sh.block == BSV && sh.ipl == KV) return launch_shape<Pol, BSV, KV>(a, nsplit, stream);
    NB_ADJ_CASE(64, 1) NB_ADJ_CASE(64, 2)
    NB_ADJ_CASE(128, 1) NB_ADJ_CASE(128, 2)
    NB_ADJ_CASE(256, 1) NB_ADJ_CASE(256, 2)
    NB_ADJ_CASE(512, 1) NB_ADJ_CASE(512, 2)
#undef NB_ADJ_CASE
    return hipErrorInvalidValue;
}

}  // namespace

Shape choose_adjoint_shape(int prec, int64_t n, Pick pick) {
    // Sources on the lanes, for the policies whose sums may be regrouped: us
    // per entry pass and per walked-back step against the split ranges below,
    // measured on MI355X,
    //            2000              4001              6000              12287
    //   FP64     15, 17 / 19, 24   25, 32 / 42, 38   52, 61 / 67, 77   201, 223 / 210, 229
    //   FP32     15, 18 / 18, 21   16, 21 / 26, 31   29, 38 / 44, 53   103, 132 / 116, 135
    //   acc64    17, 23 / 17, 25   27, 34 / 29, 48   52, 61 / 52, 67   172, 195 / 142, 183
    // so up to 6000 particles for FP64 sums of FP32 terms.
    const bool regroup = prec == NB_F64 || prec == NB_F32 || prec == NB_MIX_ACC64;
    if (pick == Pick::Best && regroup && n <= (prec == NB_MIX_ACC64 ? 6000 : 12287)) {
        Shape s{4, LB, LB};
        s.lanes = true;
        return s;
    }
    // Measured on MI355X: one sink per lane (the fused pair body is long
    // enough to hide latency on its own; two sinks per lane run 13 % slower),
    // 512-lane workgroups from 2^19 sinks up, 256 from 4096, 64 below; a
    // source split up to ~128K wavefronts (8 ranges at 2^20), every range
    // >= 2 tiles long (4 below 32768 sinks) -- or, below 16384 sinks, as
    // short as one tile up to 32 ranges (2.2-2.8x faster at N = 1024 and
    // 2048, where the pass is otherwise a handful of workgroups).
    Shape s{1, n >= (1 << 19) ? 512 : (n <= 2048 ? 64 : 256), 1};
    const int64_t waves = (n + s.block - 1) / s.block * (s.block / 64);
    const int64_t want = 131072;
    int64_t split = (want + waves - 1) / waves;
    const int64_t long_ranges = n / ((n < 32768 ? 4 : 2) * (int64_t)s.block);
    const int64_t short_ranges = n < 16384 ? std::min<int64_t>(32, n / (int64_t)s.block) : 0;
    const int64_t max_ranges = std::max(long_ranges, short_ranges);
    if (split > max_ranges) split = max_ranges;
    if (split > 256) split = 256;
    if (split < 1) split = 1;
    // ranges as short as one tile until there are 8 waves per SIMD, as the
    // force pass (and not for the same two policies): entry pass 37.0 instead
    // of 56.9 us at 2500 particles, 39.1 instead of 59.6 at 5003, 84.9
    // instead of 96.5 at 10000
    if (pick != Pick::Least && prec != NB_MIX_ACC32 && prec != NB_MIX_KAHAN)
        split = std::max<int64_t>(split_ranges(n, split, s.block),
                                  short_tile_ranges(n, s.block, waves, 8192));
    s.split = (int)split;
    return s;
}

bool adjoint_shape_supported(const Shape& s) {
    const bool bs_ok = s.block == 64 || s.block == 128 || s.block == 256 || s.block == 512;
    return bs_ok && (s.ipl == 1 || s.ipl == 2) && s.split >= 1 && s.split <= 256;
}

size_t adjoint_partials_bytes(const Shape& s, int64_t n) {
    if (s.lanes) return 0;
    return (size_t)s.split * NQ * (size_t)n * sizeof(double);
}

hipError_t launch_adjoint(int prec, const Shape& sh, int64_t n, const void* x, const void* m,
                          const void* lam_v, double eps, double G, double c, bool update_state,
                          double h, void* acc, void* v, void* lam_x, double* lam_m, void* ws,
                          hipStream_t stream, const WalkNext& next, bool* entered) {
    hipError_t err = hipErrorInvalidValue;
    if (entered) *entered = false;
    dispatch_prec(prec, [&](auto tag) {
        using Pol = decltype(tag);
        using pos_t = typename Pol::pos_t;
        using mass_t = typename Pol::mass_t;
        using calc_t = typename Pol::calc_t;
        AdjArgs<Pol> a{};
        const pos_t* px = static_cast<const pos_t*>(x);
        const pos_t* pl = static_cast<const pos_t*>(lam_v);
        a.x = px; a.y = px + n; a.z = px + 2 * n;
        a.m = static_cast<const mass_t*>(m);
        a.lx = pl; a.ly = pl + n; a.lz = pl + 2 * n;
        a.n = (int)n;
        a.eps2 = calc_t(eps) * calc_t(eps);
        a.G = G;
        a.c = c;
        a.h = h;
        a.update_state = update_state ? 1 : 0;
        pos_t* pa = static_cast<pos_t*>(acc);
        pos_t* pv = static_cast<pos_t*>(v);
        pos_t* pg = static_cast<pos_t*>(lam_x);
        a.ax = pa; a.ay = pa + n; a.az = pa + 2 * n;
        a.vx = pv; a.vy = pv + n; a.vz = pv + 2 * n;
        a.gx = pg; a.gy = pg + n; a.gz = pg + 2 * n;
        a.gm = lam_m;
        if (sh.lanes) {
            if constexpr (std::is_same<typename Pol::sum_t, SumKahan>::value ||
                          std::is_same<typename Pol::sum_t, SumTile>::value ||
                          std::is_same<Pol, PolMixAcc32>::value) {
                return;
            } else {
                const int org = choose_adjoint_shape(prec, n, Pick::Least).block;
                auto grid = [&](int sinks) { return dim3((unsigned)((n + sinks - 1) / sinks)); };
                if (update_state)
                    hipLaunchKernelGGL((adjoint_lanes_kernel<Pol, true>), grid(lane_sinks<Pol, true>),
                                       dim3(LB), 0, stream, a, org);
                else
                    hipLaunchKernelGGL((adjoint_lanes_kernel<Pol, false>), grid(lane_sinks<Pol, false>),
                                       dim3(LB), 0, stream, a, org);
                err = hipGetLastError();
                return;
            }
        }
        const int span = split_span(n, sh.split, sh.block);
        const int nsplit = split_ranges(n, sh.split, sh.block);
        a.jspan = span;
        if (nsplit == 1) {  // sinks finish while others still read x and lam_v: no drift
            a.part = nullptr;
            err = launch_any<Pol>(sh, a, 1, stream);
            return;
        }
        a.next = WalkArgs<pos_t>(next, lam_v);
        if (entered) *entered = next.x != nullptr;
        a.part = static_cast<double*>(ws);
        err = launch_any<Pol>(sh, a, nsplit, stream);
        if (err != hipSuccess) return;
        const dim3 grid = reduce_grid(sh, n);
        if (update_state)
            hipLaunchKernelGGL((adjoint_reduce_kernel<Pol, true>), grid, dim3(256), 0, stream, a, nsplit);
        else
            hipLaunchKernelGGL((adjoint_reduce_kernel<Pol, false>), grid, dim3(256), 0, stream, a, nsplit);
        err = hipGetLastError();
    });
    return err;
}

}  // namespace nb
