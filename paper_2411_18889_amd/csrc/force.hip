// Pair-force kernels of Eq. (1) (section "N-body simulation") for gfx950.
//
// Design (one launch = ni sinks against a range of sources):
//  * a workgroup of BS threads owns BS*K sinks; each lane keeps K sinks in
//    registers (sink k of lane t is i = group*BS*K + k*BS + t, so the SoA
//    loads and stores of a wave are contiguous);
//  * the sources are streamed in j-tiles of BS particles: every lane loads
//    one source from the SoA arrays (coalesced), rounds it to the pair
//    arithmetic type (in the mixed policies relative to the centroid of the
//    workgroup's sinks, see sink_block_origin) and stores it in LDS as
//    (x, y, z, m); after a barrier
//    every lane walks the whole tile, and every LDS read is a broadcast (all
//    lanes read the same address, so no bank conflicts);
//  * per pair: 3 subtractions, 3 FMAs for |d|^2 + eps^2 (eps^2 innermost, as
//    the listing), one reciprocal square root, 3 multiplications for
//    m_j / s^(3/2), 3 FMAs into the sums; no MFMA, since nothing here is a
//    dense contraction;
//  * small N: the source range is split over gridDim.y workgroups (j-split).
//    Each writes its FP64 partial sums to the workspace and a second kernel
//    adds them in a fixed order: no atomics, bitwise reproducible; for the
//    policies whose sums may be regrouped the smallest sets put the sources
//    on the lanes instead (force_lanes_kernel, one launch);
//  * the sum over sources includes j = i, which adds exactly 0 to a_i (d = 0)
//    and m_i / eps to the potential sum; that term is removed at the end.
#include <algorithm>

#include "common.h"

namespace nb {

namespace {

constexpr int NQ = 4;  // partial quantities per sink: ax, ay, az, potential

template <class Pol>
struct ForceArgs {
    using pos_t = typename Pol::pos_t;
    using mass_t = typename Pol::mass_t;
    using calc_t = typename Pol::calc_t;
    const pos_t *xi, *yi, *zi;
    const pos_t *xj, *yj, *zj;
    const mass_t* mj;
    const mass_t* mi;     // masses of the sinks (self set only, for the potential)
    int ni, nj;
    int jspan;            // sources per j-split range, a multiple of BS
    calc_t eps2;
    double G;
    int self_pot;         // remove the j = i term m_i / eps from the potential
    pos_t *ax, *ay, *az, *pot;  // final outputs (part == nullptr)
    TailArgs<pos_t> tail;
    double* part;         // [nsplit][NQ][ni] FP64 partial sums, or nullptr
};

// The potential of sink i from its sum sp.
template <class Pol>
__device__ __forceinline__ void finish_pot(const ForceArgs<Pol>& a, int i, double sp) {
    using calc_t = typename Pol::calc_t;
    double self = 0.0;
    if (a.self_pot) {
        // the j = i term exactly as the pair loop added it
        typename Pol::sum_t t;
        t.init();
        t.add_fma(calc_t(a.mi[i]), rsqrt_pair(a.eps2));
        self = t.total();
    }
    a.pot[i] = typename Pol::pos_t(-a.G * (sp - self));
}

// TAIL: also the leapfrog's tail, from what tail.load gave for the three
// components. The pair kernel leaves it out (it costs
// registers, and with them waves, there: 46 -> 91 VGPRs and 20 % with Kahan
// sums at 262144) but, with one sink per lane, for the closing half-kick alone
// (the same registers), which ends a call: a single step of 200 particles, which
// the pass does in one range, 13.1 us with it, 14.1 with a launch for it.
enum class Tail { None, Kick, All };
template <class Pol, bool POT, Tail TAIL>
__device__ __forceinline__ void finish_sink(const ForceArgs<Pol>& a, int i, double sx, double sy,
                                            double sz, double sp,
                                            const typename TailArgs<typename Pol::pos_t>::In* in = nullptr) {
    using pos_t = typename Pol::pos_t;
    const pos_t ax = pos_t(a.G * sx), ay = pos_t(a.G * sy), az = pos_t(a.G * sz);
    a.ax[i] = ax;
    a.ay[i] = ay;
    a.az[i] = az;
    if (TAIL != Tail::None && a.tail.v) {
        const size_t n = a.ni, n3 = 3 * n;
        if (TAIL == Tail::All) {
            a.tail.apply(i, n3, in[0], ax);
            a.tail.apply(n + i, n3, in[1], ay);
            a.tail.apply(2 * n + i, n3, in[2], az);
        } else {
            pos_t* const v = a.tail.v;
            const pos_t h = a.tail.h;
            v[i] = fmat(h, ax, v[i]);
            v[n + i] = fmat(h, ay, v[n + i]);
            v[2 * n + i] = fmat(h, az, v[2 * n + i]);
        }
    }
    if (POT) finish_pot(a, i, sp);
}

// FEW: built for few waves in flight (kFewWaves): 5003 particles, tile-
// compensated, 20.0 -> 19.1 us a pass, 9377 43.7 -> 42.2; with plain FP32 sums
// 9377 42.9 -> 41.9 (Kahan 60.5 -> 65.6 and FP64 sums 53.9 -> 55.8, so not
// there). Not with the
// potential, whose kernel that build makes slower (9558 particles 46 -> 52 us,
// 128 sinks of 205175 sources 62 -> 89).
template <class Pol, int BS, int K, bool ACC, bool POT, bool FEW>
__global__ __launch_bounds__(BS) NB_WAVES_PER_EU(FEW) void force_kernel(ForceArgs<Pol> a) {
    using calc_t = typename Pol::calc_t;
    using sum_t = typename Pol::sum_t;
    using V4 = typename Vec4<calc_t>::type;
    __shared__ V4 tile[BS];

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
            if (i < a.ni) {
                cx += a.xi[i];
                cy += a.yi[i];
                cz += a.zi[i];
            }
        }
        sink_block_origin<BS / 64>(cx, cy, cz, min(a.ni - b0, BS * K), org, ox, oy, oz);
    }
    calc_t xi[K], yi[K], zi[K];
    sum_t sx[K], sy[K], sz[K], sp[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = i0 + k * BS;
        const bool ok = i < a.ni;
        xi[k] = ok ? pair_coord<Pol>(a.xi[i], ox) : calc_t(0);
        yi[k] = ok ? pair_coord<Pol>(a.yi[i], oy) : calc_t(0);
        zi[k] = ok ? pair_coord<Pol>(a.zi[i], oz) : calc_t(0);
        sx[k].init(); sy[k].init(); sz[k].init(); sp[k].init();
    }
    const calc_t eps2 = a.eps2;
    const int jbeg = blockIdx.y * a.jspan;
    const int jend = min(a.nj, jbeg + a.jspan);

    for (int jt = jbeg; jt < jend; jt += BS) {
        const int j = jt + tid;
        V4 p;
        if (j < jend) {
            p.x = pair_coord<Pol>(a.xj[j], ox);
            p.y = pair_coord<Pol>(a.yj[j], oy);
            p.z = pair_coord<Pol>(a.zj[j], oz);
            p.w = calc_t(a.mj[j]);
        } else {  // zero-mass padding: contributes exactly 0
            p.x = calc_t(0); p.y = calc_t(0); p.z = calc_t(0); p.w = calc_t(0);
        }
        __syncthreads();
        tile[tid] = p;
        __syncthreads();
#pragma unroll 8
        for (int jj = 0; jj < BS; ++jj) {
            const V4 q = tile[jj];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const calc_t dx = q.x - xi[k];
                const calc_t dy = q.y - yi[k];
                const calc_t dz = q.z - zi[k];
                const calc_t s = fmat(dz, dz, fmat(dy, dy, fmat(dx, dx, eps2)));
                const calc_t r = rsqrt_pair(s);
                if (ACC) {
                    calc_t w = r * (r * r);
                    w = w * q.w;
                    sx[k].add_fma(dx, w);
                    sy[k].add_fma(dy, w);
                    sz[k].add_fma(dz, w);
                }
                if (POT) sp[k].add_fma(q.w, r);
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            sx[k].tile_end(); sy[k].tile_end(); sz[k].tile_end(); sp[k].tile_end();
        }
    }

#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = i0 + k * BS;
        if (i >= a.ni) continue;
        if (a.part) {
            double* q = a.part + (size_t)blockIdx.y * NQ * a.ni;
            if (ACC) {
                q[i] = sx[k].total();
                q[(size_t)a.ni + i] = sy[k].total();
                q[(size_t)2 * a.ni + i] = sz[k].total();
            }
            if (POT) q[(size_t)3 * a.ni + i] = sp[k].total();
        } else if (ACC) {
            constexpr Tail KICK = !POT && K == 1 ? Tail::Kick : Tail::None;
            finish_sink<Pol, POT, KICK>(a, i, sx[k].total(), sy[k].total(), sz[k].total(), sp[k].total());
        }
    }
}

// Adds the nsplit partial sums of every sink in a fixed order, then finishes:
// wave g of a group of W adds ranges g, g + W, ... of 64 sinks (eight ranges'
// loads in flight together), and the first wave the W sums in wave order. At
// small ni the kernel is one load latency after another, so four waves share
// them; from 16384 sinks, and up to four ranges, one wave is as fast.
template <class Pol, bool POT, int W>
__global__ __launch_bounds__(256) void force_reduce_kernel(ForceArgs<Pol> a, int nsplit) {
    constexpr int N = POT ? 4 : 3;
    __shared__ double other[W > 1 ? W - 1 : 1][N][64];
    const int lane = threadIdx.x & 63;
    const int g = W > 1 ? threadIdx.x >> 6 : 0;
    const int i = W > 1 ? reduce_first_sink() + lane : blockIdx.x * 256 + threadIdx.x;
    const size_t stride = (size_t)NQ * a.ni;
    double s[N] = {};
    typename TailArgs<typename Pol::pos_t>::In in[3];  // in flight with the partials
    if (!POT && g == 0 && i < a.ni)
#pragma unroll
        for (int c = 0; c < 3; ++c) in[c] = a.tail.load(c * (size_t)a.ni + i, a.xi);
    if (i < a.ni) {
        for (int r0 = g; r0 < nsplit; r0 += W * 8) {
            double t[8][N];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int r = r0 + W * u;
                const double* q = a.part + r * stride + i;
#pragma unroll
                for (int c = 0; c < N; ++c) t[u][c] = r < nsplit ? q[(size_t)c * a.ni] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int c = 0; c < N; ++c) s[c] += t[u][c];
        }
    }
    if constexpr (W > 1) {
        if (g)
#pragma unroll
            for (int c = 0; c < N; ++c) other[g - 1][c][lane] = s[c];
        __syncthreads();
        if (g) return;
#pragma unroll
        for (int v = 0; v < W - 1; ++v)
#pragma unroll
            for (int c = 0; c < N; ++c) s[c] += other[v][c][lane];
    }
    if (i >= a.ni) return;
    finish_sink<Pol, POT, (POT ? Tail::None : Tail::All)>(a, i, s[0], s[1], s[2], POT ? s[N - 1] : 0.0, in);
}

// Sources on the lanes: a workgroup of LB lanes owns LS sinks and each lane
// takes every LB-th source, straight from the SoA arrays (coalesced; the sinks
// are the same for every lane), so that a thousand sinks make 256 workgroups of
// a few pairs per lane; the lanes' sums meet in LDS, 16 lanes a sum, and the
// workgroup finishes its sinks: one launch and no partials where the split
// ranges take two (FP64, 1024 particles: 6.8 us of the pair kernel's latency
// and 4.2 of the reduction's; 4.7 us a leapfrog step so). For the policies whose
// sums may be regrouped: FP64, FP32 terms summed in FP64, plain FP32 (one FP32 sum per lane, the
// lanes' sums added in FP64). The leapfrog's drift goes to another array,
// since other workgroups still read the positions. Up to 3072 sinks (768
// workgroups, so fewer than 3 waves per SIMD with 256 lanes) 512 lanes, which
// halve a lane's chain: us per leapfrog step with 256 and with 512 lanes
// (both before the tail's loads went ahead of the sums, which take 1 off),
//            500        1024       2000       3000        4001        6000
//   FP64     5.7, 5.2   6.1, 5.7   8.2, 8.0   12.0, 11.7  16.6, 16.6  32.2, 33.0
//   FP32     6.7, 6.7   5.1, 4.9   6.6, 6.2   7.9, 7.9    10.4, 11.3  16.5, 16.9
// (not for the policy with a block origin, which is that of 256 sinks).
constexpr int LS = 4;

template <class Pol, bool POT, int LB>
__global__ __launch_bounds__(LB) void force_lanes_kernel(ForceArgs<Pol> a) {
    using calc_t = typename Pol::calc_t;
    using sum_t = typename Pol::sum_t;
    constexpr int N = POT ? 4 : 3, V = LS * N;
    __shared__ double lsum[V][LB + 1];
    const int tid = threadIdx.x;
    const int i0 = blockIdx.x * LS;
    // 16 lanes add sum v, component (or potential) qc of sink iv, and the
    // first of them finishes it; its tail's loads go ahead of everything (one
    // thread a sink, three components one after another with their loads
    // behind the sums, was 1.0-1.4 us a leapfrog step longer: FP64 1024 5.9 ->
    // 4.7, 3000 13.0 -> 10.9, FP32 2000 6.4 -> 5.3)
    const int v = tid >> 4, l = tid & 15, iv = i0 + v / N, qc = v % N;
    const bool last = v < V && l == 0 && iv < a.ni;
    const size_t n = a.ni, kc = qc * n + iv;
    typename TailArgs<typename Pol::pos_t>::In in;
    if (!POT && last) in = a.tail.load(kc, a.xi);  // (no leapfrog asks for the potential)
    // the origin of the one-sided kernel's 256-sink workgroups
    double ox = 0.0, oy = 0.0, oz = 0.0;
    if constexpr (Pol::origin) {
        static_assert(LB == 256);
        __shared__ double org[LB / 64][3];
        const int b0 = i0 / LB * LB, i = b0 + tid;
        const bool ok = i < a.ni;
        sink_block_origin<LB / 64>(ok ? a.xi[i] : 0.0, ok ? a.yi[i] : 0.0, ok ? a.zi[i] : 0.0,
                                   min(a.ni - b0, LB), org, ox, oy, oz);
    }
    calc_t xi[LS], yi[LS], zi[LS];
    sum_t s[LS][N];
#pragma unroll
    for (int k = 0; k < LS; ++k) {
        const int i = min(i0 + k, a.ni - 1);
        xi[k] = pair_coord<Pol>(a.xi[i], ox);
        yi[k] = pair_coord<Pol>(a.yi[i], oy);
        zi[k] = pair_coord<Pol>(a.zi[i], oz);
#pragma unroll
        for (int c = 0; c < N; ++c) s[k][c].init();
    }
#pragma unroll 2
    for (int j = tid; j < a.nj; j += LB) {
        const calc_t x = pair_coord<Pol>(a.xj[j], ox), y = pair_coord<Pol>(a.yj[j], oy),
                     z = pair_coord<Pol>(a.zj[j], oz), m = calc_t(a.mj[j]);
#pragma unroll
        for (int k = 0; k < LS; ++k) {
            const calc_t dx = x - xi[k], dy = y - yi[k], dz = z - zi[k];
            const calc_t ss = fmat(dz, dz, fmat(dy, dy, fmat(dx, dx, a.eps2)));
            const calc_t r = rsqrt_pair(ss);
            calc_t w = r * (r * r);
            w = w * m;
            s[k][0].add_fma(dx, w);
            s[k][1].add_fma(dy, w);
            s[k][2].add_fma(dz, w);
            if (POT) s[k][3].add_fma(m, r);
        }
    }
#pragma unroll
    for (int k = 0; k < LS; ++k)
#pragma unroll
        for (int c = 0; c < N; ++c) lsum[k * N + c][tid] = s[k][c].total();
    __syncthreads();
    if (v >= V) return;
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < LB / 16; ++q) t += lsum[v][q * 16 + l];
#pragma unroll
    for (int mask = 8; mask >= 1; mask >>= 1) t += __shfl_xor(t, mask, 64);
    if (!last) return;
    if (POT && qc == 3) {
        finish_pot(a, iv, t);
        return;
    }
    const typename Pol::pos_t acc = typename Pol::pos_t(a.G * t);
    a.ax[kc] = acc;
    if (!POT && a.tail.v) a.tail.apply(kc, 3 * n, in, acc);
}

// The leapfrog's tail after a pass in one range, whose workgroups finish their
// own sinks while others still read the positions (where it is more than the
// half-kick).
template <class Pol>
__global__ __launch_bounds__(256) void force_tail_kernel(ForceArgs<Pol> a) {
    const size_t k = blockIdx.x * (size_t)256 + threadIdx.x, n3 = 3 * (size_t)a.ni;
    if (k < n3) a.tail.apply(k, n3, a.xi, a.ax[k]);
}

template <class Pol>
ForceArgs<Pol> make_args(int64_t ni, const void* xi, int64_t nj, const void* xj, const void* mj,
                         double eps, double G, bool self_set, void* acc, void* pot) {
    using pos_t = typename Pol::pos_t;
    using mass_t = typename Pol::mass_t;
    using calc_t = typename Pol::calc_t;
    ForceArgs<Pol> a{};
    const pos_t* pi = static_cast<const pos_t*>(xi);
    const pos_t* pj = static_cast<const pos_t*>(xj);
    a.xi = pi; a.yi = pi + ni; a.zi = pi + 2 * ni;
    a.xj = pj; a.yj = pj + nj; a.zj = pj + 2 * nj;
    a.mj = static_cast<const mass_t*>(mj);
    a.mi = self_set ? a.mj : nullptr;
    a.ni = (int)ni;
    a.nj = (int)nj;
    a.eps2 = calc_t(eps) * calc_t(eps);
    a.G = G;
    a.self_pot = (self_set && pot) ? 1 : 0;
    pos_t* po = static_cast<pos_t*>(acc);
    if (po) { a.ax = po; a.ay = po + ni; a.az = po + 2 * ni; }
    a.pot = static_cast<pos_t*>(pot);
    return a;
}

template <class Pol, bool ACC, bool POT, int BS, int K>
hipError_t launch_shape(ForceArgs<Pol> a, int nsplit, hipStream_t stream) {
    dim3 grid((a.ni + BS * K - 1) / (BS * K), nsplit);
    using sum_t = typename Pol::sum_t;
    if constexpr (K == 1 && !POT && (std::is_same<sum_t, SumTile>::value ||
                                     std::is_same<sum_t, SumPlain<float>>::value)) {
        if ((int64_t)grid.x * nsplit * (BS / 64) < 2 * kFewWaves) {
            hipLaunchKernelGGL((force_kernel<Pol, BS, K, ACC, POT, true>), grid, dim3(BS), 0, stream, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((force_kernel<Pol, BS, K, ACC, POT, false>), grid, dim3(BS), 0, stream, a);
    return hipGetLastError();
}

template <class Pol, bool ACC, bool POT>
hipError_t launch_any(const Shape& sh, ForceArgs<Pol> a, int nsplit, hipStream_t stream) {
#define NB_FORCE_CASE(BSV, KV) \
    if (sh.block == BSV && sh.ipl == KV) return launch_shape<Pol, ACC, POT, BSV, KV>(a, nsplit, stream);
    NB_FORCE_CASE(64, 1) NB_FORCE_CASE(64, 2) NB_FORCE_CASE(64, 4)
    NB_FORCE_CASE(128, 1) NB_FORCE_CASE(128, 2) NB_FORCE_CASE(128, 4)
    NB_FORCE_CASE(256, 1) NB_FORCE_CASE(256, 2) NB_FORCE_CASE(256, 4)
    NB_FORCE_CASE(512, 1) NB_FORCE_CASE(512, 2) NB_FORCE_CASE(512, 4)
    NB_FORCE_CASE(1024, 1) NB_FORCE_CASE(1024, 2) NB_FORCE_CASE(1024, 4)
#undef NB_FORCE_CASE
    return hipErrorInvalidValue;
}

template <class Pol, bool ACC, bool POT>
hipError_t run_force(const Shape& sh, ForceArgs<Pol> a, void* ws, bool partials_only,
                     hipStream_t stream, bool* drifted = nullptr) {
    if (sh.lanes) {
        if constexpr (std::is_same<typename Pol::sum_t, SumKahan>::value ||
                      std::is_same<typename Pol::sum_t, SumTile>::value ||
                      std::is_same<Pol, PolMixAcc32>::value) {
            return hipErrorInvalidValue;
        } else {
            if (a.tail.x == a.xi) a.tail.x = nullptr;
            if (drifted) *drifted = a.tail.x != nullptr;
            a.part = nullptr;
            const dim3 grid((a.ni + LS - 1) / LS);
            if constexpr (!Pol::origin) {
                if (sh.block == 512) {
                    hipLaunchKernelGGL((force_lanes_kernel<Pol, POT, 512>), grid, dim3(512), 0, stream, a);
                    return hipGetLastError();
                }
            }
            hipLaunchKernelGGL((force_lanes_kernel<Pol, POT, 256>), grid, dim3(256), 0, stream, a);
            return hipGetLastError();
        }
    }
    const int span = split_span(a.nj, sh.split, sh.block);
    const int nsplit = split_ranges(a.nj, sh.split, sh.block);
    a.jspan = span;
    if (drifted) *drifted = a.tail.x != nullptr;
    if (nsplit == 1 && !partials_only) {
        a.part = nullptr;
        // a tail of the half-kick alone in the pair kernel, else after it
        ForceArgs<Pol> pass = a;
        if (sh.ipl > 1 || !a.tail.close || a.tail.store || a.tail.x) pass.tail.v = nullptr;
        const hipError_t e = launch_any<Pol, ACC, POT>(sh, pass, 1, stream);
        if (e != hipSuccess || pass.tail.v == a.tail.v) return e;
        hipLaunchKernelGGL(force_tail_kernel<Pol>, dim3((unsigned)((3 * (int64_t)a.ni + 255) / 256)),
                           dim3(256), 0, stream, a);
        return hipGetLastError();
    }
    a.part = static_cast<double*>(ws);
    hipError_t e = launch_any<Pol, ACC, POT>(sh, a, nsplit, stream);
    if (e != hipSuccess || partials_only) return e;
    if (a.ni < 16384 && nsplit > 4)
        hipLaunchKernelGGL((force_reduce_kernel<Pol, POT, 4>), reduce_grid(sh, a.ni), dim3(256), 0,
                           stream, a, nsplit);
    else
        hipLaunchKernelGGL((force_reduce_kernel<Pol, POT, 1>), dim3((a.ni + 255) / 256), dim3(256), 0,
                           stream, a, nsplit);
    return hipGetLastError();
}

}  // namespace

bool shape_supported(const Shape& s) {
    const bool bs_ok = s.block == 64 || s.block == 128 || s.block == 256 || s.block == 512 ||
                       s.block == 1024;
    const bool k_ok = s.ipl == 1 || s.ipl == 2 || s.ipl == 4;
    return bs_ok && k_ok && s.split >= 1 && s.split <= 256;
}

size_t force_partials_bytes(const Shape& s, int64_t ni) {
    if (s.lanes) return 0;
    return (size_t)s.split * NQ * (size_t)ni * sizeof(double);
}

// Policies whose small passes take ranges as short as one tile: not those
// that keep a plain or compensated FP32 sum over the range, whose length is
// part of their arithmetic. And the waves up to which they do, 6 per SIMD.
static bool tile_ranges(int prec) { return prec != NB_MIX_ACC32 && prec != NB_MIX_KAHAN; }
constexpr int64_t kRangeWaves = 6144;

// Upper bound of force_partials_bytes(choose_force_shape(prec, ni, nj), ni)
// over every ni, nj <= n (a small sink set against a large source set takes
// the most ranges). From the rule below:
//  * a range is at least 4 tiles of >= 128 sources, or 8 of 64, i.e. >= 512
//    sources, except that below 16384 sources ranges as short as one tile
//    are allowed, at most 64 of them: split <= max(n/512, min(64, nj/64));
//  * split <= 256;
//  * split > 1 only while waves < 65536, where split <= 65536/waves + 1 and
//    ni <= waves * 64 * ipl, so split * ni < 2^23 * ipl <= 2^24 for the
//    shapes with ipl <= 2; the shape with ipl = 4 serves fewer than 65536
//    sinks, so there split * ni <= 256 * 65536 = 2^24 as well.
// and, for the policies with tile-long ranges of few waves (kRangeWaves at
// most in all, each range 256 sources or more):
//  * split <= min(256, ceil(n / 256)) and split * waves <= kRangeWaves, where
//    a wave has 64 * ipl sinks: ipl is 4 at most in FP64, 2 otherwise.
size_t force_partials_bound(int prec, int64_t n) {
    const int64_t short_ranges = std::min<int64_t>(64, std::min<int64_t>(n, 16383) / 64);
    const int64_t split = std::min<int64_t>(256, std::max<int64_t>(n / 512, short_ranges));
    int64_t rows = split > 1 ? std::min<int64_t>(split * n, int64_t(1) << 24) : 0;  // split * ni
    if (tile_ranges(prec)) {
        const int64_t most = std::min<int64_t>(256, (n + 255) / 256);
        const int64_t few = std::min<int64_t>(most * n, kRangeWaves * 64 * (prec == NB_F64 ? 4 : 2));
        if (most > 1) rows = std::max(rows, few);
    }
    return (size_t)rows * NQ * sizeof(double);
}

Shape choose_force_shape(int prec, int64_t ni, int64_t nj, Pick pick) {
    // Sources on the lanes (force_lanes_kernel), for the policies whose sums
    // may be regrouped, as long as a lane has few sources: us per leapfrog
    // step against the split ranges below, measured on MI355X,
    //            1024        4001         8000         12000
    //   FP64     4.7, 10.0   15.9, 24.2   49.5, 58.0   104.8, 112.2
    //   FP32     4.5, 13.2    9.1, 14.6   24.2, 29.7   47.4, 60.6
    //   acc64    6.0, 16.7   16.0, 18.7   44.4, 41.7   88.2, 86.4
    // so up to 6000 sources for FP64 sums of FP32 terms, whose lanes carry
    // the longest chain, and for few FP64 sinks, where a lane's sources are
    // the whole time (100 against 12000: 15.3, 14.3; 1000: 16.4, 19.7), and not
    // above 12032 sinks and sources in FP64, where a range of 256 sources has 48
    // workgroups, a multiple of the XCDs (a pass alone and with the potential:
    // 12287 109.1, 101.3 and 110.8, 106.8; but 12001 105.7, 103.8 and 107.5,
    // 111.0).
    // Larger sets on themselves have the symmetric pass in FP64 and FP32.
    const bool regroup = prec == NB_F64 || prec == NB_F32 || prec == NB_MIX_ACC64;
    const int64_t most = prec == NB_MIX_ACC64 || (prec == NB_F64 && ni < 512) ? 6000
                         : prec == NB_F64 && ni > 12032                       ? 12032
                                                                              : 12287;
    if (pick == Pick::Best && regroup && ni <= 12287 && nj <= most) {
        const int lanes = prec != NB_MIX_ACC64 && ni <= 3072 && nj > 256 ? 512 : 256;
        Shape s{LS, lanes, lanes};
        s.lanes = true;
        return s;
    }
    // Measured on MI355X (launch-shape sweeps at N = 2^10 .. 2^20):
    //  * FP32 pair arithmetic: 1 sink per lane in 256-lane workgroups up to
    //    12288 sinks, then 2 sinks per lane, 128-lane workgroups, and
    //    512-lane ones (fewer barriers per pair) from 65536 sinks up;
    //  * FP64: 64-lane workgroups below 65536 sinks (1 sink per lane below
    //    3072, else 4), 256 lanes above;
    //  * many more workgroups than the chip holds at once balance the CUs
    //    better even when one round would already fill every SIMD: split the
    //    source range until there are ~64K wavefronts (8 ranges at 2^20, 32
    //    at 2^18, 5-16 % faster), keeping every range >= 4 tiles long (8
    //    for the 64-lane FP64 shape) -- or, below 16384 sources, as short as
    //    one tile, up to 32 ranges (64 in FP64): 6x faster at N = 1024 in
    //    FP64, 2.6x at 4096 in FP32, where the pass is otherwise a handful
    //    of workgroups.
    Shape s;
    if (prec == NB_F64) {
        s = ni < 3072 ? Shape{1, 64, 1} : (ni < 65536 ? Shape{4, 64, 1} : Shape{1, 256, 1});
    } else {
        s = ni <= 12288 ? Shape{1, 256, 1} : Shape{2, ni >= 65536 ? 512 : 128, 1};
    }
    const int64_t groups = (ni + (int64_t)s.block * s.ipl - 1) / ((int64_t)s.block * s.ipl);
    const int64_t waves = groups * (s.block / 64);
    const int64_t want = 65536;
    int64_t split = (want + waves - 1) / waves;
    const int64_t min_tiles = (prec == NB_F64 && s.block == 64) ? 8 : 4;
    const int64_t long_ranges = nj / (min_tiles * (int64_t)s.block);
    const int64_t short_ranges =
        nj < 16384 ? std::min<int64_t>(prec == NB_F64 ? 64 : 32, nj / (int64_t)s.block) : 0;
    const int64_t max_ranges = std::max(long_ranges, short_ranges);
    if (split > max_ranges) split = max_ranges;
    if (split > 256) split = 256;
    if (split < 1) split = 1;
    // Ranges as short as one tile, whatever nj, until there are 6 waves per
    // SIMD: with fewer, the pass takes as long as one range does (the
    // rule above rounds 5003 sources in 19 ranges up to 10 ranges of two
    // tiles on 800 waves). Not for the policies that keep a plain or
    // compensated FP32 sum over the range: its length is part of their
    // arithmetic. With both changes of the reduction and the ranges a pass
    // takes 13.7 us instead of 21.9 at 1000 particles and 20.3 instead of
    // 23.8 at 5003 (at 11239 with the potential, 44 ranges of one tile are
    // 2 % slower than 22 of two). From 3.5 waves per SIMD with the rule above on
    // only if they make 5.5: between, some SIMDs have five waves and others
    // four (FP64 sums, us without and with them: 15000, 3540 waves, 125.5, 117.0;
    // 15500, 3782 to 5002, 130.1, 134.3; 16384, 4096 to 5504, 126.5, 133.4;
    // 17000, 3618 to 6030, 151.8, 140.6).
    if (pick != Pick::Least && tile_ranges(prec)) {
        const int64_t some = split_ranges(nj, split, s.block);
        const int64_t more = short_tile_ranges(nj, s.block, waves, kRangeWaves);
        if (some * waves < kFewWaves * 7 / 8 || more * waves >= 5632) split = std::max(some, more);
    }
    s.split = (int)split;
    return s;
}

hipError_t launch_force(int prec, const Shape& shape, int64_t ni, const void* xi, int64_t nj,
                        const void* xj, const void* mj, double eps, double G, bool self_set,
                        void* acc, void* pot, void* ws, hipStream_t stream, const StepTail& tail,
                        bool* drifted) {
    hipError_t err = hipErrorInvalidValue;
    if (drifted) *drifted = false;
    dispatch_prec(prec, [&](auto tag) {
        using Pol = decltype(tag);
        using pos_t = typename Pol::pos_t;
        auto a = make_args<Pol>(ni, xi, nj, xj, mj, eps, G, self_set, acc, pot);
        if (self_set) a.tail = TailArgs<pos_t>(tail);
        err = pot ? run_force<Pol, true, true>(shape, a, ws, false, stream, drifted)
                  : run_force<Pol, true, false>(shape, a, ws, false, stream, drifted);
    });
    return err;
}

}  // namespace nb
