// O(N) kernels of the kick-drift-kick leapfrog and of its reverse walk (the
// closing half-kick of a step runs in the force kernel's epilogue). Each
// thread updates components of the 3n-element SoA arrays; all accesses are
// unit-stride and coalesced. These kernels are bound by HBM traffic, not
// arithmetic: per component a kick-drift moves 5 values, a reverse drift 7.
#include "common.h"

namespace nb {

namespace {

constexpr int TPB = 256;

inline dim3 grid_for(int64_t count) {
    int64_t blocks = (count + TPB - 1) / TPB;
    if (blocks > 65536) blocks = 65536;  // grid-stride beyond this
    return dim3((unsigned)blocks);
}

// v <- v + h a; xout <- x + dt v (xout may be x)
template <typename T>
__global__ __launch_bounds__(TPB) void kick_drift_kernel(const T* x, T* xout, T* __restrict__ v,
                                                         const T* __restrict__ a, T h, T dt,
                                                         int64_t count) {
    for (int64_t k = blockIdx.x * (int64_t)TPB + threadIdx.x; k < count;
         k += (int64_t)gridDim.x * TPB) {
        const T vh = fmat(h, a[k], v[k]);  // the same FMAs as the force epilogue's
        v[k] = vh;
        xout[k] = fmat(dt, vh, x[k]);
    }
}

// Reverse of a drift and of the kick before it:
// lam_v <- lam_v + dt lam_x; v <- v - h a; x <- x - dt v.
template <typename T>
__global__ __launch_bounds__(TPB) void reverse_drift_kernel(T* __restrict__ x, T* __restrict__ v,
                                                            const T* __restrict__ a,
                                                            const T* __restrict__ lx,
                                                            T* __restrict__ lv, T h, T dt,
                                                            int64_t count) {
    for (int64_t k = blockIdx.x * (int64_t)TPB + threadIdx.x; k < count;
         k += (int64_t)gridDim.x * TPB) {
        lv[k] = fmat(dt, lx[k], lv[k]);  // the same FMAs as the adjoint epilogue's
        const T vh = fmat(-h, a[k], v[k]);
        v[k] = vh;
        x[k] = fmat(-dt, vh, x[k]);
    }
}

// A checkpoint slot receives (x, v, a): one launch for the three arrays.
template <typename T>
__global__ __launch_bounds__(TPB) void store_kernel(const T* __restrict__ x, const T* __restrict__ v,
                                                    const T* __restrict__ a, T* __restrict__ slot,
                                                    int64_t count) {
    for (int64_t k = blockIdx.x * (int64_t)TPB + threadIdx.x; k < count;
         k += (int64_t)gridDim.x * TPB) {
        slot[k] = x[k];
        slot[count + k] = v[k];
        slot[2 * count + k] = a[k];
    }
}

// lam_v <- lam_v + dt lam_x, and the state of a checkpoint slot: x, and v and
// a where whole.
template <typename T>
__global__ __launch_bounds__(TPB) void reload_kernel(T* __restrict__ x, T* __restrict__ v,
                                                     T* __restrict__ a, const T* __restrict__ lx,
                                                     T* __restrict__ lv, T dt,
                                                     const T* __restrict__ slot, int whole,
                                                     int64_t count) {
    for (int64_t k = blockIdx.x * (int64_t)TPB + threadIdx.x; k < count;
         k += (int64_t)gridDim.x * TPB) {
        lv[k] = fmat(dt, lx[k], lv[k]);
        x[k] = slot[k];
        if (whole) {
            v[k] = slot[count + k];
            a[k] = slot[2 * count + k];
        }
    }
}

}  // namespace

hipError_t launch_kick_drift(int prec, int64_t n, const void* x, void* xout, void* v,
                             const void* acc, double h, double dt, hipStream_t stream) {
    const int64_t c = 3 * n;
    if (prec == NB_F32)
        hipLaunchKernelGGL(kick_drift_kernel<float>, grid_for(c), dim3(TPB), 0, stream,
                           static_cast<const float*>(x), static_cast<float*>(xout),
                           static_cast<float*>(v), static_cast<const float*>(acc), float(h),
                           float(dt), c);
    else
        hipLaunchKernelGGL(kick_drift_kernel<double>, grid_for(c), dim3(TPB), 0, stream,
                           static_cast<const double*>(x), static_cast<double*>(xout),
                           static_cast<double*>(v), static_cast<const double*>(acc), h, dt, c);
    return hipGetLastError();
}

hipError_t launch_reverse_drift(int prec, int64_t n, void* x, void* v, const void* acc,
                                const void* lam_x, void* lam_v, double h, double dt,
                                hipStream_t stream) {
    const int64_t c = 3 * n;
    if (prec == NB_F32)
        hipLaunchKernelGGL(reverse_drift_kernel<float>, grid_for(c), dim3(TPB), 0, stream,
                           static_cast<float*>(x), static_cast<float*>(v),
                           static_cast<const float*>(acc), static_cast<const float*>(lam_x),
                           static_cast<float*>(lam_v), float(h), float(dt), c);
    else
        hipLaunchKernelGGL(reverse_drift_kernel<double>, grid_for(c), dim3(TPB), 0, stream,
                           static_cast<double*>(x), static_cast<double*>(v),
                           static_cast<const double*>(acc), static_cast<const double*>(lam_x),
                           static_cast<double*>(lam_v), h, dt, c);
    return hipGetLastError();
}

namespace {
template <typename T>
hipError_t store_any(int64_t c, const void* x, const void* v, const void* acc, void* slot,
                     hipStream_t stream) {
    hipLaunchKernelGGL(store_kernel<T>, grid_for(c), dim3(TPB), 0, stream, static_cast<const T*>(x),
                       static_cast<const T*>(v), static_cast<const T*>(acc), static_cast<T*>(slot), c);
    return hipGetLastError();
}

template <typename T>
hipError_t reload_any(int64_t c, void* x, void* v, void* acc, const void* lam_x, void* lam_v,
                      double dt, const void* slot, bool whole, hipStream_t stream) {
    hipLaunchKernelGGL(reload_kernel<T>, grid_for(c), dim3(TPB), 0, stream, static_cast<T*>(x),
                       static_cast<T*>(v), static_cast<T*>(acc), static_cast<const T*>(lam_x),
                       static_cast<T*>(lam_v), T(dt), static_cast<const T*>(slot), int(whole), c);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_store(int prec, int64_t n, const void* x, const void* v, const void* acc,
                        void* slot, hipStream_t stream) {
    return prec == NB_F32 ? store_any<float>(3 * n, x, v, acc, slot, stream)
                          : store_any<double>(3 * n, x, v, acc, slot, stream);
}

hipError_t launch_reload(int prec, int64_t n, void* x, void* v, void* acc, const void* lam_x,
                         void* lam_v, double dt, const void* slot, bool whole, hipStream_t stream) {
    return prec == NB_F32
               ? reload_any<float>(3 * n, x, v, acc, lam_x, lam_v, dt, slot, whole, stream)
               : reload_any<double>(3 * n, x, v, acc, lam_x, lam_v, dt, slot, whole, stream);
}

}  // namespace nb
