// Device helpers shared by the kernel files: loads and stores through the
// global, constant and LDS address spaces, cross-lane moves, and the
// fixed-order sums of the reductions.
#pragma once

#include "cuth_internal.hpp"

#include <cmath>
#include <type_traits>

namespace cuth {
namespace {

template <typename T, int VX>
struct alignas(sizeof(T) * VX) Vec {
    T a[VX];
};

// Device memory (hipMalloc'd buffers only: never LDS or private memory) is
// reached through global-address-space pointers: the vectors and coefficients
// come from descriptors in memory, so the compiler cannot place them and would
// emit flat accesses, which also count against the LDS counter (a wait for a
// cross-lane exchange would then wait for every load in flight).
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(1))) T *as_global(const T *p) {
    return (const __attribute__((address_space(1))) T *)p;
}
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T *as_global(T *p) {
    return (__attribute__((address_space(1))) T *)p;
}
// Raw words of B bytes (class types are moved through these, because
// address-space-qualified class objects cannot be copied in host passes).
template <int B> struct Words;
template <> struct Words<2> { using type = unsigned short; };
template <> struct Words<4> { using type = unsigned int; };
template <> struct Words<8> { using type = unsigned int __attribute__((ext_vector_type(2))); };
template <> struct Words<16> { using type = unsigned int __attribute__((ext_vector_type(4))); };

// One value (a number, or a struct of 32-bit words such as LayerCoef).
template <typename T>
__device__ __forceinline__ T gld(const T *p) {
    if constexpr (std::is_arithmetic<T>::value) {
        return *as_global(p);
    } else {
        static_assert(sizeof(T) % 4 == 0, "whole 32-bit words");
        const __attribute__((address_space(1))) unsigned int *q =
            (const __attribute__((address_space(1))) unsigned int *)(const void *)p;
        unsigned int w[sizeof(T) / 4];
#pragma unroll
        for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = q[i];
        T v;
        __builtin_memcpy(&v, w, sizeof(T));
        return v;
    }
}

// A value that no kernel writes while it runs and every lane of the wavefront
// reads at the same address (per-layer coefficients): loaded through the
// constant address space, so that it can come through scalar loads.
template <typename T>
__device__ __forceinline__ T gldc(const T *p) {
    static_assert(sizeof(T) % 4 == 0, "whole 32-bit words");
    const __attribute__((address_space(4))) unsigned int *q =
        (const __attribute__((address_space(4))) unsigned int *)(const void *)p;
    unsigned int w[sizeof(T) / 4];
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = q[i];
    T v;
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}

template <typename T, int VX>
__device__ __forceinline__ Vec<T, VX> vload(const T *p) {
    // callers pass cells whose index is a multiple of VX (VX divides nx)
    using W = typename Words<(int)sizeof(Vec<T, VX>)>::type;
    const void *a = __builtin_assume_aligned(p, sizeof(T) * VX);
    const W w = *(const __attribute__((address_space(1))) W *)a;
    return __builtin_bit_cast(Vec<T, VX>, w);
}

template <typename T, int VX>
__device__ __forceinline__ void vstore(T *p, const Vec<T, VX> &v) {
    using W = typename Words<(int)sizeof(Vec<T, VX>)>::type;
    *(__attribute__((address_space(1))) W *)(void *)p = __builtin_bit_cast(W, v);
}

// Vectors of the workgroup's LDS (pointers derived from a __shared__ array,
// which the compiler turns into LDS instructions).  vload/vstore must never
// see such a pointer: an LDS address taken as a global one is unmapped.
template <typename T, int VX>
__device__ __forceinline__ Vec<T, VX> lds_load(const T *p) {
    return *reinterpret_cast<const Vec<T, VX> *>(p);
}
template <typename T, int VX>
__device__ __forceinline__ void lds_store(T *p, const Vec<T, VX> &v) {
    *reinterpret_cast<Vec<T, VX> *>(p) = v;
}

// The value held by the lane to the left (lane - 1) or to the right (lane + 1)
// in the wavefront, moved by a DPP wavefront shift (a VALU operation, no LDS
// traffic); lane 0, respectively lane 63, receives 0.
template <int CTRL, typename T>
__device__ __forceinline__ T dpp_move(T v) {
    static_assert(sizeof(T) % 4 == 0, "whole 32-bit words");
    int w[sizeof(T) / 4];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i)
        w[i] = __builtin_amdgcn_update_dpp(0, w[i], CTRL, 0xf, 0xf, false);
    T r;
    __builtin_memcpy(&r, w, sizeof(T));
    return r;
}
template <typename T>
__device__ __forceinline__ T lane_left(T v) {
    return dpp_move<0x138>(v);   // wave_shr:1
}
template <typename T>
__device__ __forceinline__ T lane_right(T v) {
    return dpp_move<0x130>(v);   // wave_shl:1
}

// 1/d for the Jacobi scaling: the hardware reciprocal in FP32 (within 1 ulp:
// the preconditioner only needs a fixed positive diagonal), a division in FP64.
template <typename T>
__device__ __forceinline__ T recip(T d) {
    if constexpr (sizeof(T) == 4) return __builtin_amdgcn_rcpf(d);
    else return T(1) / d;
}

template <typename T, int VX>
__device__ __forceinline__ Vec<T, VX> vzero() {
    Vec<T, VX> v;
#pragma unroll
    for (int e = 0; e < VX; ++e) v.a[e] = T(0);
    return v;
}

// VX FP16 values (bit patterns) promoted to T and multiplied by the layer's
// scale factor hs = 2^-e_l (exact: a power of two).
template <typename T, int VX>
__device__ __forceinline__ Vec<T, VX> h16load(const uint16_t *p, T hs) {
    const Vec<uint16_t, VX> b = vload<uint16_t, VX>(p);
    Vec<T, VX> v;
#pragma unroll
    for (int e = 0; e < VX; ++e) v.a[e] = (T)(float)__builtin_bit_cast(_Float16, b.a[e]) * hs;
    return v;
}

__device__ __forceinline__ float h16one(uint16_t b) {
    return (float)__builtin_bit_cast(_Float16, b);
}

__device__ __forceinline__ int tid_lin() { return threadIdx.x + kWave * threadIdx.y; }
__device__ __forceinline__ int nthreads() { return kWave * blockDim.y; }

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

template <typename T>
__device__ __forceinline__ bool finite_val(T v) {
    return isfinite(v);
}

// Sum (or max for the values whose bit is set in maxmask; those are >= 0) of
// v[k] over the workgroup; written by thread 0 to part[k*nb + slot].
template <typename T, int NV>
__device__ __forceinline__ void block_partials(T (&v)[NV], unsigned maxmask, T *part, int nb,
                                               int slot) {
    __shared__ T sh[NV][kMaxBY];
    const int lane = threadIdx.x, w = threadIdx.y, nw = blockDim.y;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const bool mx = (maxmask >> k) & 1u;
        const T x = mx ? wave_max(v[k]) : wave_sum(v[k]);
        if (lane == 0) sh[k][w] = x;
    }
    __syncthreads();
    if (tid_lin() == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const bool mx = (maxmask >> k) & 1u;
            T a = sh[k][0];
            for (int q = 1; q < nw; ++q) a = mx ? fmax(a, sh[k][q]) : a + sh[k][q];
            part[(size_t)k * nb + slot] = a;
        }
    }
}

// Fixed-order sum of np partials written by the previous kernel; every thread
// of every workgroup obtains the same value.
template <typename T>
__device__ __forceinline__ T reduce_prev(const T *part, int np) {
    __shared__ T sh[kMaxBY];
    // 16 independent loads in flight per lane (one L2 round trip per 1024
    // partials of a 64-lane workgroup), then a fixed-order combine
    constexpr int U = 16;
    const int n = nthreads();
    T acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = T(0);
    int q = tid_lin();
    for (; q + (U - 1) * n < np; q += U * n) {
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] += part[q + u * n];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (q + u * n < np) acc[u] += part[q + u * n];
    T a = T(0);
#pragma unroll
    for (int u = 0; u < U; ++u) a += acc[u];
    a = wave_sum(a);
    if (threadIdx.x == 0) sh[threadIdx.y] = a;
    __syncthreads();
    T s = sh[0];
    for (int q = 1; q < (int)blockDim.y; ++q) s += sh[q];
    __syncthreads();
    return s;
}

// Slot of this workgroup in the XCD-banded order.
__device__ __forceinline__ int xcd_slot() {
    const int nb = gridDim.x, b = blockIdx.x;
    const int xcd = b & 7, k = b >> 3;
    const int per = nb >> 3, rem = nb & 7;
    return xcd * per + (xcd < rem ? xcd : rem) + k;
}

// Problem pidx's sum of the previous kernel's partials: summed here by every
// workgroup (red == 0), or already summed by k_reduce_b into part_in[pidx].
template <typename T>
__device__ __forceinline__ T prev_sum(const T *part_in, int red, int pidx, const InnerProb<T> &P) {
    if (red) return part_in[pidx];
    return reduce_prev(part_in + P.tile0, P.ntiles);
}

// Convergence test of the first kernel after a CG update: every workgroup of
// the problem obtains the same r^T r and agrees.
template <typename T>
__device__ __forceinline__ bool conv_test(CgState<T> *st, const T *part_in, int red, int pidx,
                                          const InnerProb<T> &P, bool lead) {
    const T tol2 = st->tol2;
    const T rr = prev_sum(part_in, red, pidx, P);
    const bool stop = !(rr > tol2) || !finite_val(rr);
    if (lead && tid_lin() == 0) {
        st->rr = rr;
        st->iter = st->iter + 1;
        if (stop) st->done = finite_val(rr) ? 1 : 4;
    }
    return stop;
}

}  // namespace
}  // namespace cuth
