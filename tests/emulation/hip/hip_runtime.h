// Host stand-ins for what the on-chip preconditioner's kernel takes from the HIP
// headers and the compiler, for running it on the CPU (onchip_emulation.cpp): a
// lane is a fiber, a workgroup an operating-system thread, and one wavefront of all
// runs at a time, from one cross-lane operation or barrier to its next.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstring>

#define __host__
#define __device__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n)

using std::isfinite;
using std::min;
using hipStream_t = void *;
using hipError_t = int;
struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};

namespace emu {
enum Kind { kShiftUp = 0x138, kShiftDown = 0x130, kLane, kXor, kAnd, kWave };   // (the first two: DPP controls)
struct Here {
    dim3 thread, block, dim, grid;
};
Here &here();
uint64_t cross(Kind kind, uint64_t v, int q);   // every lane of the wavefront calls it
void barrier(int line);
unsigned char *dynamic_lds();

inline int dpp(int v, int ctrl) { return (int)cross((Kind)ctrl, (uint32_t)v, 0); }
inline int readlane(int v, int q) { return (int)cross(kLane, (uint32_t)v, q); }
template <typename T>
T shfl_xor(T v, int o) {
    uint64_t w = 0;
    std::memcpy(&w, &v, sizeof v);
    w = cross(kXor, w, o);
    std::memcpy(&v, &w, sizeof v);
    return v;
}
}  // namespace emu

#define threadIdx (emu::here().thread)
#define blockIdx (emu::here().block)
#define blockDim (emu::here().dim)
#define gridDim (emu::here().grid)
#define __syncthreads() emu::barrier(__LINE__)
#define __shfl_xor(v, o, w) emu::shfl_xor(v, o)
#define __all(p) (emu::cross(emu::kAnd, (p) ? 1 : 0, 0) != 0)
#define __builtin_amdgcn_update_dpp(old, v, ctrl, rows, banks, zero) emu::dpp(v, ctrl)
#define __builtin_amdgcn_readlane(v, q) emu::readlane(v, q)
#define __builtin_amdgcn_readfirstlane(v) emu::readlane(v, 0)
#define __builtin_amdgcn_s_setprio(p) ((void)0)
#define __builtin_amdgcn_s_waitcnt(m) ((void)0)
#define __builtin_amdgcn_sched_barrier(m) ((void)0)
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __hip_atomic_store(p, v, order, scope) ((void)(*(p) = (v)))
#define __hip_atomic_load(p, order, scope) (*(p))
#define hipLaunchKernelGGL(...) ((void)++emu_launches)
inline int emu_launches = 0;
