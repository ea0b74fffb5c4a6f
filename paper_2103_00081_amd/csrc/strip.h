// Shared by the strip kernels (op_q1s.hip, op_q2s.hip, op_hexs.hip): raw buffer access, lane
// shifts, and where a launch finds its work.
#pragma once
#include <type_traits>

#include "common.h"
#include "dev_util.h"

namespace hts {

// ----------------------------------------------- raw buffer access, lane shifts
constexpr uint32_t OOB = 0xFF000000u;   // byte offset past any plane (planes stay below 2^31 bytes)

using Rsrc = __amdgpu_buffer_rsrc_t;
// `bytes` bytes from p; 0: every access is out of range (loads give zero)
__device__ __forceinline__ static Rsrc rsrc(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
template <typename T>
__device__ __forceinline__ static T bld(Rsrc r, uint32_t off)
{
    if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
template <typename T>
__device__ __forceinline__ static void bst(Rsrc r, uint32_t off, T v)
{
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    if constexpr (sizeof(T) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, 0, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, off, 0, 0);
}

// the value of lane + 1 (wave_shl:1) and of lane - 1 (wave_shr:1); zero past
// the ends.  All 64 lanes are active where these are used.
template <int CTRL>
__device__ __forceinline__ static float wshift(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ static double wshift(double v)
{
    struct P { int lo, hi; } p = __builtin_bit_cast(P, v);
    p.lo = __builtin_amdgcn_update_dpp(0, p.lo, CTRL, 0xf, 0xf, true);
    p.hi = __builtin_amdgcn_update_dpp(0, p.hi, CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, p);
}
template <typename T>
__device__ __forceinline__ static T from_right(T v) { return wshift<0x130>(v); }
template <typename T>
__device__ __forceinline__ static T from_left(T v) { return wshift<0x138>(v); }

__device__ __forceinline__ static float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ static double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Where a launch finds its operator and work: in device tables (batches), or in
// its own arguments (one mesh: two dependent reads less before a wave starts)
struct Tabled {
    const OpDev *ops;
    const WorkItem *work;
    __device__ __forceinline__ WorkItem item() const { return work[blockIdx.x]; }
    __device__ __forceinline__ const OpDev &op(int inst) const { return ops[inst]; }
};
struct Solo {
    OpDev o;
    int32_t ntx, zc, total, per;   // work item i: tile i % ntx, planes from (i / ntx) zc; per = blocks of an XCD
    __device__ __forceinline__ WorkItem item() const
    {
        const int i = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
        WorkItem w{};
        w.inst = i < total ? 0 : -1;
        w.tx = i % ntx;
        w.z0 = i / ntx * zc;
        w.z1 = min(o.NZ, w.z0 + zc);
        return w;
    }
    __device__ __forceinline__ const OpDev &op(int) const { return o; }
};

// argument of a one-mesh launch over ntx blocks per plane range of zc
inline Solo solo_work(const OpDev &op, int ntx, int zc)
{
    Solo a{op, ntx, zc, 0, 0};
    a.total = ntx * ((op.NZ + zc - 1) / zc);
    a.per = (a.total + 7) / 8;
    return a;
}

}  // namespace hts
