// Device helpers shared by the grouped engines (rt_group.hip, rt_group_f32.hip).
#pragma once
#include "rt_ll.h"

namespace rt {

// A pointer read out of the kernel's arguments by a computed index is a generic address to the compiler; all of these are
// global memory.
template <typename T> __device__ __forceinline__ T *as_global(T *p)
{
    return (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
}

struct GroupWait {   // what the bounded waits of rt_ll.h need
    long long spin_limit;
    unsigned long long *bar;
};

// a word at a 32-bit offset from a uniform base: no 64-bit address per lane
__device__ __forceinline__ void word_store(unsigned long long *base, unsigned idx, unsigned tag, unsigned payload)
{
    ll_store(reinterpret_cast<ll_t *>(reinterpret_cast<char *>(base) + (size_t)(idx * 8u)), tag, payload);
}

template <int CTRL> __device__ __forceinline__ unsigned quad_move(unsigned v)
{
    return (unsigned)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}

// The four rows of 16 lanes hold partial sums: fold2 adds the halves of two accumulators (low lanes get a's sum, high lanes
// b's), fold1 the rows 0 + 1 and 2 + 3 (row 0: a low, row 1: b low, row 2: a high, row 3: b high).
__device__ __forceinline__ float fold2(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float fold1(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ float tile_sum(const float *red, int row4b)   // row4b = 4 row + batch row
{
    float v[kPW];
#pragma unroll
    for (int w = 0; w < kPW; ++w) v[w] = red[w * 256 + row4b];
    return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
}
// value of lane + 4 inside a row of 16 lanes (row_shl:4): the partner of a bf16 pair where the lanes are [row][4]
__device__ __forceinline__ float row_partner(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x104, 0xF, 0xF, true));
}
// sum over the lanes that are equal modulo 4
__device__ __forceinline__ float sum_mod4(float v)
{
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xF, 0xF, true));   // row_ror:8
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x124, 0xF, 0xF, true));
    v = fold1(v, v);
    return fold2(v, v);
}

// Workgroup barrier behind which every wavefront leaves when one has given up waiting (G: GroupWait, flag_s: LDS flags).
#define RT_GROUP_SYNC(cond)                                                                                               \
    do {                                                                                                                  \
        if (cond) flag_s[1] = 1;                                                                                          \
        __syncthreads();                                                                                                  \
        if (flag_s[1] != 0) {                                                                                             \
            if (threadIdx.x == 0) __hip_atomic_store(G.bar + 8, 1ULL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);        \
            return;                                                                                                       \
        }                                                                                                                 \
    } while (0)

}  // namespace rt
