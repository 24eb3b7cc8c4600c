// Device helpers shared by the grouped engines (rt_group.hip, rt_group_f32.hip, rt_backward_persistent.hip).
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

// word of element pair (k, k + 1), k even, of batch row b: 16-byte pieces of four elements, runs of RUN pieces per batch row
template <int RUN, int BM> __device__ __forceinline__ unsigned piece_word(unsigned k, unsigned b)
{
    const unsigned p = k >> 2;
    return (((p / RUN) * BM + b) * RUN + p % RUN) * 2 + ((k >> 1) & 1);
}

// Operands of v_mfma_f32_4x4x4_16b_bf16 (16 blocks, block i = lanes 4i .. 4i+3): A: lane holds A[row = lane%4][k = 0..3] of
// its block, B: lane holds B[k = 0..3][col = lane%4], D: register r holds D[row r][col = lane%4].  Rows are the batch rows,
// columns the outputs.  With CBSZ = 2, ABID = j the blocks 4q .. 4q+3 all take block 4q + j of A: one instruction multiplies
// 16 outputs (16 t + lane%16) by 16 contraction indices, four in each row q of 16 lanes.
typedef short s16x4_t __attribute__((ext_vector_type(4)));
union Piece {
    uint2 u;
    s16x4_t v;
};
union WFrag {
    uint4 u;
    uint2 h[2];
};

// What the loads of a pull brought -> the A operands: with fewer than four batch rows by moves inside the four lanes of a block.
template <int BM, int NC, int NL> __device__ __forceinline__ void rows_in_place(const v4u_t (&v)[NL], Piece (&act)[NC])
{
    constexpr int CPL = 4 / BM;
#pragma unroll
    for (int m = 0; m < NC; ++m) {
        const unsigned lo = v[m / CPL][0], hi = v[m / CPL][2];
        if (BM == 4) act[m].u = make_uint2(lo, hi);
        else if (BM == 2) act[m].u = m & 1 ? make_uint2(quad_move<0xEE>(lo), quad_move<0xEE>(hi)) : make_uint2(lo, hi);
        else if ((m & 3) == 0) act[m].u = make_uint2(lo, hi);
        else if ((m & 3) == 1) act[m].u = make_uint2(quad_move<0x55>(lo), quad_move<0x55>(hi));
        else if ((m & 3) == 2) act[m].u = make_uint2(quad_move<0xAA>(lo), quad_move<0xAA>(hi));
        else act[m].u = make_uint2(quad_move<0xFF>(lo), quad_move<0xFF>(hi));
    }
}

// This wavefront's share (NC chunks of 64 elements, LEN elements in all) of an exchanged vector of BM batch rows: act[m] of lane l
// holds elements 64 m + 4 (l/4) .. + 3 of batch row l%4 % BM - the A operand of the product, nothing is staged in LDS.  With
// fewer than four batch rows the lanes of the unused rows fetch the pieces of the chunks that follow, and a move inside the
// four lanes of a block brings them where they belong.
template <int NC, int LEN, int RUN, int BM>
__device__ __forceinline__ void slice_pull(const ll_t *vec, int wave, int lane, int B, unsigned tag, const GroupWait &A, Piece (&act)[NC],
                                           int &fail, int units)
{
    constexpr int CPL = 4 / BM;                  // chunks per load
    constexpr int NL = (NC + CPL - 1) / CPL;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<ll_t *>(vec) + (size_t)wave * (LEN * BM / 2), 0, LEN * BM * 4, 0x00020000);
    v4u_t v[NL];
    const int b = lane & (BM - 1), p0 = (lane >> 2) + 16 * ((lane & 3) / BM);   // piece of the load's first chunk, batch row
    const int off0 = ((p0 / RUN * BM + b) * RUN + p0 % RUN) * 16;               // a load is 1 KB in either layout
    unsigned need = 0;
#pragma unroll
    for (int n = 0; n < NL; ++n) {
        v[n] = v4u_t{0u, 0u, 0u, 0u};
        if (b < B && ((n + 1) * 64 * CPL <= LEN || n * 64 * CPL + 4 * p0 < LEN)) need |= 1u << n;
    }
    long long spins = 0;
    for (int i = 0; i < units; ++i) __builtin_amdgcn_s_sleep(4);
    while (__any(need != 0)) {
#pragma unroll
        for (int n = 0; n < NL; ++n)
            if (need & (1u << n)) v[n] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off0 + n * 1024, 0, kAuxAgent);
#pragma unroll
        for (int n = 0; n < NL; ++n)
            if ((need & (1u << n)) && v[n][1] == tag && v[n][3] == tag) need &= ~(1u << n);
        if (++spins > A.spin_limit || ((spins & 255) == 0 && ll_load(A.bar + 8) != 0)) { fail = 1; break; }
    }
    rows_in_place<BM, NC, NL>(v, act);
}

// The same for a vector of which bf16 heads and bf16 remainders are exchanged (the remainders lie lo_words behind the heads), and,
// with SUMS, the producers' partial sums of squares: 64 words of each batch row, of which this wavefront takes eight; lanes below
// BM hold their sum.
template <int NC, int LEN, int RUN, int BM, bool SUMS>
__device__ __forceinline__ void slice_pull_split(const ll_t *vec, unsigned lo_words, const ll_t *sums, int wave, int lane, int B, unsigned tag,
                                                 const GroupWait &A, Piece (&hi)[NC], Piece (&lo)[NC], float &ss, int &fail, int units)
{
    constexpr int CPL = 4 / BM;
    constexpr int NL = (NC + CPL - 1) / CPL;
    const int lo_off = (int)(lo_words * 8u);
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<ll_t *>(vec) + (size_t)wave * (LEN * BM / 2), 0,
                                                                          lo_off + LEN * BM * 4, 0x00020000);
    v4u_t vh[NL], vl[NL];
    ll_t sw = 0;
    const int b = lane & (BM - 1), p0 = (lane >> 2) + 16 * ((lane & 3) / BM);
    const int off0 = ((p0 / RUN * BM + b) * RUN + p0 % RUN) * 16;
    const ll_t *sp = sums + (wave * 8 * BM + (lane & (8 * BM - 1)));
    unsigned need = 0;
#pragma unroll
    for (int n = 0; n < NL; ++n) {
        vh[n] = vl[n] = v4u_t{0u, 0u, 0u, 0u};
        if (b < B && ((n + 1) * 64 * CPL <= LEN || n * 64 * CPL + 4 * p0 < LEN)) need |= 0x10001u << n;
    }
    if (SUMS && lane < 8 * BM && b < B) need |= 0x8000u;
    static_assert(NL <= 15, "bit 15 is the sums'");
    long long spins = 0;
    for (int i = 0; i < units; ++i) __builtin_amdgcn_s_sleep(4);
    while (__any(need != 0)) {
#pragma unroll
        for (int n = 0; n < NL; ++n) {
            if (need & (1u << n)) vh[n] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off0 + n * 1024, 0, kAuxAgent);
            if (need & (0x10000u << n)) vl[n] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off0 + n * 1024, lo_off, kAuxAgent);
        }
        if (SUMS && (need & 0x8000u)) sw = ll_load(sp);
#pragma unroll
        for (int n = 0; n < NL; ++n) {
            if ((need & (1u << n)) && vh[n][1] == tag && vh[n][3] == tag) need &= ~(1u << n);
            if ((need & (0x10000u << n)) && vl[n][1] == tag && vl[n][3] == tag) need &= ~(0x10000u << n);
        }
        if (SUMS && (need & 0x8000u) && (unsigned)(sw >> 32) == tag) need &= ~0x8000u;
        if (++spins > A.spin_limit || ((spins & 255) == 0 && ll_load(A.bar + 8) != 0)) { fail = 1; break; }
    }
    rows_in_place<BM, NC, NL>(vh, hi);
    rows_in_place<BM, NC, NL>(vl, lo);
    if (SUMS) {
        ss = lane < 8 * BM && b < B ? __uint_as_float((unsigned)sw) : 0.f;
        ss += __shfl_xor(ss, BM, 64);
        ss += __shfl_xor(ss, 2 * BM, 64);
        ss += __shfl_xor(ss, 4 * BM, 64);
    }
}
template <int J> __device__ __forceinline__ f32x4_t mfma4(const Piece &a, const uint2 &w, f32x4_t c)
{
    Piece b;
    b.u = w;
    return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(a.v, b.v, c, 2, J, 0);
}
// one tile's 64 contraction indices of a chunk, one accumulator per J
__device__ __forceinline__ void chunk_product4(const Piece &a, const WFrag &w0, const WFrag &w1, f32x4_t (&acc)[4])
{
    acc[0] = mfma4<0>(a, w0.h[0], acc[0]);
    acc[1] = mfma4<1>(a, w0.h[1], acc[1]);
    acc[2] = mfma4<2>(a, w1.h[0], acc[2]);
    acc[3] = mfma4<3>(a, w1.h[1], acc[3]);
}
__device__ __forceinline__ f32x4_t chunk_product(const Piece &a, const WFrag &w0, const WFrag &w1, f32x4_t acc)
{
    acc = mfma4<0>(a, w0.h[0], acc);
    acc = mfma4<1>(a, w0.h[1], acc);
    acc = mfma4<2>(a, w1.h[0], acc);
    return mfma4<3>(a, w1.h[1], acc);
}
// partial products of NT tiles -> red[wave][16 tile + lane%16][batch row]
template <int NT> __device__ __forceinline__ void tiles_store(float *red, int wave, int lane, const f32x4_t (&acc)[NT])
{
    f32x4_t s;
    const int q = lane >> 4;
    int tile;
    if (NT == 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) { const float v = fold2(acc[0][r], acc[0][r]); s[r] = fold1(v, v); }
        tile = q == 0 ? 0 : NT;
    } else if (NT == 2) {
#pragma unroll
        for (int r = 0; r < 4; ++r) { const float v = fold2(acc[0][r], acc[NT - 1][r]); s[r] = fold1(v, v); }
        tile = q == 0 ? 0 : (q == 2 ? 1 : NT);
    } else {   // rows hold tiles 0, 2, 1, 3
#pragma unroll
        for (int r = 0; r < 4; ++r)
            s[r] = fold1(fold2(acc[0][r], acc[1][r]), fold2(acc[NT > 2 ? 2 : 0][r], NT > 3 ? acc[NT - 1][r] : 0.f));
        tile = q == 1 ? 2 : (q == 2 ? 1 : q);
    }
    if (tile < NT) *reinterpret_cast<f32x4_t *>(red + ((size_t)wave * 64 + tile * 16 + (lane & 15)) * 4) = s;
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
