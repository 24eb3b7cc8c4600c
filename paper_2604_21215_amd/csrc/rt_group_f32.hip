// Grouped single-launch engine of the sequential loop, fp32 storage (d = 128, 256 or 384, F = 4 d).
//
// rt_group.hip's scheme for small fp32 layers: the chip's 256 workgroups form eight groups of 32 (one XCD each; d = 384: four
// groups of 64 on two), every group holds the whole layer and runs the loop for its own sequences.  Everything stays fp32:
// weights in LDS, W2's in registers (11 d^2 * 4 bytes over the group's workgroups: 22 / 88 / 99 KB each), one fp32 value per exchanged word, products with
// v_mfma_f32_4x4x1_16b_f32 (fp32 operands and accumulation), exact erf and expf.
//
// What bounds it: five exchanges per position.  The launch-per-position engine it replaces (rt_stepwise.hip, which keeps every
// other shape, parameter and RT_FLAG_HIP_GRAPH) spends six dependent launches on one.
// Measured (ms per call, launches per position / here): d = 128, B = 1, N = 256: 7.9 / 1.8, N = 2000: 64 / 15.4; d = 256, B = 4, N = 512:
// 19.1 / 4.5; d = 256, B = 32, N = 300: 43 / 3.0; d = 384, B = 3, N = 300: 10.8 / 3.0.  Distance from fp64 as before or smaller (y 1.0e-7
// at d = 256, N = 290; launches 1.3e-7 at N = 150).
#include "rt_group.h"
#include "rt_group_device.h"

#include <cstdlib>
#include <mutex>

namespace rt {

constexpr int kF32Levels = 16;     // stored-partial levels of a query
constexpr int kF32Slot = 3 * 64 + 2 * 20 + kF32Levels * 64;
// Blocks of at least this many keys are spread over the group, between two fenced barriers.  ms per call with 64 / 128 / never:
// d = 128, N = 256 1.78 / 1.87 / 1.97; d = 256, B = 4, N = 512 4.51 / 4.61 / 5.41; d = 128, N = 2000 15.4 / 15.8 / 36.9
constexpr int kF32SpreadP = 64;
constexpr int kF32Tile = 8;        // outputs of a tile

constexpr int f32_ranks(int D) { return D <= 2 ? 32 : 64; }    // workgroups of a group, D = d / 128
constexpr int f32_rows(int D) { return 128 * D / f32_ranks(D); }                 // rows of Wo and W2 per workgroup: 4, 8, 6
constexpr int f32_tiles(int rows) { return (rows + kF32Tile - 1) / kF32Tile; }
constexpr int f32_chunks(int len) { return (len + 31) / 32; }  // chunks of 32 contraction indices in a wavefront's share
constexpr int f32_frags_o(int D) { return f32_tiles(f32_rows(D)) * kPW * f32_chunks(16 * D); }
constexpr int f32_frags_1(int D) { return f32_tiles(4 * f32_rows(D)) * kPW * f32_chunks(16 * D); }
constexpr int f32_frags_2(int D) { return f32_tiles(f32_rows(D)) * kPW * f32_chunks(64 * D); }
constexpr int f32_frags_kv(int D) { return f32_tiles(2 * f32_rows(D)) * kPW * f32_chunks(16 * D); }
constexpr int f32_frags_lds(int D) { return f32_frags_o(D) + f32_frags_1(D) + f32_frags_kv(D); }   // W2 follows, kept in registers
constexpr int f32_frags_all(int D) { return f32_frags_lds(D) + f32_frags_2(D); }

struct F32Args {
    int B, N, H, BH, groups;
    int log2_pmin, slots;
    float alpha, scale, eps, alibi;
    int norm_free;
    unsigned tag_base;
    long long spin_limit;
    unsigned long long *bar, *words;
    size_t group_stride;
    const float4 *packed;
    const float *g_k, *x, *Q, *Kt, *Vt;
    float *y, *K, *V, *pm, *pl, *po;
};
// words of one group and parity for BM sequences: a, h, z, u, kv, zss
__host__ __device__ inline size_t f32_words(int d, int BM, size_t *at)
{
    const size_t v = (size_t)BM * d;
    at[0] = 0; at[1] = v; at[2] = 2 * v; at[3] = 3 * v; at[4] = 7 * v; at[5] = 9 * v;
    return 9 * v + (size_t)BM * 64;
}
// word of element k of batch row b: pieces of two elements, the batch rows side by side
template <int BM> __device__ __forceinline__ unsigned f32_word(unsigned k, unsigned b) { return ((k >> 1) * BM + b) * 2 + (k & 1); }

// This wavefront's share (LEN elements) of an exchanged vector: elements 32 m + 2 (l/4), + 1 of batch row l%4 % BM in act[m][0], act[m][1]
// of lane l, the A operands of two products (the contraction indices may be in any order that the weights share).
template <int NC, int LEN, int BM>
__device__ __forceinline__ void f32_pull(const ll_t *vec, int wave, int lane, int B, unsigned tag, const GroupWait &A, float (&act)[NC][2],
                                         int &fail)
{
    constexpr int CPL = 4 / BM;
    constexpr int NL = (NC + CPL - 1) / CPL;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<ll_t *>(vec) + (size_t)wave * (LEN * BM), 0, LEN * BM * 8, 0x00020000);
    v4u_t v[NL];
    const int b = lane & (BM - 1), p0 = (lane >> 2) + 16 * ((lane & 3) / BM);
    const int off0 = (p0 * BM + b) * 16;
    unsigned need = 0;
#pragma unroll
    for (int n = 0; n < NL; ++n) {
        v[n] = v4u_t{0u, 0u, 0u, 0u};
        if (b < B && n * 32 * CPL + 2 * p0 < LEN) need |= 1u << n;
    }
    long long spins = 0;
    while (__any(need != 0)) {
#pragma unroll
        for (int n = 0; n < NL; ++n)
            if (need & (1u << n)) v[n] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off0 + n * 1024, 0, kAuxAgent);
#pragma unroll
        for (int n = 0; n < NL; ++n)
            if ((need & (1u << n)) && v[n][1] == tag && v[n][3] == tag) need &= ~(1u << n);
        if (++spins > A.spin_limit || ((spins & 255) == 0 && ll_load(A.bar + 8) != 0)) { fail = 1; break; }
    }
#pragma unroll
    for (int m = 0; m < NC; ++m)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const unsigned w = v[m / CPL][2 * e];
            unsigned r = w;
            if (BM == 1) r = (m & 3) == 0 ? w : ((m & 3) == 1 ? quad_move<0x55>(w) : ((m & 3) == 2 ? quad_move<0xAA>(w) : quad_move<0xFF>(w)));
            else if (BM == 2) r = (m & 1) ? quad_move<0xEE>(w) : w;
            act[m][e] = __uint_as_float(r);
        }
}
// Tile of 8 outputs x 32 contraction indices.  CBSZ = 1, ABID = j: the blocks 2q, 2q + 1 take block 2q + j of A, so a lane multiplies
// output lane%8 with the elements of piece 2 (l/8) + j; w = {e 0 j 0, e 0 j 1, e 1 j 0, e 1 j 1}.
__device__ __forceinline__ f32x4_t f32_product(const float (&a)[2], const float4 &w, f32x4_t acc)
{
    acc = __builtin_amdgcn_mfma_f32_4x4x1f32(a[0], w.x, acc, 1, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_4x4x1f32(a[0], w.y, acc, 1, 1, 0);
    acc = __builtin_amdgcn_mfma_f32_4x4x1f32(a[1], w.z, acc, 1, 0, 0);
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a[1], w.w, acc, 1, 1, 0);
}
// products of this wavefront's share with NT tiles -> red[wave][8 tile + lane%8][batch row]
template <int NT, int NC, typename WEIGHT>
__device__ __forceinline__ void f32_tiles_out(WEIGHT weight, const float (&act)[NC][2], float *red, int wave, int lane)
{
    f32x4_t acc[NT][2] = {};
#pragma unroll
    for (int m = 0; m < NC; ++m)
#pragma unroll
        for (int i = 0; i < NT; ++i) acc[i][m & 1] = f32_product(act[m], weight(i, m), acc[i][m & 1]);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        f32x4_t s = acc[i][0] + acc[i][1];
#pragma unroll
        for (int r = 0; r < 4; ++r) {   // the eight groups of eight lanes
            float v = s[r];
            v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xF, 0xF, true));   // row_ror:8
            v = fold1(v, v);
            s[r] = fold2(v, v);
        }
        if (lane < 8) *reinterpret_cast<f32x4_t *>(red + ((size_t)wave * 64 + i * 8 + lane) * 4) = s;
    }
}

// ---- Pre-merge of query t (all but its two newest keys), see rt_group.hip
__device__ __forceinline__ int f32_window(int t) { return t >= 2 ? max(((t - 1) & 31) - 1, 0) : 0; }
__device__ __forceinline__ void f32_fetch(const F32Args &A, int t, int u, float *slot, int lane)
{
    const size_t off = (size_t)t * A.BH * kHeadDim + (unsigned)(u * kHeadDim + lane);
    const float q = A.Q[off], kt = A.Kt[off], vt = A.Vt[off];
    float *sm = slot + 192, *sl = sm + 20, *so = sl + 20;
    int n = 0, bits = t >= 2 ? (t - 1) >> A.log2_pmin : 0;
    for (int lr = 0; bits; ++lr, bits >>= 1) {
        if (!(bits & 1)) continue;
        const size_t idx = partial_index(lr, partial_slot(lr + A.log2_pmin, t - 1), A.slots, A.BH, u);
        const float m = A.pm[idx], l = A.pl[idx], o = A.po[idx * kHeadDim + lane];
        if (lane == 0) { sm[n] = m; sl[n] = l; }
        so[n * 64 + lane] = o;
        ++n;
    }
    slot[lane] = q; slot[64 + lane] = kt; slot[128 + lane] = vt;
}
__device__ __forceinline__ void f32_merge(const F32Args &A, int t, int u, const float *slot, const float *wk, const float *wv, float *out, int lane)
{
    const float *sm = slot + 192, *sl = sm + 20, *so = sl + 20;
    const float q = slot[lane];
    const float s0 = A.scale * fast_sum(q * slot[64 + lane]);
    const int n = t >= 2 ? __popc((t - 1) >> A.log2_pmin) : 0, w = f32_window(t);
    float m = s0;
    for (int i = 0; i < n; ++i) m = fmaxf(m, sm[i]);
    float logit = -INFINITY;
    if (w > 0) {
        const bool valid = lane < w;
        const float *krow = wk + (size_t)(valid ? lane : 0) * (kHeadDim + 4);
        float acc[2] = {0.f, 0.f};
#pragma unroll
        for (int c8 = 0; c8 < 8; ++c8) {
            float kk[8];
            load8(krow + c8 * 8, kk);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e & 1] = fmaf(lane_bcast(q, c8 * 8 + e), kk[e], acc[e & 1]);
        }
        const float s = (acc[0] + acc[1]) * A.scale;
        logit = valid ? fmaf(-alibi_slope(A.alibi, u % A.H, A.H), (float)(w + 2 - lane), s) : -INFINITY;
        m = fmaxf(m, fast_max(logit));
    }
    const float e0 = expf(s0 - m);
    float l = e0, o = slot[128 + lane] * e0;
    for (int i = 0; i < n; ++i) {
        const float f = expf(sm[i] - m);
        l = fmaf(sl[i], f, l);
        o = fmaf(so[i * 64 + lane], f, o);
    }
    if (w > 0) {
        const float p = expf(logit - m);
        l += fast_sum(p);
        for (int j0 = 0; j0 < w; j0 += 8) {
            float vv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) vv[e] = wv[(size_t)min(j0 + e, w - 1) * kHeadDim + lane];
#pragma unroll
            for (int e = 0; e < 8; ++e) o = fmaf(lane_bcast(p, j0 + e), vv[e], o);
        }
    }
    out[lane] = q; out[64 + lane] = m; out[128 + lane] = l; out[192 + lane] = o;
}

// D = d / 128, BM: sequences per group the exchanged vectors are laid out for (1 or 4)
template <int D, int BM>
__global__ __launch_bounds__(kPThreads) void group_f32_kernel(F32Args A)
{
    constexpr int d = 128 * D, RANKS = f32_ranks(D), RO = f32_rows(D), R1 = 4 * RO, RKV = 2 * RO;
    constexpr int LD = d / kPW, LF = 4 * d / kPW, CD = f32_chunks(LD), CF = f32_chunks(LF);
    constexpr int TO = f32_tiles(RO), T1 = f32_tiles(R1), TKV = f32_tiles(RKV);
    static_assert(8 * T1 <= 64 && 4 * RO <= 64, "one wavefront finishes phases O and 2; a tile row per lane of the partial sums");
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int xcd = blockIdx.x & 7;
    const int grp = RANKS == 32 ? xcd : xcd >> 1;
    const int rank = (int)(blockIdx.x >> 3) + (RANKS == 32 ? 0 : (xcd & 1) * 32);
    const int B = (A.B - grp + A.groups - 1) / A.groups;   // sequences grp, grp + groups, ...
    if (B <= 0) return;

    float4 *w_s = reinterpret_cast<float4 *>(smem);
    const float4 *wo_s = w_s, *w1_s = wo_s + f32_frags_o(D) * 64, *wkv_s = w1_s + f32_frags_1(D) * 64;
    float *red0 = reinterpret_cast<float *>(w_s + f32_frags_lds(D) * 64), *red1 = red0 + kPW * 256;
    float *sqh = red1 + kPW * 256;                 // [kPW][4]
    float *xs = sqh + kPW * 4;                     // [16][4]
    int *flag_s = reinterpret_cast<int *>(xs + 64);
    float *win_k = reinterpret_cast<float *>(flag_s + 4);   // [32][64 + 4]
    float *win_v = win_k + 32 * (kHeadDim + 4);    // [32][64]
    float *pre_s = win_v + 32 * kHeadDim, *pre_in = pre_s + 512;

    GroupWait G;
    G.spin_limit = A.spin_limit;
    G.bar = A.bar + grp * 16;
    unsigned long long *words = A.words + grp * A.group_stride;
    size_t at[6];
    const size_t per = f32_words(d, BM, at);
    const float4 *packed = A.packed + (size_t)rank * f32_frags_all(D) * 64;
    for (int i = threadIdx.x; i < f32_frags_lds(D) * 64; i += kPThreads) w_s[i] = packed[i];
    float4 w2[TO * CF];   // this wavefront's share of W2
#pragma unroll
    for (int m = 0; m < TO * CF; ++m) w2[m] = packed[(size_t)(f32_frags_lds(D) + (m / CF * kPW + wave) * CF + m % CF) * 64 + lane];
    if (threadIdx.x == 0) flag_s[1] = 0;

    const size_t rs = (size_t)A.BH * kHeadDim;
    const int units = B * A.H;
    const bool has_u = rank < units;
    const int ub = rank / A.H, uh = rank - ub * A.H;
    const int ug = (grp + A.groups * ub) * A.H + uh;
    const float my_gk = (has_u && A.g_k) ? A.g_k[uh * kHeadDim + lane] : 1.f;
    const float slope = alibi_slope(A.alibi, uh, A.H);
    const bool is_owner = has_u && wave == 0, is_helper = has_u && wave == 4, is_fetcher = has_u && wave == 5;
    const int erow = lane >> 2, eb = lane & 3;     // epilogue rows of wavefront 0 in phases O and 2
    const bool e_own = erow < RO && eb < B;
    const size_t e_off = (size_t)(grp + A.groups * eb) * A.N * d + rank * RO + erow;
    float s1 = 0.f, v1 = 0.f;
    unsigned long long nbar = 0;

    __syncthreads();
    if (is_helper) {
        f32_fetch(A, 0, ug, pre_in, lane);
        wave_sync_lds();
        f32_merge(A, 0, ug, pre_in, win_k, win_v, pre_s, lane);
    }
    __syncthreads();

    auto phase_m = [&](int t, int &fail) {
        const int par = t & 1, ppar = par ^ 1;
        const unsigned tag = A.tag_base | (unsigned)(t + 1), ptag = A.tag_base | (unsigned)t;
        if (is_owner) {
            const float *st = pre_s + par * 256;
            const float q = st[lane];
            float m = st[64 + lane], l = st[128 + lane], o = st[192 + lane];
            float kr = 0.f, vr = 0.f;
            if (t >= 1) {
                const unsigned long long *wp = words + ppar * per;
                const unsigned ko = uh * kHeadDim + lane, vo = d + ko;
                const ll_t *p[3] = {wp + at[5] + (lane & (RANKS - 1)) * BM + ub, wp + at[4] + (ko / RKV * BM + ub) * RKV + ko % RKV,
                                    wp + at[4] + (vo / RKV * BM + ub) * RKV + vo % RKV};
                const bool act[3] = {lane < RANKS, true, true};
                ll_t w3[3];
                if (((t - 1) & 31) != 0) {   // key t - 2, the newest of the window
                    const float mn = fmaxf(m, s1);
                    const float e1 = expf(m - mn), e2 = expf(s1 - mn);
                    l = l * e1 + e2;
                    o = o * e1 + v1 * e2;
                    m = mn;
                }
                ll_wait_n<3>(p, act, ptag, G, w3, fail);
                const float k0 = __uint_as_float((unsigned)w3[1]);
                const float kg = A.norm_free ? k0 : k0 * my_gk;
                const float Sz = fast_sum(act[0] ? __uint_as_float((unsigned)w3[0]) : 0.f), Sk = fast_sum(k0 * k0), Sq = fast_sum(q * kg);
                const float rz = A.norm_free ? 1.f : rsqrtf(Sz / (float)d + A.eps);
                const float kscale = A.norm_free ? 1.f : rz * rsqrtf(rz * rz * Sk / (float)kHeadDim + A.eps);
                kr = kg * kscale;
                vr = __uint_as_float((unsigned)w3[2]) * rz;
                if (t < A.N) {   // the newest key is one position before the query
                    const float sn = A.scale * (Sq * kscale) - slope;
                    const float m_new = fmaxf(m, sn);
                    const float e1 = expf(m - m_new), e2 = expf(sn - m_new);
                    l = l * e1 + e2;
                    o = o * e1 + vr * e2;
                }
            }
            if (t < A.N)
                word_store(words + par * per + at[0], f32_word<BM>(uh * kHeadDim + lane, ub), tag, __float_as_uint(o / l));
            if (t >= 1) {
                v1 = vr;
                if (t + 1 < A.N && (t & 31) != 0)   // key t - 1 is two positions before query t + 1
                    s1 = A.scale * fast_sum(pre_in[((t + 1) & 1) * kF32Slot + lane] * kr) - 2.f * slope;
                const size_t off = (size_t)(t - 1) * rs + (unsigned)(ug * kHeadDim + lane);
                A.K[off] = kr;
                A.V[off] = vr;
                const int slot = (t - 1) & 31;
                win_k[slot * (kHeadDim + 4) + lane] = kr;
                win_v[slot * kHeadDim + lane] = vr;
            }
        } else if (wave == 1) {
            if (t < A.N && e_own) xs[lane] = A.x[e_off + (size_t)t * d];
        } else if (is_helper) {
            if ((t & 31) != 0 && t + 1 < A.N) f32_merge(A, t + 1, ug, pre_in + ((t + 1) & 1) * kF32Slot, win_k, win_v, pre_s + ppar * 256, lane);
        } else if (is_fetcher) {
            if ((t & 31) != 0 && ((t + 1) & 31) != 0 && t + 2 < A.N) f32_fetch(A, t + 2, ug, pre_in + (t & 1) * kF32Slot, lane);
        }
    };

    int fail = 0;
    phase_m(0, fail);
    RT_GROUP_SYNC(fail);
    for (int t = 0; t < A.N; ++t) {
        if ((t & 31) == 0) {
            if (t > 0 && t < A.N - 1) {
                // The block ending at key t - 1 folded into the next queries, one query per wavefront at a time.
                const int P = t & -t, nq = min(P, A.N - 1 - t);
                int level = A.log2_pmin;
                while ((1 << level) < P) ++level;
                auto query = [&](int u, int j) {
                    const size_t kb = (size_t)(t - P) * rs + (size_t)u * kHeadDim;
                    const float q = A.Q[(size_t)(t + 1 + j) * rs + (unsigned)(u * kHeadDim + lane)];
                    float m = -INFINITY, l = 0.f, o = 0.f;
                    attend_keys<float>(q, A.K + kb, A.V + kb, rs, P, A.scale, m, l, o, nullptr, alibi_slope(A.alibi, u % A.H, A.H), P + 1 + j);
                    const size_t idx = partial_index(level - A.log2_pmin, partial_slot(level, t + j), A.slots, A.BH, u);
                    if (lane == 0) { A.pm[idx] = m; A.pl[idx] = l; }
                    A.po[idx * kHeadDim + lane] = o;
                };
                if (P < kF32SpreadP) {   // the owner of the (b, h) wrote its keys and values and reads the states itself
                    if (has_u) {
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                        __syncthreads();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                        for (int j = wave; j < nq; j += kPW) query(ug, j);
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                        __syncthreads();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                    }
                } else {                 // all wavefronts of the group
                    if (grid_barrier(G, (++nbar) * (unsigned long long)RANKS, flag_s)) fail = 1;
                    RT_GROUP_SYNC(fail);
                    for (int i = rank * kPW + wave; i < units * nq; i += RANKS * kPW) {
                        const int ul = i % units, lb = ul / A.H;
                        query((grp + A.groups * lb) * A.H + ul - lb * A.H, i / units);
                    }
                    if (grid_barrier(G, (++nbar) * (unsigned long long)RANKS, flag_s)) fail = 1;
                    RT_GROUP_SYNC(fail);
                }
            }
            if (is_helper && t + 1 < A.N) {
                f32_fetch(A, t + 1, ug, pre_in + ((t + 1) & 1) * kF32Slot, lane);
                wave_sync_lds();
                f32_merge(A, t + 1, ug, pre_in + ((t + 1) & 1) * kF32Slot, win_k, win_v, pre_s + ((t + 1) & 1) * 256, lane);
            } else if (is_fetcher && t + 2 < A.N) {
                f32_fetch(A, t + 2, ug, pre_in + (t & 1) * kF32Slot, lane);
            }
        }
        const unsigned tag = A.tag_base | (unsigned)(t + 1);
        unsigned long long *wp = words + (t & 1) * per;
        // ---- phase O:  h = x_t + alpha Wo a
        {
            float act[CD][2];
            f32_pull<CD, LD, BM>(wp + at[0], wave, lane, B, tag, G, act, fail);
            f32_tiles_out<TO, CD>([&](int i, int m) { return wo_s[((i * kPW + wave) * CD + m) * 64 + lane]; }, act, red0, wave, lane);
        }
        RT_GROUP_SYNC(fail);
        float hv = 0.f;
        if (wave == 0) {
            hv = xs[lane] + A.alpha * tile_sum(red0, lane);
            if (e_own) word_store(wp + at[1], f32_word<BM>(rank * RO + erow, eb), tag, __float_as_uint(hv));
        }
        __syncthreads();
        // ---- phase 1:  u = gelu(W1 h / rms(h))
        {
            float act[CD][2];
            f32_pull<CD, LD, BM>(wp + at[1], wave, lane, B, tag, G, act, fail);
            f32_tiles_out<T1, CD>([&](int i, int m) { return w1_s[((i * kPW + wave) * CD + m) * 64 + lane]; }, act, red1, wave, lane);
            float ss = 0.f;
#pragma unroll
            for (int m = 0; m < CD; ++m) {
                // (a share that ends inside a chunk: the lanes beyond it hold zeros or, moved from other lanes, elements that are not this chunk's)
                const bool in = 32 * (m + 1) <= LD || 32 * m + 2 * (lane >> 2) < LD;
                if (in) ss = fmaf(act[m][0], act[m][0], fmaf(act[m][1], act[m][1], ss));
            }
            ss = sum_mod4(ss);
            if (lane < 4) sqh[wave * 4 + lane] = ss;
        }
        RT_GROUP_SYNC(fail);
        for (int e = threadIdx.x; e < R1 * 4; e += kPThreads) {
            const int row = e >> 2, b = e & 3;
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < kPW; ++w) s += sqh[w * 4 + b];
            const float rinv = A.norm_free ? 1.f : rsqrtf(s / (float)d + A.eps);
            const float uv = gelu_erf(tile_sum(red1, e) * rinv);
            if (b < B) word_store(wp + at[3], f32_word<BM>(rank * R1 + row, b), tag, __float_as_uint(uv));
        }
        __syncthreads();
        // ---- phase 2:  z = h + alpha W2 u
        {
            float act[CF][2];
            f32_pull<CF, LF, BM>(wp + at[3], wave, lane, B, tag, G, act, fail);
            f32_tiles_out<TO, CF>([&](int i, int m) { return w2[i * CF + m]; }, act, red0, wave, lane);
        }
        RT_GROUP_SYNC(fail);
        if (wave == 0) {
            const float zv = hv + A.alpha * tile_sum(red0, lane);
            if (e_own) word_store(wp + at[2], f32_word<BM>(rank * RO + erow, eb), tag, __float_as_uint(zv));
            const float s = sum_mod4(e_own ? zv * zv : 0.f);
            if (lane < B) word_store(wp + at[5], rank * BM + lane, tag, __float_as_uint(s));
            if (e_own) A.y[e_off + (size_t)t * d] = zv;
        }
        __syncthreads();
        // ---- phase KV:  [Wk; Wv] (z g_kv)
        {
            float act[CD][2];
            f32_pull<CD, LD, BM>(wp + at[2], wave, lane, B, tag, G, act, fail);
            f32_tiles_out<TKV, CD>([&](int i, int m) { return wkv_s[((i * kPW + wave) * CD + m) * 64 + lane]; }, act, red1, wave, lane);
        }
        RT_GROUP_SYNC(fail);
        if (threadIdx.x < RKV * 4) {
            const int row = (int)threadIdx.x >> 2, b = lane & 3;
            if (b < B) word_store(wp + at[4], (rank * BM + b) * RKV + row, tag, __float_as_uint(tile_sum(red1, threadIdx.x)));
        }
        phase_m(t + 1, fail);
        RT_GROUP_SYNC(fail);
    }
}

// The loop matrices in fragment order, gains folded in: lane l of fragment (tile, wavefront, chunk m) holds the elements
// 32 m + 2 p + e, p = 2 (l/8) + j, of the wavefront's share of row 8 tile + l%8, as {e 0 j 0, e 0 j 1, e 1 j 0, e 1 j 1}.
__global__ __launch_bounds__(256) void group_f32_pack_kernel(const float *Wo, const float *W1, const float *W2, const float *Wk, const float *Wv,
                                                             const float *g_mlp, const float *g_kv, int D, float4 *dst)
{
    const int d = 128 * D, per = f32_frags_all(D), RO = f32_rows(D);
    const int f_all = (int)((blockIdx.x * 256 + threadIdx.x) >> 6), lane = threadIdx.x & 63;
    if (f_all >= per * f32_ranks(D)) return;
    const int rank = f_all / per;
    int f = f_all - rank * per, rows = RO, K = d;
    const float *src = nullptr, *gain = nullptr;
    bool pairs = false;
    if (f < f32_frags_o(D)) { src = Wo; }
    else if ((f -= f32_frags_o(D)) < f32_frags_1(D)) { src = W1; rows = 4 * RO; gain = g_mlp; }
    else if ((f -= f32_frags_1(D)) < f32_frags_kv(D)) { rows = 2 * RO; gain = g_kv; pairs = true; }
    else { f -= f32_frags_kv(D); src = W2; K = 4 * d; }
    const int len = K / kPW, chunks = f32_chunks(len), m = f % chunks, w = f / chunks % kPW, tile = f / (chunks * kPW);
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (tile * 8 + (lane & 7) < rows) {
        int row = rank * rows + tile * 8 + (lane & 7);
        if (pairs) { src = row < d ? Wk : Wv; row = row < d ? row : row - d; }
        for (int i = 0; i < 4; ++i) {
            const int e = i >> 1, j = i & 1, kk = 32 * m + 2 * (2 * (lane >> 3) + j) + e;
            if (kk < len) v[i] = src[(size_t)row * K + w * len + kk] * (gain ? gain[w * len + kk] : 1.f);
        }
    }
    dst[(size_t)f_all * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
}

// =============================================================================================
// Host side
// =============================================================================================
__global__ void group_f32_clear_kernel(unsigned long long *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0ULL;
}

typedef void (*f32_fn)(F32Args);
static f32_fn pick_kernel(int d, int BM)
{
    switch (d) {
    case 128: return BM == 1 ? group_f32_kernel<1, 1> : group_f32_kernel<1, 4>;
    case 256: return BM == 1 ? group_f32_kernel<2, 1> : group_f32_kernel<2, 4>;
    case 384: return BM == 1 ? group_f32_kernel<3, 1> : group_f32_kernel<3, 4>;
    default: return nullptr;
    }
}
static size_t lds_bytes(int D)
{
    return (size_t)f32_frags_lds(D) * 1024 + (2 * kPW * 256 + kPW * 4 + 64 + 4 + 32 * (kHeadDim + 4) + 32 * kHeadDim + 512 + 2 * kF32Slot) * 4;
}
static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

rt_status group_f32_create(GroupF32State &P, const rt_config &cfg, const LayerDims &D)
{
    P.available = false;
    if (cfg.dtype != RT_F32 || (cfg.flags & RT_FLAG_NO_MFMA) || D.F != 4 * D.d || !pick_kernel(D.d, 1) || D.p_min != 32)
        return RT_ERR_UNSUPPORTED;
    int cus = 0, coop = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, cfg.device) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, cfg.device) != hipSuccess)
        return RT_ERR_HIP;
    if (cus != 256 || !coop) return RT_ERR_UNSUPPORTED;
    const int D1 = D.d / 128;
    P.groups = 256 / f32_ranks(D1);
    P.lds = lds_bytes(D1);
    if (P.lds > (size_t)160 * 1024) return RT_ERR_UNSUPPORTED;
    {   // once per device and kernel
        static std::mutex mu;
        static uint64_t raised[4] = {};
        std::lock_guard<std::mutex> lock(mu);
        const uint64_t bit = 1ULL << (cfg.device & 63);
        for (int BM = 1; BM <= 4 && !(raised[D1] & bit); BM += 3)
            if (hipFuncSetAttribute((const void *)pick_kernel(D.d, BM), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) {
                (void)hipGetLastError();
                return RT_ERR_UNSUPPORTED;
            }
        raised[D1] |= bit;
    }
    const int most = 4 * P.groups;
    P.max_batch = cfg.max_batch < most ? cfg.max_batch : most;
    size_t at[6], off = 0;
    auto carve = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    const size_t o_bar = carve((size_t)P.groups * 16 * 8);
    P.group_stride = align_up(2 * f32_words(D.d, 4, at), 32);
    const size_t o_w = carve(P.group_stride * P.groups * 8);
    P.exchange_bytes = off;
    const size_t o_p = carve((size_t)f32_frags_all(D1) * f32_ranks(D1) * 1024);
    P.slab_bytes = off;
    if (hipMalloc(&P.slab, P.slab_bytes) != hipSuccess) {
        (void)hipGetLastError();
        P.slab = nullptr; P.slab_bytes = 0;
        return RT_ERR_OOM;
    }
    if (hipMemset(P.slab, 0, P.exchange_bytes) != hipSuccess) {
        (void)hipFree(P.slab);
        P.slab = nullptr;
        return RT_ERR_HIP;
    }
    P.bar = (unsigned long long *)((char *)P.slab + o_bar);
    P.words = (unsigned long long *)((char *)P.slab + o_w);
    P.packed = (char *)P.slab + o_p;
    const char *sl = getenv("RT_SPIN_LIMIT");
    P.spin_limit = sl ? atoll(sl) : (1LL << 21);
    if (P.spin_limit < 1) P.spin_limit = 1;
    P.available = true;
    return RT_OK;
}

void group_f32_destroy(GroupF32State &P)
{
    if (P.slab) (void)hipFree(P.slab);
    P.slab = nullptr;
    P.available = false;
}

bool group_f32_supported(const GroupF32State &P, const LayerDims &D)
{
    // the first positions do not pay for laying out the weights (us per call, launches per position / here, B = 2): N = 1 54 / 63, 73 / 87 and
    // 93 / 127 at d = 128, 256, 384; N = 2 88 / 70, 106 / 95 and 124 / 136; N = 3, d = 384 155 / 144
    return P.available && D.B <= P.max_batch && D.N >= (D.d == 384 ? 3 : 2) && D.N < (1 << 20) - 2;
}

rt_status group_f32_prefill(GroupF32State &P, const LayerDims &D, const Weights &W, const Scratch &S, const void *x, void *y, void *K, void *V,
                            hipStream_t st, std::string &err)
{
    auto hip_fail = [&](hipError_t e, const char *where) {
        err = std::string(where) + ": " + hipGetErrorString(e);
        return RT_ERR_HIP;
    };
    const int D1 = D.d / 128, frags = f32_frags_all(D1) * f32_ranks(D1);
    hipLaunchKernelGGL(group_f32_pack_kernel, dim3((unsigned)((frags + 3) / 4)), dim3(256), 0, st, (const float *)W.Wo, (const float *)W.W1,
                       (const float *)W.W2, (const float *)W.Wk, (const float *)W.Wv, D.norm_free ? nullptr : (const float *)W.g_mlp,
                       D.norm_free ? nullptr : (const float *)W.g_kv, D1, (float4 *)P.packed);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "group_f32_pack_kernel");
    // tags as in rt_group.hip: 1 .. 4094 in turn, words cleared when the number wraps; a captured launch has a number of its own
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    if (st && (e = hipStreamIsCapturing(st, &capturing)) != hipSuccess) return hip_fail(e, "hipStreamIsCapturing");
    const bool captured = capturing != hipStreamCaptureStatusNone;
    if (!captured) P.nonce = (P.nonce % 4094u) + 1u;
    const bool all = captured || (P.nonce == 1u && P.launched);
    hipLaunchKernelGGL(group_f32_clear_kernel, dim3(all ? 64 : 1), dim3(256), 0, st, P.bar, all ? P.exchange_bytes / 8 : (size_t)P.groups * 16);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "group_f32_clear_kernel");
    F32Args A = {};
    A.B = D.B; A.N = D.N; A.H = D.H; A.BH = D.B * D.H; A.groups = P.groups;
    A.log2_pmin = D.log2_pmin; A.slots = S.slots;
    A.alpha = D.alpha; A.scale = D.scale; A.eps = D.eps; A.alibi = D.alibi; A.norm_free = D.norm_free;
    A.tag_base = (captured ? 4095u : P.nonce) << 20;
    A.spin_limit = P.spin_limit; A.bar = P.bar; A.words = P.words; A.group_stride = P.group_stride;
    A.packed = (const float4 *)P.packed;
    A.g_k = (const float *)W.g_k; A.x = (const float *)x; A.Q = (const float *)S.Q; A.Kt = (const float *)S.Kt; A.Vt = (const float *)S.Vt;
    A.y = (float *)y; A.K = (float *)K; A.V = (float *)V; A.pm = S.pm; A.pl = S.pl; A.po = S.po;
    void *args[] = {&A};
    e = hipLaunchCooperativeKernel((const void *)pick_kernel(D.d, D.B <= P.groups ? 1 : 4), dim3(256), dim3(kPThreads), args,
                                   (unsigned int)P.lds, st);
    if (e != hipSuccess) return hip_fail(e, "hipLaunchCooperativeKernel");
    P.launched = true;
    return RT_OK;
}

int group_f32_wait_expired(GroupF32State &P)
{
    if (!P.slab || !P.launched) return 0;
    unsigned long long v[8 * 16];
    if (hipMemcpy(v, P.bar, (size_t)P.groups * 16 * 8, hipMemcpyDeviceToHost) != hipSuccess) return -1;
    for (int g = 0; g < P.groups; ++g)
        if (v[g * 16 + 8] != 0) return 1;
    return 0;
}

}  // namespace rt
