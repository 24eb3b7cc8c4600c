// The reverse loop of the backward pass (paper Sec. 6.4) as a single launch per block of 32 positions, bf16 storage: the
// structure of the forward's grouped engine (rt_group.hip) applied to the transposed chain.
//
// Per position i the loop has to take the complete gradient of the persistent pair (dK_i, dV_i) back to the attention
// output of that position:
//     d_rz = Wk^T dkraw + Wv^T dV_i                     dkraw = per-head normalisation backward of dK_i
//     Gz   = gy_i + RMS-backward_z(d_rz)                (gradient of z_i)
//     dpre = gelu'(pre_i) * (W2^T alpha Gz)
//     t1   = W1^T dpre,   dh = Gz + RMS-backward_h(t1)
//     dc   = Wo^T alpha dh                              -> softmax backward of query i, which adds to dK_j, dV_j, j < i
// Sequences are independent: four groups of 64 workgroups (two XCDs each) run the loop for up to two sequences each.  A group
// holds the four transposed matrices (11 d^2 elements): Wo^T and [Wk^T | Wv^T] in LDS, W2^T and W1^T in registers as
// matrix-core fragments; the vectors between the products cross the chip in self-validating words (rt_ll.h) and are matrix
// operands as they arrive.  An RMS backward needs a sum over the whole row, dot = <unit, w>, which would cost an exchange of its
// own; instead it is applied AFTER the next product, which is linear in it:
//     W (base + r (w - unit dot / d)) = W base + r (W w - (dot / d) W unit),
// where W base and W unit (base = gy_i or, for dh, the terms of Gz; unit = the normalised z_i or h_i) do not depend on the
// loop and are formed for all positions by batched products before it (A_gy, A_uz = W2^T gy, W2^T unit_z; C_gy, C_uz,
// C_uh = Wo^T gy, Wo^T unit_z, Wo^T unit_h), and every workgroup forms dot itself from the vector it has just pulled.
// Five exchanges per position:
//   U    per (b, h) wavefront: dK_i, dV_i (complete) -> dkraw                                   -> [dkraw | dV_i]
//   G1   d_rz rows = [Wk^T | Wv^T] [dkraw; dV_i];  w = d_rz g_kv                                 -> w
//   G2   dot = <unit_z, w>;  W2^T w and Wo^T w;  dpre rows                                       -> dpre;   Gz rows
//   G3   t1 rows = W1^T dpre;  w2 = t1 g_mlp                                                     -> w2
//   G4   dot2 = <unit_h, w2>;  Wo^T w2;  dc rows, dh rows                                        -> dc
//   A    per (b, h) wavefront: softmax backward of query i: its own temporary pair (dq, dk_tmp, dv_tmp of the row) and
//        the keys of its block before it, whose K, V rows and dK, dV accumulators this workgroup keeps in LDS.
// A launch covers the positions of ONE block of 32 (i_hi down to i_lo): the keys before the block receive this block's
// queries through Algorithm 1's tiles run backwards (bw_event_kernel), which are ordinary launches between two of these.
// Every wait is bounded (spin limit -> abort word -> every workgroup leaves).
//
// What bounds it: the chain of exchanges.  A launch of 32 positions takes 319 us at d = 1024, B = 8 (10 us per position), 655 us as one
// group of 256 workgroups with W1^T's contraction split in four (six exchanges); backward pass of 2048 positions 42.3 -> 27.0 ms,
// B = 1: 36.2 -> 21.3 ms; d = 768, B = 3, N = 1000: 17.7 -> 11.0 ms.
#include "rt_backward_persistent.h"
#include "rt_group_device.h"
#include <cstdlib>
#include <cstring>
#include <mutex>

namespace rt {

constexpr int kBwpBlock = 32;          // positions per launch = the block below which queries reach keys directly
constexpr int kWinLd = kHeadDim + 4;   // row stride of the window tiles in floats
constexpr int kBwpGroups = 4, kBwpRanks = 64, kBwpRows = 2;

// fragments of one workgroup (1 KB: 64 lanes x 16 bytes): [Wo^T | Wk^T Wv^T | W2^T | W1^T], see rt_group.hip
constexpr int bwp_chunks_d(int KSD) { return (KSD + 1) / 2; }
constexpr int bwp_frags_o(int KSD) { return kPW * bwp_chunks_d(KSD) * 2; }
constexpr int bwp_frags_kv(int KSD) { return kPW * KSD * 2; }
constexpr int bwp_frags_2(int KSD) { return KSD * kPW * bwp_chunks_d(KSD) * 2; }
constexpr int bwp_frags_1(int KSD) { return kPW * 2 * KSD * 2; }
constexpr int bwp_frags_all(int KSD) { return bwp_frags_o(KSD) + bwp_frags_kv(KSD) + bwp_frags_2(KSD) + bwp_frags_1(KSD); }

struct BwpArgs {
    int B, N, H, BH;
    int i_hi, i_lo;
    float alpha, scale, alibi;
    int norm_free;
    const uint4 *packed;
    const bf16_t *g_kv, *g_mlp, *g_k;
    const bf16_t *gy;                            // [B][N][d]
    const float *unit_k, *rk;                    // [M][2d] (first d columns), [M][H]
    const float *unit_z, *rinv_z, *unit_h, *rinv_h;
    const float *gp, *A_gy, *A_uz;               // [M][F]
    const float *C_gy, *C_uz, *C_uh;             // [M][d]
    const float *Qn, *Ktn, *Vt, *Kp, *Vp, *c, *lse;
    float *dK, *dV;                              // [M][d]: read at launch (upstream + tiles), final values written back
    float *dkraw, *d_rz, *Gz, *dpre, *t1, *d_h, *dc, *Ds, *dq, *dkt, *dvt;
    unsigned tag_base;
    unsigned long long *bar, *words;             // [8] abort word; exchange words, two parities per group
    size_t group_stride;
    long long spin_limit;
    int sl_1, sl_2, sl_3, sl_4;                  // waits before the first poll of the four pulls, units of 4 x 64 clocks
};
// words of one group and parity for two sequences: pairs of bf16 [dkraw | dV], w, dpre, w2; dc one fp32 per word
struct BwpWords {
    size_t e1, e2, e3, e5, e6, all;
};
__host__ __device__ inline BwpWords bwp_words(int d)
{
    BwpWords w;
    const size_t pair = (size_t)kBwpRows * d / 2;
    w.e1 = 0; w.e2 = 2 * pair; w.e3 = 3 * pair; w.e5 = 7 * pair; w.e6 = 8 * pair; w.all = 10 * pair;
    return w;
}

// sum over a wavefront's share of a row of <unit, received values>: lane l holds elements 64 m + 4 (l/4) .. + 3 of batch row l%4
template <int NC> __device__ __forceinline__ float share_dot(const float4 (&u)[NC], const Piece (&act)[NC])
{
    float s = 0.f;
#pragma unroll
    for (int m = 0; m < NC; ++m) {
        s = fmaf(u[m].x, __uint_as_float(act[m].u.x << 16), s);
        s = fmaf(u[m].y, __uint_as_float(act[m].u.x & 0xFFFF0000u), s);
        s = fmaf(u[m].z, __uint_as_float(act[m].u.y << 16), s);
        s = fmaf(u[m].w, __uint_as_float(act[m].u.y & 0xFFFF0000u), s);
    }
    return sum_mod4(s);
}

struct BwpLds {
    int wo, wkv, red, dots, win_k, win_v, acc_k, acc_v, share, flag, all;
};
__host__ __device__ constexpr BwpLds bwp_lds(int KSD)
{
    BwpLds L = {};
    int o = 0;
    L.wo = o; o += bwp_frags_o(KSD) * 1024;
    L.wkv = o; o += bwp_frags_kv(KSD) * 1024;
    L.red = o; o += 2 * kPW * 256 * 4;
    L.dots = o; o += 2 * kPW * 4 * 4;
    L.win_k = o; o += kBwpBlock * kWinLd * 4;
    L.win_v = o; o += kBwpBlock * kWinLd * 4;
    L.acc_k = o; o += kBwpBlock * kHeadDim * 4;
    L.acc_v = o; o += kBwpBlock * kHeadDim * 4;
    L.share = o; o += 4 * 64 * 4;
    L.flag = o; o += 16;
    L.all = o;
    return L;
}

// KSD = d / 256; BM: sequences per group the exchanged vectors are laid out for (1 or 2)
template <int KSD, int BM>
__global__ __launch_bounds__(kPThreads) void bwp_kernel(BwpArgs A)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int xcd = blockIdx.x & 7, grp = xcd >> 1;
    const int rank = (int)(blockIdx.x >> 3) + ((xcd & 1) << 5);
    constexpr int d = 256 * KSD, F = 4 * d, RO = 4 * KSD, R1 = 16 * KSD;
    constexpr int CD = bwp_chunks_d(KSD), CF = 2 * KSD, LD = d / kPW, LF = F / kPW;
    const int B = (A.B - grp + kBwpGroups - 1) / kBwpGroups;   // sequences grp, grp + 4
    if (B <= 0) return;

    const BwpLds L = bwp_lds(KSD);
    const uint4 *wo_s = reinterpret_cast<const uint4 *>(smem + L.wo) + wave * CD * 128;
    const uint4 *wkv_s = reinterpret_cast<const uint4 *>(smem + L.wkv) + wave * KSD * 128;
    float *red0 = reinterpret_cast<float *>(smem + L.red), *red1 = red0 + kPW * 256;
    float *dot_s = reinterpret_cast<float *>(smem + L.dots), *dot2_s = dot_s + kPW * 4;
    float *winK = reinterpret_cast<float *>(smem + L.win_k), *winV = reinterpret_cast<float *>(smem + L.win_v);
    float *accK = reinterpret_cast<float *>(smem + L.acc_k), *accV = reinterpret_cast<float *>(smem + L.acc_v);
    float *sh = reinterpret_cast<float *>(smem + L.share);   // p, dS of the window's keys, gradient and query of the position
    int *flag_s = reinterpret_cast<int *>(smem + L.flag);

    GroupWait G;
    G.spin_limit = A.spin_limit;
    G.bar = A.bar;
    unsigned long long *words = A.words + grp * A.group_stride;
    const BwpWords X = bwp_words(d);

    const uint4 *packed = A.packed + (size_t)rank * bwp_frags_all(KSD) * 64;
    WFrag w2t[KSD][CD][2], w1t[CF][2];   // W2^T, W1^T: this wavefront's eighth of the contraction
    {
        uint4 *dst = reinterpret_cast<uint4 *>(smem + L.wo);
        constexpr int n = (bwp_frags_o(KSD) + bwp_frags_kv(KSD)) * 64 / kPThreads;   // both slices: one run
        uint4 t[n];
#pragma unroll
        for (int i = 0; i < n; ++i) t[i] = packed[i * kPThreads + threadIdx.x];
        const uint4 *p2 = packed + (size_t)(bwp_frags_o(KSD) + bwp_frags_kv(KSD)) * 64, *p1 = p2 + (size_t)bwp_frags_2(KSD) * 64;
#pragma unroll
        for (int i = 0; i < KSD; ++i)
#pragma unroll
            for (int m = 0; m < CD; ++m)
#pragma unroll
                for (int j = 0; j < 2; ++j) w2t[i][m][j].u = p2[(((i * kPW + wave) * CD + m) * 2 + j) * 64 + lane];
#pragma unroll
        for (int m = 0; m < CF; ++m)
#pragma unroll
            for (int j = 0; j < 2; ++j) w1t[m][j].u = p1[((wave * CF + m) * 2 + j) * 64 + lane];
#pragma unroll
        for (int i = 0; i < n; ++i) dst[i * kPThreads + threadIdx.x] = t[i];
    }
    if (threadIdx.x == 0) flag_s[1] = 0;

    const size_t rs = (size_t)A.BH * kHeadDim;   // = B d: one position of a position-first tensor
    const int blk_lo = A.i_lo;                   // first position of the block
    const bool has_u = rank < B * A.H;           // this workgroup's (b, h), wavefront 4 does its softmax backward
    const int ub = rank / A.H, uh = rank - ub * A.H, bg = grp + kBwpGroups * ub;
    const int ug = bg * A.H + uh;
    const bool is_owner = has_u && wave == 4;
    if (has_u) {   // the block's keys, values and gradient accumulators, every wavefront four rows
        float kv4[kBwpBlock / kPW][4];
#pragma unroll
        for (int jj = 0; jj < kBwpBlock / kPW; ++jj) {
            const int pos = min(blk_lo + wave + kPW * jj, A.N - 1);
            const size_t o = (size_t)pos * rs + (unsigned)(ug * kHeadDim + lane);
            kv4[jj][0] = A.Kp[o]; kv4[jj][1] = A.Vp[o]; kv4[jj][2] = A.dK[o]; kv4[jj][3] = A.dV[o];
        }
#pragma unroll
        for (int jj = 0; jj < kBwpBlock / kPW; ++jj) {
            const int j = wave + kPW * jj;
            winK[j * kWinLd + lane] = kv4[jj][0];
            winV[j * kWinLd + lane] = kv4[jj][1];
            accK[j * kHeadDim + lane] = kv4[jj][2];
            accV[j * kHeadDim + lane] = kv4[jj][3];
        }
    }

    const float inv_d = 1.f / (float)d;
    float gkv_o = 1.f, gmlp_o = 1.f;             // gains of wavefront 0's epilogue rows
    if (wave == 0 && (lane >> 2) < RO && !A.norm_free) {
        if (A.g_kv) gkv_o = bf16_to_f32(A.g_kv[rank * RO + (lane >> 2)]);
        if (A.g_mlp) gmlp_o = bf16_to_f32(A.g_mlp[rank * RO + (lane >> 2)]);
    }
    const float gk_u = (is_owner && A.g_k) ? bf16_to_f32(A.g_k[uh * kHeadDim + lane]) : 1.f;
    const float slope = alibi_slope(A.alibi, uh, A.H);

    // What a position needs from the recompute is requested at the end of the position after it: behind the polls of that
    // position, and early enough not to hold up its own.
    float e_gy = 0.f, e_uz = 0.f, e_uh = 0.f, e_cgy = 0.f, e_cuz = 0.f, e_cuh = 0.f, e_rz = 1.f, e_rh = 1.f;   // wavefront 0: rows of the d-long products
    float e_gp = 0.f, e_agy = 0.f, e_auz = 0.f;                                                               // wavefronts 0 .. KSD - 1: rows of W2^T
    float4 uz[CD], un_h[CD];                                                                                  // unit rows, the wavefront's share
    float a_q = 0.f, a_kt = 0.f, a_vt = 0.f, a_c = 0.f, a_L = 0.f, a_un = 0.f, a_rk = 1.f;                    // owner
    auto request = [&](int i, int ln) {
        const size_t r0 = (size_t)i * A.B;
        const int b = ln & 3, bb = grp + kBwpGroups * b;
        const bool live = b < B;
        if (wave < KSD && live) {   // 64 rows of W2^T and 16 of the others per wavefront
            const size_t r = r0 + bb;
            e_rz = A.rinv_z[r];
            const size_t f = r * F + (unsigned)(rank * R1 + wave * 16 + (ln >> 2));
            e_gp = A.gp[f]; e_agy = A.A_gy[f]; e_auz = A.A_uz[f];
            if (wave == 0 && (ln >> 2) < RO) {
                e_rh = A.rinv_h[r];
                const unsigned col = rank * RO + (ln >> 2);
                const size_t o = r * d + col;
                e_gy = bf16_to_f32(A.gy[((size_t)bb * A.N + i) * d + col]);
                e_uz = A.unit_z[o]; e_uh = A.unit_h[o];
                e_cgy = A.C_gy[o]; e_cuz = A.C_uz[o]; e_cuh = A.C_uh[o];
            }
        }
#pragma unroll
        for (int m = 0; m < CD; ++m) {
            uz[m] = un_h[m] = make_float4(0.f, 0.f, 0.f, 0.f);
            const int k = 64 * m + 4 * (ln >> 2);
            if (live && k < LD) {
                const size_t o = (r0 + bb) * d + (unsigned)(wave * LD + k);
                uz[m] = *reinterpret_cast<const float4 *>(A.unit_z + o);
                un_h[m] = *reinterpret_cast<const float4 *>(A.unit_h + o);
            }
        }
        if (is_owner) {
            const size_t off = (size_t)i * rs + (unsigned)(ug * kHeadDim + ln);
            a_q = A.Qn[off]; a_kt = A.Ktn[off]; a_vt = A.Vt[off]; a_c = A.c[off];
            a_L = A.lse[(size_t)i * A.BH + ug];
        }
    };
    auto request_pair = [&](int i, int ln) {   // what phase U of position i needs
        if (is_owner && !A.norm_free && i >= A.i_lo) {
            const size_t r = (size_t)i * A.B + bg;
            a_un = A.unit_k[r * 2 * d + (unsigned)(uh * kHeadDim + ln)];
            a_rk = A.rk[r * A.H + uh];
        }
    };
    // Phase U: the complete pair gradient (dk, dv) of position i goes out as the vectors of the step with that tag and parity.
    auto phase_u = [&](int i, int par, unsigned tag, float dk, float dv, int ln) {
        const size_t off = (size_t)i * rs + (unsigned)(ug * kHeadDim + ln);
        float du = dk;
        if (!A.norm_free) {
            const float wv = dk * gk_u;
            du = a_rk * (wv - a_un * (fast_sum(a_un * wv) * (1.f / (float)kHeadDim)));
        }
        const float dun = dpp_odd_neighbour(du), dvn = dpp_odd_neighbour(dv);
        if (!(ln & 1)) {
            // a wavefront's share of [dkraw | dV]: its share of both
            const unsigned k = uh * kHeadDim + ln, kk = k / LD * (2 * LD) + k % LD;
            word_store(words + par * X.all + X.e1, piece_word<8, BM>(kk, ub), tag, (unsigned)f32_to_bf16(du) | ((unsigned)f32_to_bf16(dun) << 16));
            word_store(words + par * X.all + X.e1, piece_word<8, BM>(kk + LD, ub), tag, (unsigned)f32_to_bf16(dv) | ((unsigned)f32_to_bf16(dvn) << 16));
        }
        A.dK[off] = dk;
        A.dV[off] = dv;
        A.dkraw[off] = du;
        request_pair(i - 1, ln);
    };

    request(A.i_hi, lane);
    request_pair(A.i_hi, lane);
    __syncthreads();
    if (is_owner) {
        const int slot = A.i_hi - blk_lo;
        phase_u(A.i_hi, 0, A.tag_base | 1u, accK[slot * kHeadDim + lane], accV[slot * kHeadDim + lane], lane);
    }

    int fail = 0;
    for (int i = A.i_hi; i >= A.i_lo; --i) {
        const int step = A.i_hi - i, par = step & 1;
        const unsigned tag = A.tag_base | (unsigned)(step + 1);
        const size_t r0 = (size_t)i * A.B;
        unsigned long long *wp = words + par * X.all;
        int ln = lane;
        asm volatile("" : "+v"(ln));   // opaque: what depends on the lane is formed in every position, registers are for the weights
        const int erow = ln >> 2, eb = ln & 3;
        const bool e_own = wave == 0 && erow < RO && eb < B;
        const size_t e_r = r0 + grp + kBwpGroups * eb;
        const unsigned e_col = rank * RO + erow;

        // ================================================================ G1: d_rz = Wk^T dkraw + Wv^T dV_i
        {
            Piece act[KSD];
            slice_pull<KSD, 2 * LD, 8, BM>(wp + X.e1, wave, ln, B, tag, G, act, fail, A.sl_1);
            f32x4_t acc[4] = {};
#pragma unroll
            for (int m = 0; m < KSD; ++m) {
                WFrag w0, w1;
                w0.u = lds_load16(wkv_s + (m * 2) * 64 + ln);
                w1.u = lds_load16(wkv_s + (m * 2 + 1) * 64 + ln);
                chunk_product4(act[m], w0, w1, acc);
            }
            const f32x4_t s[1] = {(acc[0] + acc[1]) + (acc[2] + acc[3])};
            tiles_store<1>(red0, wave, ln, s);
        }
        RT_GROUP_SYNC(fail);
        float wv = 0.f;
        if (wave == 0) {
            const float drz = tile_sum(red0, ln);
            wv = drz * gkv_o;
            const float wn = row_partner(wv);
            if (e_own && !(erow & 1))
                word_store(wp + X.e2, piece_word<1, BM>(e_col, eb), tag, (unsigned)f32_to_bf16(wv) | ((unsigned)f32_to_bf16(wn) << 16));
            if (e_own) A.d_rz[e_r * d + e_col] = drz;
        }
        __syncthreads();

        // ================================================================ G2: dot, W2^T w, Wo^T w; dpre rows, Gz rows
        {
            Piece act[CD];
            slice_pull<CD, LD, 1, BM>(wp + X.e2, wave, ln, B, tag, G, act, fail, A.sl_2);
            f32x4_t acc[KSD] = {};
#pragma unroll
            for (int m = 0; m < CD; ++m)
#pragma unroll
                for (int t = 0; t < KSD; ++t) acc[t] = chunk_product(act[m], w2t[t][m][0], w2t[t][m][1], acc[t]);
            tiles_store<KSD>(red1, wave, ln, acc);
            f32x4_t ao[4] = {};
#pragma unroll
            for (int m = 0; m < CD; ++m) {
                WFrag w0, w1;
                w0.u = lds_load16(wo_s + (m * 2) * 64 + ln);
                w1.u = lds_load16(wo_s + (m * 2 + 1) * 64 + ln);
                chunk_product4(act[m], w0, w1, ao);
            }
            const f32x4_t s[1] = {(ao[0] + ao[1]) + (ao[2] + ao[3])};
            tiles_store<1>(red0, wave, ln, s);
            const float dt = share_dot<CD>(uz, act);
            if (ln < 4) dot_s[wave * 4 + ln] = dt;
        }
        RT_GROUP_SYNC(fail);
        float gz = 0.f, cw = 0.f, k1 = 0.f;
        if (wave < KSD) {
            float dot = 0.f;
#pragma unroll
            for (int w = 0; w < kPW; ++w) dot += dot_s[w * 4 + eb];
            k1 = A.norm_free ? 0.f : dot * inv_d;
            const int tn = wave * 64 + ln;
            const float v = tile_sum(red1, tn);
            const float lin = A.norm_free ? e_agy + v : e_agy + e_rz * (v - k1 * e_auz);
            const float dp = e_gp * A.alpha * lin;
            const float dn = row_partner(dp);
            const unsigned row = rank * R1 + wave * 16 + erow;
            if (!(erow & 1) && eb < B)
                word_store(wp + X.e3, piece_word<1, BM>(row, eb), tag, (unsigned)f32_to_bf16(dp) | ((unsigned)f32_to_bf16(dn) << 16));
            if (eb < B) A.dpre[e_r * F + row] = dp;
            if (wave == 0) {
                gz = A.norm_free ? e_gy + wv : e_gy + e_rz * (wv - e_uz * k1);
                cw = tile_sum(red0, ln);
                if (e_own) A.Gz[e_r * d + e_col] = gz;
            }
        }
        __syncthreads();

        // ================================================================ G3: t1 rows = W1^T dpre, w2 = t1 g_mlp
        {
            Piece act[CF];
            slice_pull<CF, LF, 1, BM>(wp + X.e3, wave, ln, B, tag, G, act, fail, A.sl_3);
            f32x4_t acc[4] = {};
#pragma unroll
            for (int m = 0; m < CF; ++m) chunk_product4(act[m], w1t[m][0], w1t[m][1], acc);
            const f32x4_t s[1] = {(acc[0] + acc[1]) + (acc[2] + acc[3])};
            tiles_store<1>(red1, wave, ln, s);
        }
        RT_GROUP_SYNC(fail);
        float w2v = 0.f;
        if (wave == 0) {
            const float t1v = tile_sum(red1, ln);
            w2v = t1v * gmlp_o;
            const float wn = row_partner(w2v);
            if (e_own && !(erow & 1))
                word_store(wp + X.e5, piece_word<1, BM>(e_col, eb), tag, (unsigned)f32_to_bf16(w2v) | ((unsigned)f32_to_bf16(wn) << 16));
            if (e_own) A.t1[e_r * d + e_col] = t1v;
        }
        __syncthreads();

        // ================================================================ G4: dot2, Wo^T w2; dc rows, dh rows
        {
            Piece act[CD];
            slice_pull<CD, LD, 1, BM>(wp + X.e5, wave, ln, B, tag, G, act, fail, A.sl_4);
            f32x4_t ao[4] = {};
#pragma unroll
            for (int m = 0; m < CD; ++m) {
                WFrag w0, w1;
                w0.u = lds_load16(wo_s + (m * 2) * 64 + ln);
                w1.u = lds_load16(wo_s + (m * 2 + 1) * 64 + ln);
                chunk_product4(act[m], w0, w1, ao);
            }
            const f32x4_t s[1] = {(ao[0] + ao[1]) + (ao[2] + ao[3])};
            tiles_store<1>(red0, wave, ln, s);
            const float dt = share_dot<CD>(un_h, act);
            if (ln < 4) dot2_s[wave * 4 + ln] = dt;
        }
        RT_GROUP_SYNC(fail);
        if (wave == 0) {
            const float v = tile_sum(red0, ln);
            float dcv, dh;
            if (A.norm_free) {
                dcv = A.alpha * (e_cgy + cw + v);
                dh = gz + w2v;
            } else {
                float k2 = 0.f;
#pragma unroll
                for (int w = 0; w < kPW; ++w) k2 += dot2_s[w * 4 + eb];
                k2 *= inv_d;
                dcv = A.alpha * (e_cgy + e_rz * (cw - k1 * e_cuz) + e_rh * (v - k2 * e_cuh));
                dh = gz + e_rh * (w2v - e_uh * k2);
            }
            if (e_own) {
                word_store(wp + X.e6, (rank * BM + eb) * RO + erow, tag, __float_as_uint(dcv));
                A.dc[e_r * d + e_col] = dcv;
                A.d_h[e_r * d + e_col] = dh;
            }
        }

        // ================================================================ A: softmax backward of query i
        const int w = i - blk_lo;   // keys of the block before the query: slots 0 .. w - 1
        if (is_owner) {
            const size_t off = (size_t)i * rs + (unsigned)(ug * kHeadDim + ln);
            const float q = a_q, kt = a_kt;
            // what does not need the gradient of the attention output is formed before the wait for it: the query's own
            // weight and the weights of the window
            const float p_own = __expf(A.scale * fast_sum(q * kt) - a_L);
            const float *krow = winK + (size_t)min(ln, max(w - 1, 0)) * kWinLd, *vrow = winV + (size_t)min(ln, max(w - 1, 0)) * kWinLd;
            float p = 0.f;
            if (w > 0) {
                float s = 0.f;
#pragma unroll
                for (int c8 = 0; c8 < 8; ++c8) {
                    float kk[8];
                    load8(krow + c8 * 8, kk);
#pragma unroll
                    for (int e = 0; e < 8; ++e) s = fmaf(lane_bcast(q, c8 * 8 + e), kk[e], s);
                }
                p = ln < w ? __expf(fmaf(-slope, (float)(w - ln), s * A.scale) - a_L) : 0.f;
            }
            const unsigned o6 = uh * kHeadDim + ln;
            const ll_t wd = ll_wait(wp + X.e6 + (size_t)((o6 / RO * BM + ub) * RO + o6 % RO), true, tag, G, fail);
            const float g = __uint_as_float((unsigned)wd);
            const float Dsum = fast_sum(g * a_c);
            const float ds_own = p_own * (fast_sum(g * a_vt) - Dsum);
            if (w > 0) {
                float dp = 0.f;
#pragma unroll
                for (int c8 = 0; c8 < 8; ++c8) {
                    float vv[8];
                    load8(vrow + c8 * 8, vv);
#pragma unroll
                    for (int e = 0; e < 8; ++e) dp = fmaf(lane_bcast(g, c8 * 8 + e), vv[e], dp);
                }
                const float ds = p * (dp - Dsum);
                // the newest slot first: with it the pair gradient of position i - 1 is complete and goes out at once
                const int j = w - 1;
                const float dvn = fmaf(lane_bcast(p, j), g, accV[j * kHeadDim + ln]);
                const float dkn = fmaf(A.scale * lane_bcast(ds, j), q, accK[j * kHeadDim + ln]);
                phase_u(i - 1, par ^ 1, tag + 1u, dkn, dvn, ln);
                sh[ln] = p; sh[64 + ln] = ds; sh[128 + ln] = g; sh[192 + ln] = q;   // for the older slots, below
            }
            // the query's own gradients follow the pair gradient of the next position: only that one is waited for
            A.dvt[off] = p_own * g;
            A.dkt[off] = A.scale * ds_own * q;
            A.dq[off] = A.scale * ds_own * kt;
            if (ln == 0) A.Ds[(size_t)i * A.BH + ug] = Dsum;
        }
        if (i > A.i_lo) request(i - 1, ln);
        RT_GROUP_SYNC(fail);
        if (has_u) {   // the older slots, four at most per wavefront, while the pair gradient crosses the chip
            const float g = sh[128 + ln], q = sh[192 + ln];
            for (int j = wave; j < w - 1; j += kPW) {
                accV[j * kHeadDim + ln] = fmaf(sh[j], g, accV[j * kHeadDim + ln]);
                accK[j * kHeadDim + ln] = fmaf(A.scale * sh[64 + j], q, accK[j * kHeadDim + ln]);
            }
        }
    }
}

// The transposed matrices in the fragment order above.  Lane l of fragment (tile, wavefront, chunk m, j) holds W[row0 + 16 tile + l%16][k .. k + 7],
// k the wavefront's share's element 64 m + 16 (l/16) + 8 j; a share of [Wk^T | Wv^T] is the share of both.
__global__ __launch_bounds__(256) void bwp_pack_kernel(const bf16_t *WkvT, const bf16_t *W2T, const bf16_t *W1T, const bf16_t *WoT, int KSD, uint4 *dst)
{
    const int per = bwp_frags_all(KSD), d = 256 * KSD, LD = d / kPW;
    const int f_all = (int)((blockIdx.x * 256 + threadIdx.x) >> 6), lane = threadIdx.x & 63;
    if (f_all >= per * kBwpRanks) return;
    const int rank = f_all / per;
    int f = f_all - rank * per, rows = 4 * KSD, chunks = bwp_chunks_d(KSD), K = d;
    const bf16_t *src = WoT;
    bool pairs = false;
    if (f < bwp_frags_o(KSD)) {
    } else if ((f -= bwp_frags_o(KSD)) < bwp_frags_kv(KSD)) {
        src = WkvT; chunks = KSD; K = 2 * d; pairs = true;
    } else if ((f -= bwp_frags_kv(KSD)) < bwp_frags_2(KSD)) {
        src = W2T; rows = 16 * KSD;
    } else {
        f -= bwp_frags_2(KSD);
        src = W1T; chunks = 2 * KSD; K = 4 * d;
    }
    const int j = f & 1, m = (f >> 1) % chunks, w = (f >> 1) / chunks % kPW, tile = (f >> 1) / (chunks * kPW);
    const int kk = 64 * m + 16 * (lane >> 4) + 8 * j;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (tile * 16 + (lane & 15) < rows && kk < K / kPW) {
        const int row = rank * rows + tile * 16 + (lane & 15);
        const int k = pairs ? (kk < LD ? w * LD + kk : d + w * LD + kk - LD) : w * (K / kPW) + kk;
        v = *reinterpret_cast<const uint4 *>(src + (size_t)row * K + k);
    }
    dst[(size_t)f_all * 64 + lane] = v;
}

// =============================================================================================
// Host side
// =============================================================================================
namespace {
typedef void (*bwp_fn)(BwpArgs);
bwp_fn pick(int d, int BM)
{
    switch (d) {
    case 256: return BM == 1 ? bwp_kernel<1, 1> : bwp_kernel<1, 2>;
    case 512: return BM == 1 ? bwp_kernel<2, 1> : bwp_kernel<2, 2>;
    case 768: return BM == 1 ? bwp_kernel<3, 1> : bwp_kernel<3, 2>;
    case 1024: return BM == 1 ? bwp_kernel<4, 1> : bwp_kernel<4, 2>;
    default: return nullptr;
    }
}
size_t up256(size_t v) { return (v + 255) / 256 * 256; }
bool shape_ok(int d, int F) { return d % 256 == 0 && d <= 1024 && F == 4 * d; }
size_t group_stride(int d) { return up256(2 * bwp_words(d).all * 8) / 8; }
size_t word_bytes(int d) { return 256 + kBwpGroups * group_stride(d) * 8; }   // counters and exchange words; the packed matrices follow
__global__ void bwp_clear_kernel(unsigned long long *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0ULL;
}
}  // namespace

size_t bwp_exchange_bytes(int d, int F)
{
    return shape_ok(d, F) ? word_bytes(d) + (size_t)bwp_frags_all(d / 256) * kBwpRanks * 1024 : 256;
}

bool bwp_create(BwpState &P, int device, int d, int F, int H, int max_batch, bool bf16_mfma)
{
    P.available = false;
    if (!bf16_mfma || getenv("RT_BWD_NO_PERSISTENT")) return false;
    if (!shape_ok(d, F) || max_batch < 1 || kBwpRows * H > kBwpRanks) return false;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return false;
    if (cus != kBwpGroups * kBwpRanks) return false;
    P.lds_bytes = (size_t)bwp_lds(d / 256).all;
    if (P.lds_bytes > (size_t)160 * 1024) return false;
    {   // once per device and kernel
        static std::mutex mu;
        static uint64_t raised[5] = {};
        std::lock_guard<std::mutex> lock(mu);
        const uint64_t bit = 1ULL << (device & 63);
        for (int BM = 1; BM <= 2 && !(raised[d / 256] & bit); ++BM)
            if (hipFuncSetAttribute((const void *)pick(d, BM), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) {
                (void)hipGetLastError();
                return false;
            }
        raised[d / 256] |= bit;
    }
    P.H = H;
    const char *sl = getenv("RT_SPIN_LIMIT");
    P.spin_limit = sl ? atoll(sl) : (1LL << 21);
    if (P.spin_limit < 1) P.spin_limit = 1;
    P.available = true;
    return true;
}

bool bwp_supported(const BwpState &P, const LayerDims &D)
{
    return P.available && D.B <= kBwpGroups * kBwpRows && D.H == P.H;
}

hipError_t bwp_pack(const LayerDims &D, const BwpTensors &T, void *exchange, hipStream_t st)
{
    const int KSD = D.d / 256, frags = bwp_frags_all(KSD) * kBwpRanks;
    hipLaunchKernelGGL(bwp_pack_kernel, dim3((unsigned)((frags + 3) / 4)), dim3(256), 0, st, T.WkvT, T.W2T, T.W1T, T.WoT, KSD,
                       (uint4 *)((char *)exchange + word_bytes(D.d)));
    return hipGetLastError();
}

hipError_t bwp_run_block(BwpState &P, const LayerDims &D, const BwpTensors &T, void *exchange, int i_hi, int i_lo, hipStream_t st)
{
    BwpArgs A;
    A.B = D.B; A.N = D.N; A.H = D.H; A.BH = D.B * D.H;
    A.i_hi = i_hi; A.i_lo = i_lo;
    A.alpha = D.alpha; A.scale = D.scale; A.alibi = D.alibi; A.norm_free = D.norm_free;
    A.g_kv = T.g_kv; A.g_mlp = T.g_mlp; A.g_k = T.g_k; A.gy = T.gy;
    A.unit_k = T.unit_k; A.rk = T.rk; A.unit_z = T.unit_z; A.rinv_z = T.rinv_z; A.unit_h = T.unit_h; A.rinv_h = T.rinv_h;
    A.gp = T.gp; A.A_gy = T.A_gy; A.A_uz = T.A_uz; A.C_gy = T.C_gy; A.C_uz = T.C_uz; A.C_uh = T.C_uh;
    A.Qn = T.Qn; A.Ktn = T.Ktn; A.Vt = T.Vt; A.Kp = T.Kp; A.Vp = T.Vp; A.c = T.c; A.lse = T.lse;
    A.dK = T.dK; A.dV = T.dV; A.dkraw = T.dkraw; A.d_rz = T.d_rz; A.Gz = T.Gz; A.dpre = T.dpre; A.t1 = T.t1; A.d_h = T.d_h;
    A.dc = T.dc; A.Ds = T.Ds; A.dq = T.dq; A.dkt = T.dkt; A.dvt = T.dvt;
    A.bar = (unsigned long long *)exchange;
    A.words = A.bar + 32;
    A.group_stride = group_stride(D.d);
    A.packed = (const uint4 *)((const char *)exchange + word_bytes(D.d));
    A.spin_limit = P.spin_limit;
    // d = 1024, B = 8, N = 2048, ms per backward pass: 0011 27.00, 0000 27.04, 0111 27.11, 0212 27.49, 0222 27.73
    int sl[4] = {0, 0, 1, 1};
    if (const char *ps = getenv("RT_BWD_PRE_SLEEPS"))   // four digits: the pulls of phases G1, G2, G3, G4
        for (int k = 0; k < 4 && ps[k]; ++k) sl[k] = ps[k] - '0';
    A.sl_1 = sl[0]; A.sl_2 = sl[1]; A.sl_3 = sl[2]; A.sl_4 = sl[3];
    // Tags: 1 .. 4094 in turn; when they start over no word of an earlier launch may survive.  A captured launch is replayed with the
    // same tag: it has one of its own and clears the words first.
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    hipError_t e = st ? hipStreamIsCapturing(st, &capturing) : hipSuccess;
    if (e != hipSuccess) return e;
    const bool captured = capturing != hipStreamCaptureStatusNone;
    if (captured || P.nonce >= 4094u) {
        hipLaunchKernelGGL(bwp_clear_kernel, dim3(256), dim3(256), 0, st, A.words, kBwpGroups * A.group_stride);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (!captured) P.nonce = 0;
    }
    if (!captured) P.nonce += 1;
    A.tag_base = (captured ? 4095u : P.nonce) << 20;
    // an ordinary launch: one workgroup fills a compute unit and the grid is one workgroup per compute unit, so all of
    // them are resident once the kernels before it on the stream have drained (the cooperative queue costs about
    // 20 us per launch, measured on the decoding step)
    hipLaunchKernelGGL(pick(D.d, D.B <= kBwpGroups ? 1 : 2), dim3(kBwpGroups * kBwpRanks), dim3(kPThreads), (unsigned int)P.lds_bytes, st, A);
    return hipGetLastError();
}

}  // namespace rt
