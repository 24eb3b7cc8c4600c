// Grouped single-launch engine of the sequential loop, bf16 storage (d in {256, 512, 768, 1024}, F = 4 d, up to 16 sequences).
//
// The loop is a chain of dependent exchanges, and an exchange costs more the more workgroups take part and the further they
// are apart.  Measured on MI355X (all-to-all of a vector among workgroups of 512 threads, tagged words, no other work):
//     256 workgroups on 8 XCDs   4 KB 1.24-1.59 us   32 KB 1.55-1.88 us
//      64 workgroups on 2 XCDs   4 KB 0.74-0.94 us   32 KB 1.38-1.79 us
//      32 workgroups on 1 XCD    4 KB 0.61-0.75 us   32 KB 1.12-1.52 us
// Sequences are independent, so the 256 workgroups (one per compute unit) form four groups of two XCDs, and each group runs
// the whole layer for its own sequences (one to four): four times fewer partners per exchange, a quarter of the volume.  A
// group holds all loop matrices: 11 d^2 bf16 elements over 64 workgroups are 352 KB each at d = 1024, more than LDS.  Wo and
// [Wk; Wv] stay in LDS (96 KB); W1 and W2 are kept in registers as matrix-core fragments (128 of a lane's 256 registers at
// d = 1024), loaded again by a workgroup behind a cross-block event whose tile it computed (blocks of 64 keys and more), so
// that the tile has the registers to itself.  W2 needs no split of its contraction then (the 256-workgroup engine exchanges
// four partial sums per output), and a position has five exchanges instead of six:
//
//   M    per (b, h) wavefront: raw k, v of position t-1 and the partial sums of z^2 -> finished pair, newest key of a_t   -> a
//   O    h = x_t + alpha Wo a                                                                                            -> bf16(h)
//   1    u = gelu(W1' h / rms(h))                                                                                        -> u
//   2    z = h + alpha W2 u                                                                   -> y, bf16(z), partial sums of z^2
//   KV   [Wk'; Wv'] z                                                                                                    -> raw k, v
//
// Workgroup blockIdx.x belongs to the group (blockIdx.x % 8) / 2: consecutive workgroups are dealt to the XCDs in turn.  Only
// speed depends on that placement: the exchange words are stored and polled at agent scope (rt_ll.h).
//
// A wavefront multiplies one eighth of the contraction and pulls exactly the words of that eighth.  The products are
// v_mfma_f32_4x4x4_16b_bf16 with the batch rows as rows of A: a 16-byte word pair of an exchanged vector (four elements of one
// batch row) is a lane's A operand as it arrives, so nothing is staged in LDS and no lane holds padding rows.  (With 16x16x32
// products and the vectors staged in LDS the headline shape took 22.5 ms instead of 18.1: two trips through LDS per exchange,
// and reads that repeat every row eight times.)  Vectors are laid out in pieces of four elements of one batch row, the group's
// rows side by side (BM = 1, 2 or 4 of them: a layout for four with two in use doubles the lines that cross the chip, 2.6
// instead of 1.1 us for u); a's pieces, one producer per head and row, in runs of eight, so that a line has one producer.
//
// The pre-merge of position t+1 (temporary pair, stored partial states, direct window: all but its two newest keys) is made
// by a helper wavefront of the owning workgroup during phase M of position t, from what another wavefront fetched a position
// earlier; the owner adds the window's newest key from its registers.
//
// Measured (ms per call, this form / the 256-workgroup form of rt_persistent.hip): d = 1024, N = 2048, B = 1, 8, 16:
// 17.7 / 28.7, 17.5 / 29.1, 19.7 / 32.5; d = 768, N = 1000, B = 5 with bias 8.4 / 15.4.  A position takes 7.9 us at B = 8, of it five
// exchanges of 0.5 - 1.2 us and as many products with their epilogues of 0.6 - 0.9 us.
//
// Everything else - logits from unrounded operands, the block decomposition shifted by one, bounded waits - is as in
// rt_persistent.hip.
#include "rt_group.h"
#include "rt_group_device.h"
#include "rt_cross_tile.h"

#include <cstdlib>
#include <mutex>

namespace rt {

// Cross-block events of at least this many keys are spread over the group's workgroups, between two fenced barriers; smaller
// ones stay with the workgroup that owns the (b, h).  Measured at d = 1024, B = 8, N = 2048 (us per event, spread / owner):
// 256 keys 48 / 25, 512 keys 54 / 46, 1024 keys 97 / not taken (four passes of the one workgroup, about 90).
constexpr int kGroupSpreadP = 1024;
constexpr int kGroupLevels = 16;     // stored-partial levels of a query, and one more for the far state
constexpr int kPreSlot = 3 * 64 + 2 * 20 + (kGroupLevels + 1) * 64;   // a multiple of four floats

// Weights of one workgroup in 1 KB fragments (64 lanes x 16 bytes): [Wo | W1 | W2 | Wkv], each [tile of 16 rows][wavefront]
// [chunk of 64 contraction indices][2]; a wavefront's share of the contraction is K / 8 indices, the last chunk zero beyond.
constexpr int chunks_d(int KSD) { return (KSD + 1) / 2; }
constexpr int chunks_F(int KSD) { return 2 * KSD; }
constexpr int kv_tiles(int KSD) { return (KSD + 1) / 2; }
constexpr int frags_o(int KSD) { return kPW * chunks_d(KSD) * 2; }
constexpr int frags_1(int KSD) { return KSD * kPW * chunks_d(KSD) * 2; }
constexpr int frags_2(int KSD) { return kPW * chunks_F(KSD) * 2; }
constexpr int frags_kv(int KSD) { return kv_tiles(KSD) * kPW * chunks_d(KSD) * 2; }
constexpr int frags_all(int KSD) { return frags_o(KSD) + frags_1(KSD) + frags_2(KSD) + frags_kv(KSD); }

// exchange words of one group and one parity
struct GroupWords {
    size_t a, h, u, z, kv, zss, hss, lo, all;   // lo: remainders of a, h, z, u, each so many words behind its heads
};
__host__ __device__ constexpr GroupWords group_words(int d, bool hp)
{
    GroupWords w = {};
    size_t o = 0;
    const size_t pair = (size_t)kGroupRows * d / 2;
    w.a = o; o += pair;
    w.h = o; o += pair;
    w.z = o; o += pair;
    w.u = o; o += 4 * pair;
    w.kv = o; o += 4 * pair;
    w.zss = o; o += (size_t)kGroupRows * kGroupRanks;
    if (hp) {
        w.hss = o; o += (size_t)kGroupRows * kGroupRanks;
        w.lo = o; o += 7 * pair;
    }
    w.all = o;
    return w;
}

// ---- Pre-merge of query t (everything but its two newest keys).  slot (floats of LDS): q, k_tmp, v_tmp rows; m[20], l[20] of
// the stored states; their o rows.
__device__ __forceinline__ int pre_levels(const GroupArgs &A, int t) { return t >= 2 ? (t - 1) >> A.log2_pmin : 0; }
// keys of the direct window that the pre-merge takes: all but the window's newest, which the owner adds
__device__ __forceinline__ int pre_window(const GroupArgs &A, int t) { return t >= 2 ? max(((t - 1) & (A.p_min - 1)) - 1, 0) : 0; }
__device__ __forceinline__ void pre_fetch(const GroupArgs &A, const GroupWork &W, int t, int u, float *slot, int lane)
{
    const size_t qoff = (size_t)t * A.BH * kHeadDim + (unsigned)(u * kHeadDim + lane);
    const float q = W.Qf[qoff], kt = W.Ktf[qoff], vt = bf16_to_f32(W.Vt[qoff]);
    float *sm = slot + 192, *sl = sm + 20, *so = sl + 20;
    int n = 0;
    if (W.far_m) {
        const size_t idx = (size_t)t * A.BH + u;
        const float m = W.far_m[idx], l = W.far_l[idx], o = W.far_o[idx * kHeadDim + lane];
        if (lane == 0) { sm[0] = m; sl[0] = l; }
        so[lane] = o;
        n = 1;
    }
    int bits = pre_levels(A, t);
    for (int lr = 0; bits; ++lr, bits >>= 1) {
        if (!(bits & 1)) continue;
        const size_t idx = partial_index(lr, partial_slot(lr + A.log2_pmin, t - 1), A.slots, A.BH, u);
        const float m = W.pm[idx], l = W.pl[idx], o = W.po[idx * kHeadDim + lane];
        if (lane == 0) { sm[n] = m; sl[n] = l; }
        so[n * 64 + lane] = o;
        ++n;
    }
    slot[lane] = q; slot[64 + lane] = kt; slot[128 + lane] = vt;
}
// HP: with the full-precision exponential (the operands that follow keep 16 bits)
template <bool HP> __device__ __forceinline__ float merge_exp(float x) { return HP ? expf(x) : __expf(x); }
// the state of the query -> out: rows q, m, l, o
template <bool ALIBI, bool HP>
__device__ __forceinline__ void pre_merge(const GroupArgs &A, bool far, int t, int u, const float *slot, const float *wk, const bf16_t *wv, float *out,
                                          int lane)
{
    const float *sm = slot + 192, *sl = sm + 20, *so = sl + 20;
    const float q = slot[lane];
    const float s0 = A.scale * fast_sum(q * slot[64 + lane]);
    const int n = __popc(pre_levels(A, t)) + (far ? 1 : 0);
    const int w = pre_window(A, t);
    float m = s0;
    for (int i = 0; i < n; ++i) m = fmaxf(m, sm[i]);
    float logit = -INFINITY;
    if (w > 0) {
        const bool valid = lane < w;
        const float *krow = wk + (size_t)(valid ? lane : 0) * (kHeadDim + 4);   // rows padded against bank conflicts
        float acc[2] = {0.f, 0.f};
#pragma unroll
        for (int c8 = 0; c8 < 8; ++c8) {
            float kk[8];
            load8(krow + c8 * 8, kk);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e & 1] = fmaf(lane_bcast(q, c8 * 8 + e), kk[e], acc[e & 1]);
        }
        const float s = (acc[0] + acc[1]) * A.scale;
        // key j of the window is w + 2 - j positions before the query
        logit = valid ? (ALIBI ? fmaf(-alibi_slope(A.alibi, u % A.H, A.H), (float)(w + 2 - lane), s) : s) : -INFINITY;
        m = fmaxf(m, fast_max(logit));
    }
    const float e0 = merge_exp<HP>(s0 - m);
    float l = e0, o = slot[128 + lane] * e0;
    for (int i = 0; i < n; ++i) {
        const float f = merge_exp<HP>(sm[i] - m);
        l = fmaf(sl[i], f, l);
        o = fmaf(so[i * 64 + lane], f, o);
    }
    if (w > 0) {
        const float p = merge_exp<HP>(logit - m);   // exp(-inf) = 0 for the lanes without a key
        l += fast_sum(p);
        for (int j0 = 0; j0 < w; j0 += 8) {   // rows past the end are read from the last row with weight zero
            float vv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) vv[e] = bf16_to_f32(wv[(size_t)min(j0 + e, w - 1) * kHeadDim + lane]);
#pragma unroll
            for (int e = 0; e < 8; ++e) o = fmaf(lane_bcast(p, j0 + e), vv[e], o);
        }
    }
    out[lane] = q; out[64 + lane] = m; out[128 + lane] = l; out[192 + lane] = o;
}

// The block of p_min = 32 keys that ends at key t0 - 1, folded into the next nq <= 32 queries by all eight wavefronts of the
// owning workgroup, four queries each: keys and values are the direct window's ring in LDS, logits and weights in fp32, few
// registers, so that the weight fragments stay where they are.  q_s: 4 x 64 floats of LDS of this wavefront.
template <bool ALIBI>
__device__ __forceinline__ void window_block(const GroupArgs &A, const GroupWork &W, int t0, int nq, int u, const float *wk, const bf16_t *wv,
                                             float *q_s, int wave, int lane)
{
    const int q0 = wave * 4;
    if (q0 >= nq) return;
    const int key = lane & 31, half = lane >> 5;
    const size_t rs = (size_t)A.BH * kHeadDim;
    float qv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) qv[i] = W.Qf[(size_t)(t0 + 1 + min(q0 + i, nq - 1)) * rs + (unsigned)(u * kHeadDim + lane)];
#pragma unroll
    for (int i = 0; i < 4; ++i) q_s[i * 64 + lane] = qv[i];
    wave_sync_lds();
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    const float *krow = wk + (size_t)key * (kHeadDim + 4) + half * 32;   // each half of the wavefront takes half of the dimensions
#pragma unroll
    for (int c8 = 0; c8 < 4; ++c8) {
        float kk[8];
        load8(krow + c8 * 8, kk);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float qq[8];
            load8(q_s + i * 64 + half * 32 + c8 * 8, qq);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[i] = fmaf(qq[e], kk[e], acc[i]);
        }
    }
    const float slope = ALIBI ? alibi_slope(A.alibi, u % A.H, A.H) : 0.f;
    float p[4], m[4], l[4], o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float s = fold2(acc[i], acc[i]) * A.scale;
        const float logit = ALIBI ? fmaf(-slope, (float)(33 + q0 + i - key), s) : s;   // query t0 + 1 + q0 + i, key t0 - 32 + key
        m[i] = fast_max(logit);
        p[i] = __expf(logit - m[i]);
        l[i] = 0.5f * fast_sum(p[i]);   // both halves hold every key
        o[i] = 0.f;
    }
#pragma unroll
    for (int j0 = 0; j0 < 32; j0 += 8) {
        float vv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) vv[e] = bf16_to_f32(wv[(j0 + e) * kHeadDim + lane]);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) o[i] = fmaf(lane_bcast(p[i], j0 + e), vv[e], o[i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (q0 + i >= nq) break;
        const size_t idx = partial_index(0, partial_slot(A.log2_pmin, t0 + q0 + i), A.slots, A.BH, u);
        if (lane == 0) { W.pm[idx] = m[i]; W.pl[idx] = l[i]; }
        W.po[idx * kHeadDim + lane] = o[i];
    }
}

// Dynamic LDS of the kernel, in bytes from its start.
struct GroupLds {
    int wo, wkv, red, sqh, xs, gain, flag, win_k, win_v, pre, tiles, all;
};
__host__ __device__ constexpr GroupLds group_lds(int KSD, int win_rows)
{
    GroupLds L = {};
    int o = 0;
    L.wo = o; o += frags_o(KSD) * 1024;
    L.wkv = o; o += frags_kv(KSD) * 1024;
    L.red = o; o += 2 * kPW * 256 * 4;
    L.sqh = o; o += kPW * kGroupRows * 4;
    L.xs = o; o += 16 * kGroupRows * 4;
    L.gain = o; o += 2 * 16 * 4;
    L.flag = o; o += 16;
    L.win_k = o; o += win_rows * (kHeadDim + 4) * 4;
    L.win_v = o; o += win_rows * kHeadDim * 2;
    L.pre = o; o += 2 * 256 * 4 + 2 * kPreSlot * 4;
    L.tiles = o;
    o += cross_tile_lds_bytes<true>();   // at least the 8 KB of queries of window_block
    L.all = o;
    return L;
}

// optional wall-clock stamps of the first group's workgroups 0 and trace_rank
#define RT_GROUP_STAMP(k)                                                                                               \
    do {                                                                                                                \
        if (A.trace && wave == 0 && lane == 0 && grp == 0 && (rank == 0 || rank == A.trace_rank))                                     \
            A.trace[((size_t)(rank == 0 ? 0 : A.trace_rows) + t) * 16 + (k)] = wall_clock64();                          \
    } while (0)
// Pair (v, vn) of the elements k, k + 1 as a word of heads and, lo words behind it, one of remainders.
__device__ __forceinline__ void word_store_split(unsigned long long *base, unsigned idx, unsigned lo, unsigned tag, float v, float vn)
{
    const unsigned h = pack_bf16(v, vn);
    word_store(base, idx, tag, h);
    word_store(base, idx + lo, tag, pack_bf16(v - __uint_as_float(h << 16), vn - __uint_as_float(h & 0xFFFF0000u)));
}

// KSD = d / 256; BM: sequences per group the exchanged vectors are laid out for (1, 2 or 4).
// HP: the inputs of the four products cross the chip as bf16 head and remainder (16 bits and more of each value), the gains are applied to
// them and not to the weights, the mean square of h is that of the unrounded rows, gelu and the softmax use the exact functions - the
// arithmetic of rt_wavefront.hip, for stacks.  Otherwise one bf16 per value and gains in the weights, as in rt_persistent.hip.
template <int KSD, int BM, bool ALIBI, bool HP>
__global__ __launch_bounds__(kPThreads) void group_kernel(GroupArgs A)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int xcd = blockIdx.x & 7, grp = xcd >> 1;
    const int rank = (int)(blockIdx.x >> 3) + ((xcd & 1) << 5);
    constexpr int d = 256 * KSD, RO = 4 * KSD, R1 = 16 * KSD, RKV = 8 * KSD, TKV = kv_tiles(KSD);
    constexpr int CD = chunks_d(KSD), CF = chunks_F(KSD), LD = d / kPW, LF = 4 * d / kPW;
    GroupWork W = A.w[grp];
    const int B = W.B;
    if (B == 0) return;
    W.packed = as_global(W.packed); W.g_k = as_global(W.g_k); W.x = as_global(W.x); W.y = as_global(W.y);
    W.K = as_global(W.K); W.V = as_global(W.V); W.Q = as_global(W.Q); W.Vt = as_global(W.Vt); W.Qf = as_global(W.Qf);
    W.Ktf = as_global(W.Ktf); W.Klo = as_global(W.Klo); W.Kh = as_global(W.Kh); W.VT = as_global(W.VT); W.pm = as_global(W.pm);
    W.pl = as_global(W.pl); W.po = as_global(W.po); W.far_m = as_global(W.far_m); W.far_l = as_global(W.far_l); W.far_o = as_global(W.far_o);

    const GroupLds L = group_lds(KSD, A.win_rows);
    const uint4 *wo_s = reinterpret_cast<const uint4 *>(smem + L.wo) + wave * CD * 128;
    const uint4 *wkv_s = reinterpret_cast<const uint4 *>(smem + L.wkv) + wave * CD * 128;
    float *red0 = reinterpret_cast<float *>(smem + L.red), *red1 = red0 + kPW * 256;   // [kPW][64][4], phases in turn
    float *sqh = reinterpret_cast<float *>(smem + L.sqh);        // [kPW][4]
    float *xs = reinterpret_cast<float *>(smem + L.xs);          // [16][4]
    float *gain_s = reinterpret_cast<float *>(smem + L.gain);    // [2][16] gains of the workgroup's rows of h and of z
    int *flag_s = reinterpret_cast<int *>(smem + L.flag);
    float *win_k = reinterpret_cast<float *>(smem + L.win_k);    // [win_rows][64 + 4] unrounded keys
    bf16_t *win_v = reinterpret_cast<bf16_t *>(smem + L.win_v);  // [win_rows][64]
    float *pre_s = reinterpret_cast<float *>(smem + L.pre), *pre_in = pre_s + 512;   // states and inputs of two queries

    GroupWait G;
    G.spin_limit = A.spin_limit;
    G.bar = as_global(A.bar) + grp * 16;
    unsigned long long *words = as_global(A.words) + grp * A.group_stride;
    constexpr GroupWords X = group_words(d, HP);

    const uint4 *packed = reinterpret_cast<const uint4 *>(W.packed) + (size_t)rank * frags_all(KSD) * 64;
    const uint4 *p_1 = packed + (size_t)frags_o(KSD) * 64, *p_2 = p_1 + (size_t)frags_1(KSD) * 64;
    {
        uint4 *dst = reinterpret_cast<uint4 *>(smem + L.wo);
        for (int i = tid; i < frags_o(KSD) * 64; i += kPThreads) dst[i] = packed[i];
        const uint4 *p_kv = p_2 + (size_t)frags_2(KSD) * 64;
        dst = reinterpret_cast<uint4 *>(smem + L.wkv);
        for (int i = tid; i < frags_kv(KSD) * 64; i += kPThreads) dst[i] = p_kv[i];
    }
    // "a wavefront of this workgroup gave up waiting", or (stacks, many launches) a wait of this group expired earlier in the call
    if (tid == 0) flag_s[1] = HP ? ll_load(G.bar + 8) != 0 : 0;
    if (HP && tid < 2 * 16) {
        const bf16_t *g = as_global(A.gains[grp][tid >> 4]);
        const int r = tid & 15;
        gain_s[tid] = g && r < RO ? bf16_to_f32(g[rank * RO + r]) : 1.f;
    }

    const size_t rs = (size_t)A.BH * kHeadDim;
    const int units = B * A.H;                  // (sequence, head) pairs of the group; this workgroup owns number `rank`
    const bool has_u = rank < units;
    const int ub = rank / A.H, uh = rank - ub * A.H;                    // local batch row and head
    const int ug = (W.b0 + W.bstep * ub) * A.H + uh;                    // the pair's number in the tensors
    const float my_gk = (has_u && W.g_k) ? bf16_to_f32(W.g_k[uh * kHeadDim + lane]) : 1.f;
    const bool is_owner = has_u && wave == 0, is_helper = has_u && wave == 4, is_fetcher = has_u && wave == 5;
    const bool far = W.far_m != nullptr;
    unsigned long long nbar = 0;
    // the window's newest key of the next query, kept by the owner: its logit and its value
    float s1 = 0.f, v1 = 0.f;

    __syncthreads();
    if (HP && flag_s[1] != 0) return;   // the whole workgroup
    if (is_helper) {
        pre_fetch(A, W, 0, ug, pre_in, lane);
        wave_sync_lds();
        pre_merge<ALIBI, HP>(A, far, 0, ug, pre_in, win_k, win_v, pre_s, lane);
    }
    __syncthreads();

    // Phase M of position t: the pair of position t - 1 is finished, its key folded into the pre-merged state of query t.
    auto phase_m = [&](int t, int &fail) {
        const int par = t & 1, ppar = par ^ 1;
        const unsigned tag = A.tag_base | (unsigned)(t + 1), ptag = A.tag_base | (unsigned)t;
        int ln = lane;
        asm volatile("" : "+v"(ln));   // opaque: the addresses below are formed here and not kept in registers
        if (is_owner) {
            const float *st = pre_s + par * 256;
            const float q = st[ln];
            float m = st[64 + ln], l = st[128 + ln], o = st[192 + ln];
            float kr = 0.f;
            bf16_t kb = 0, vb = 0;
            if (t >= 1) {
                const unsigned long long *wp = words + ppar * X.all;
                const unsigned ko = uh * kHeadDim + ln, vo = d + ko;
                const unsigned long long *wz = wp + X.zss, *wkv = wp + X.kv;
                const ll_t *p[3] = {wz + (size_t)(ln * BM + ub), wkv + (size_t)((ko / RKV * BM + ub) * RKV + ko % RKV),
                                    wkv + (size_t)((vo / RKV * BM + ub) * RKV + vo % RKV)};
                const bool act[3] = {true, true, true};
                ll_t w3[3];
                if (((t - 1) & (A.p_min - 1)) != 0) {   // key t - 2, the newest of the window
                    const float mn = fmaxf(m, s1);
                    const float e1 = merge_exp<HP>(m - mn), e2 = merge_exp<HP>(s1 - mn);
                    l = l * e1 + e2;
                    o = o * e1 + v1 * e2;
                    m = mn;
                }
                ll_wait_n<3>(p, act, ptag, G, w3, fail);
                const float k0 = __uint_as_float((unsigned)w3[1]);
                const float kg = A.norm_free ? k0 : k0 * my_gk;
                const float Sz = fast_sum(__uint_as_float((unsigned)w3[0])), Sk = fast_sum(k0 * k0), Sq = fast_sum(q * kg);
                const float rz = A.norm_free ? 1.f : rsqrtf(Sz / (float)d + A.eps);
                const float kscale = A.norm_free ? 1.f : rz * rsqrtf(rz * rz * Sk / (float)kHeadDim + A.eps);
                kr = kg * kscale;
                const float vr = __uint_as_float((unsigned)w3[2]) * rz;
                kb = f32_to_bf16(kr);
                vb = f32_to_bf16(vr);
                if (t < W.N) {   // the newest key is one position before the query
                    const float sn = ALIBI ? A.scale * (Sq * kscale) - alibi_slope(A.alibi, uh, A.H) : A.scale * (Sq * kscale);
                    const float m_new = fmaxf(m, sn);
                    const float e1 = merge_exp<HP>(m - m_new), e2 = merge_exp<HP>(sn - m_new);
                    l = l * e1 + e2;
                    o = o * e1 + bf16_to_f32(vb) * e2;
                }
            }
            if (t < W.N) {
                const float av = HP ? o / l : o * __builtin_amdgcn_rcpf(l);   // (one bf16: the rounding hides the reciprocal's)
                const float an = dpp_odd_neighbour(av);
                if (!(ln & 1)) {
                    const unsigned at = piece_word<8, BM>(uh * kHeadDim + ln, ub);
                    if (HP) word_store_split(words + par * X.all + X.a, at, (unsigned)X.lo, tag, av, an);
                    else word_store(words + par * X.all + X.a, at, tag, (unsigned)f32_to_bf16(av) | ((unsigned)f32_to_bf16(an) << 16));
                }
            }
            // the rest follows a: only a is on the critical path of the position
            if (t >= 1) {
                v1 = bf16_to_f32(vb);
                if (t + 1 < W.N && (t & (A.p_min - 1)) != 0) {   // key t - 1 is two positions before query t + 1
                    s1 = A.scale * fast_sum(pre_in[((t + 1) & 1) * kPreSlot + ln] * kr);
                    if (ALIBI) s1 -= 2.f * alibi_slope(A.alibi, uh, A.H);
                }
                const size_t row = (size_t)(t - 1) * rs;
                const unsigned off = (unsigned)(ug * kHeadDim + ln);
                (W.K + row)[off] = kb;
                (W.V + row)[off] = vb;
                (W.Klo + row)[off] = f32_to_bf16(kr - bf16_to_f32(kb));   // what the stored bf16 key lost
                (W.Kh + row)[off] = f32_to_f16_bits(kr);
                const int slot = (t - 1) & (A.win_rows - 1);      // ring slot of key t-1; this workgroup alone reads it back
                win_k[slot * (kHeadDim + 4) + ln] = kr;
                win_v[slot * kHeadDim + ln] = vb;
                // the transposed value copy from the ring: 32 positions of a head dimension at a time, the last, incomplete
                // group two bytes at a time at the end
                if ((t & 31) == 0) {
                    bf16_t *dst = W.VT + ((size_t)ug * kHeadDim + ln) * A.vt_stride + (t - 32);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        uint32_t w[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int s0 = (t - 32 + 8 * j + 2 * i) & (A.win_rows - 1), s2 = (t - 31 + 8 * j + 2 * i) & (A.win_rows - 1);
                            w[i] = (uint32_t)win_v[s0 * kHeadDim + ln] | ((uint32_t)win_v[s2 * kHeadDim + ln] << 16);
                        }
                        *reinterpret_cast<uint4 *>(dst + 8 * j) = make_uint4(w[0], w[1], w[2], w[3]);
                    }
                } else if (t == W.N) {
                    for (int k = t & ~31; k < t; ++k)
                        W.VT[((size_t)ug * kHeadDim + ln) * A.vt_stride + k] = win_v[(k & (A.win_rows - 1)) * kHeadDim + ln];
                }
            }
        } else if (wave == 1) {   // the residual input of phase O, ahead of it and away from the merging wavefront's polls
            if (t < W.N && (ln >> 2) < RO && (ln & 3) < B) xs[ln] = bf16_to_f32(W.x[((size_t)(W.b0 + W.bstep * (ln & 3)) * A.rows + t) * d + rank * RO + (ln >> 2)]);
        } else if (is_helper) {
            // (behind an event the stored states of the next query are complete only there)
            if ((t & (A.p_min - 1)) != 0 && t + 1 < W.N)
                pre_merge<ALIBI, HP>(A, far, t + 1, ug, pre_in + ((t + 1) & 1) * kPreSlot, win_k, win_v, pre_s + ppar * 256, ln);
        } else if (is_fetcher) {
            if ((t & (A.p_min - 1)) != 0 && ((t + 1) & (A.p_min - 1)) != 0 && t + 2 < W.N)
                pre_fetch(A, W, t + 2, ug, pre_in + (t & 1) * kPreSlot, ln);
        }
    };

    int fail = 0;
    phase_m(0, fail);
    RT_GROUP_SYNC(fail);

    // W1 and W2 fragments of this wavefront's eighth of the contraction
    WFrag w1[KSD][CD][2], w2[CF][2];
    auto load_weights = [&]() {
#pragma unroll
        for (int i = 0; i < KSD; ++i)
#pragma unroll
            for (int m = 0; m < CD; ++m)
#pragma unroll
                for (int j = 0; j < 2; ++j) w1[i][m][j].u = p_1[(((i * kPW + wave) * CD + m) * 2 + j) * 64 + lane];
#pragma unroll
        for (int m = 0; m < CF; ++m)
#pragma unroll
            for (int j = 0; j < 2; ++j) w2[m][j].u = p_2[((wave * CF + m) * 2 + j) * 64 + lane];
    };
    load_weights();

    for (int t0 = 0; t0 < W.N; t0 += A.p_min) {
        // ================================================================ cross-block items of the block ending at key t0 - 1
        if (t0 > 0 && t0 < W.N - 1) {
            const int P = t0 & -t0;
            const int nq = min(P, W.N - 1 - t0);
            int level = A.log2_pmin;
            while ((1 << level) < P) ++level;
            unsigned char *tiles = smem + L.tiles;
            int tid_o = tid;
            asm volatile("" : "+v"(tid_o));   // opaque: keeps the tile's lane-derived addresses out of the other phases' registers
            auto tile = [&](int bh, int q0) {
                cross_tile_wg<true, kPW, 1, ALIBI>(W.Q, W.Qf, W.K, reinterpret_cast<const bf16_t *>(W.Kh), W.VT, A.vt_stride, W.pm, W.pl,
                                                   W.po, A.BH, bh, t0, 1, t0 - P, P, q0, nq, level, level - A.log2_pmin, A.slots,
                                                   A.scale, tiles, tid_o, ALIBI ? alibi_slope(A.alibi, bh % A.H, A.H) : 0.f);
            };
            if (P < kGroupSpreadP) {
                // Small blocks stay inside the workgroup that owns the (b, h): it stored all their keys and values and reads
                // the partial states itself, workgroup-scope fences suffice.
                if (has_u) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    __syncthreads();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                    if (P == 32) {
                        window_block<ALIBI>(A, W, t0, nq, ug, win_k, win_v, reinterpret_cast<float *>(tiles) + wave * 256, wave, tid_o & 63);
                    } else {
                        for (int q0 = 0; q0 < nq; q0 += 32 * kPW) {
                            tile(ug, q0 + wave * 32);
                            __syncthreads();   // the next pass overwrites the tiles
                        }
                        load_weights();   // the tile had their registers
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    __syncthreads();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                }
            } else {
                if (grid_barrier(G, (++nbar) * (unsigned long long)kGroupRanks, flag_s)) fail = 1;
                RT_GROUP_SYNC(fail);
                const int qgroups = (nq + 32 * kPW - 1) / (32 * kPW);
                for (int it = rank; it < units * qgroups; it += kGroupRanks) {
                    const int ul = it % units, qg = it / units;
                    const int lb = ul / A.H;
                    tile((W.b0 + W.bstep * lb) * A.H + ul - lb * A.H, qg * 32 * kPW + wave * 32);
                    __syncthreads();   // the next item overwrites the tiles
                }
                if (grid_barrier(G, (++nbar) * (unsigned long long)kGroupRanks, flag_s)) fail = 1;
                RT_GROUP_SYNC(fail);
                load_weights();
            }
        }
        if (is_helper && t0 + 1 < W.N) {   // the stored states of the next queries are complete now
            pre_fetch(A, W, t0 + 1, ug, pre_in + ((t0 + 1) & 1) * kPreSlot, lane);
            wave_sync_lds();
            pre_merge<ALIBI, HP>(A, far, t0 + 1, ug, pre_in + ((t0 + 1) & 1) * kPreSlot, win_k, win_v, pre_s + ((t0 + 1) & 1) * 256, lane);
        } else if (is_fetcher && t0 + 2 < W.N) {
            pre_fetch(A, W, t0 + 2, ug, pre_in + (t0 & 1) * kPreSlot, lane);
        }

        const int t1 = min(W.N, t0 + A.p_min);
        for (int t = t0; t < t1; ++t) {
            const unsigned tag = A.tag_base | (unsigned)(t + 1);
            unsigned long long *wp = words + (t & 1) * X.all;
            RT_GROUP_STAMP(0);
            // opaque: what depends on the lane is formed in every position, registers are for the weights
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const int erow = ln >> 2, eb = ln & 3;   // epilogue rows of wavefront 0 in phases O and 2
            const bool e_own = erow < RO && eb < B;
            // ============================================================ phase O:  h = x_t + alpha Wo a
            {
                WFrag w[CD][2];
#pragma unroll
                for (int m = 0; m < CD; ++m)
#pragma unroll
                    for (int j = 0; j < 2; ++j) w[m][j].u = lds_load16(wo_s + (m * 2 + j) * 64 + ln);
                Piece act[CD], rem[CD];
                float none;
                if constexpr (HP) slice_pull_split<CD, LD, 8, BM, false>(wp + X.a, (unsigned)X.lo, wp, wave, ln, B, tag, G, act, rem, none, fail, A.sl_o);
                else slice_pull<CD, LD, 8, BM>(wp + X.a, wave, ln, B, tag, G, act, fail, A.sl_o);
                RT_GROUP_STAMP(1);
                f32x4_t acc[4] = {};
#pragma unroll
                for (int m = 0; m < CD; ++m) {
                    chunk_product4(act[m], w[m][0], w[m][1], acc);
                    if constexpr (HP) chunk_product4(rem[m], w[m][0], w[m][1], acc);
                }
                const f32x4_t s[1] = {(acc[0] + acc[1]) + (acc[2] + acc[3])};
                tiles_store<1>(red0, wave, ln, s);
            }
            RT_GROUP_SYNC(fail);
            RT_GROUP_STAMP(2);
            float hv = 0.f;
            if (wave == 0) {
                hv = xs[ln] + A.alpha * tile_sum(red0, ln);
                const float hg = HP ? hv * gain_s[erow] : hv;
                const float hn = row_partner(hg);
                if (e_own && !(erow & 1)) {
                    const unsigned at = piece_word<1, BM>(rank * RO + erow, eb);
                    if (HP) word_store_split(wp + X.h, at, (unsigned)X.lo, tag, hg, hn);
                    else word_store(wp + X.h, at, tag, (unsigned)f32_to_bf16(hg) | ((unsigned)f32_to_bf16(hn) << 16));
                }
                if (HP) {
                    const float s = sum_mod4(e_own ? hv * hv : 0.f);
                    if (ln < B) word_store(wp + X.hss, rank * BM + ln, tag, __float_as_uint(s));
                }
            }
            RT_GROUP_STAMP(3);
            __syncthreads();

            // ============================================================ phase 1:  u = gelu(W1 h / rms(h))
            {
                Piece act[CD], rem[CD];
                float ss = 0.f;   // |h|^2: the partial sums of its producers, or of the received values
                if constexpr (HP)
                    slice_pull_split<CD, LD, 1, BM, true>(wp + X.h, (unsigned)X.lo, wp + X.hss, wave, ln, B, tag, G, act, rem, ss, fail, A.sl_1);
                else
                    slice_pull<CD, LD, 1, BM>(wp + X.h, wave, ln, B, tag, G, act, fail, A.sl_1);
                RT_GROUP_STAMP(4);
                f32x4_t acc[KSD] = {};
#pragma unroll
                for (int m = 0; m < CD; ++m) {
#pragma unroll
                    for (int i = 0; i < KSD; ++i) acc[i] = mfma4<0>(act[m], w1[i][m][0].h[0], acc[i]);
#pragma unroll
                    for (int i = 0; i < KSD; ++i) acc[i] = mfma4<1>(act[m], w1[i][m][0].h[1], acc[i]);
#pragma unroll
                    for (int i = 0; i < KSD; ++i) acc[i] = mfma4<2>(act[m], w1[i][m][1].h[0], acc[i]);
#pragma unroll
                    for (int i = 0; i < KSD; ++i) acc[i] = mfma4<3>(act[m], w1[i][m][1].h[1], acc[i]);
                    if constexpr (HP) {
#pragma unroll
                        for (int i = 0; i < KSD; ++i) acc[i] = chunk_product(rem[m], w1[i][m][0], w1[i][m][1], acc[i]);
                    }
                }
                if constexpr (!HP) {
#pragma unroll
                    for (int m = 0; m < CD; ++m) {
                        const bf16x2_t p0 = __builtin_bit_cast(bf16x2_t, act[m].u.x), p1 = __builtin_bit_cast(bf16x2_t, act[m].u.y);
                        ss = __builtin_amdgcn_fdot2_f32_bf16(p0, p0, ss, false);
                        ss = __builtin_amdgcn_fdot2_f32_bf16(p1, p1, ss, false);
                    }
                    ss = sum_mod4(ss);
                }
                if (ln < (HP ? BM : 4)) sqh[wave * 4 + ln] = ss;
                tiles_store<KSD>(red1, wave, ln, acc);
            }
            RT_GROUP_SYNC(fail);
            RT_GROUP_STAMP(5);
            if (wave < R1 / 16) {
                const int tn = wave * 64 + ln, row = tn >> 2, b = ln & 3;
                float s = 0.f;
#pragma unroll
                for (int w = 0; w < kPW; ++w) s += sqh[w * 4 + b];
                const float rinv = A.norm_free ? 1.f : rsqrtf(s / (float)d + A.eps);
                const float pre = tile_sum(red1, tn) * rinv;
                const float uv = HP ? gelu_erf(pre) : gelu_bf16_out(pre);
                const float un = row_partner(uv);
                if (!(row & 1) && b < B) {
                    const unsigned at = piece_word<1, BM>(rank * R1 + row, b);
                    if (HP) word_store_split(wp + X.u, at, (unsigned)X.lo, tag, uv, un);
                    else word_store(wp + X.u, at, tag, (unsigned)f32_to_bf16(uv) | ((unsigned)f32_to_bf16(un) << 16));
                }
            }
            RT_GROUP_STAMP(6);
            __syncthreads();
            RT_GROUP_STAMP(7);

            // ============================================================ phase 2:  z = h + alpha W2 u
            {
                Piece act[CF], rem[CF];
                float none;
                if constexpr (HP) slice_pull_split<CF, LF, 1, BM, false>(wp + X.u, (unsigned)X.lo, wp, wave, ln, B, tag, G, act, rem, none, fail, A.sl_2);
                else slice_pull<CF, LF, 1, BM>(wp + X.u, wave, ln, B, tag, G, act, fail, A.sl_2);
                RT_GROUP_STAMP(8);
                f32x4_t acc[4] = {};
#pragma unroll
                for (int m = 0; m < CF; ++m) {
                    chunk_product4(act[m], w2[m][0], w2[m][1], acc);
                    if constexpr (HP) chunk_product4(rem[m], w2[m][0], w2[m][1], acc);
                }
                const f32x4_t s[1] = {(acc[0] + acc[1]) + (acc[2] + acc[3])};
                tiles_store<1>(red0, wave, ln, s);
            }
            RT_GROUP_SYNC(fail);
            RT_GROUP_STAMP(9);
            if (wave == 0) {
                const float zv = hv + A.alpha * tile_sum(red0, ln);
                const float zg = HP ? zv * gain_s[16 + erow] : zv;   // (without HP the gain of RMS(z) is in the stationary Wk, Wv)
                const float zn = row_partner(zg);
                if (e_own && !(erow & 1)) {
                    const unsigned at = piece_word<1, BM>(rank * RO + erow, eb);
                    if (HP) word_store_split(wp + X.z, at, (unsigned)X.lo, tag, zg, zn);
                    else word_store(wp + X.z, at, tag, (unsigned)f32_to_bf16(zg) | ((unsigned)f32_to_bf16(zn) << 16));
                }
                const float s = sum_mod4(e_own ? zv * zv : 0.f);
                if (ln < B) word_store(wp + X.zss, rank * BM + ln, tag, __float_as_uint(s));
                if (e_own) (W.y + (size_t)t * d)[(size_t)(W.b0 + W.bstep * eb) * A.rows * d + (unsigned)(rank * RO + erow)] = f32_to_bf16(zv);
            }
            RT_GROUP_STAMP(10);
            __syncthreads();

            // ============================================================ phase KV:  [Wk; Wv] (z g_kv)
            {
                WFrag w[TKV][CD][2];
#pragma unroll
                for (int i = 0; i < TKV; ++i)
#pragma unroll
                    for (int m = 0; m < CD; ++m)
#pragma unroll
                        for (int j = 0; j < 2; ++j) w[i][m][j].u = lds_load16(wkv_s + ((i * kPW * CD + m) * 2 + j) * 64 + ln);
                Piece act[CD], rem[CD];
                float none;
                if constexpr (HP) slice_pull_split<CD, LD, 1, BM, false>(wp + X.z, (unsigned)X.lo, wp, wave, ln, B, tag, G, act, rem, none, fail, A.sl_kv);
                else slice_pull<CD, LD, 1, BM>(wp + X.z, wave, ln, B, tag, G, act, fail, A.sl_kv);
                RT_GROUP_STAMP(11);
                f32x4_t acc[TKV] = {};
#pragma unroll
                for (int m = 0; m < CD; ++m)
#pragma unroll
                    for (int i = 0; i < TKV; ++i) {
                        acc[i] = chunk_product(act[m], w[i][m][0], w[i][m][1], acc[i]);
                        if constexpr (HP) acc[i] = chunk_product(rem[m], w[i][m][0], w[i][m][1], acc[i]);
                    }
                tiles_store<TKV>(red1, wave, ln, acc);
            }
            RT_GROUP_SYNC(fail);
            RT_GROUP_STAMP(12);
            if (wave < (RKV + 15) / 16) {
                const int tn = wave * 64 + ln, row = tn >> 2, b = ln & 3;
                if (b < B && row < RKV) word_store(wp + X.kv, (rank * BM + b) * RKV + row, tag, __float_as_uint(tile_sum(red1, tn)));
            }
            RT_GROUP_STAMP(13);
            // ============================================================ phase M of the next position
            phase_m(t + 1, fail);
            RT_GROUP_STAMP(14);
            RT_GROUP_SYNC(fail);
            RT_GROUP_STAMP(15);
        }
    }
    RT_GROUP_SYNC(fail);
}

// The loop matrices in the fragment order above, with the gains given folded in (W diag(g), rounded once).  Lane l of fragment (tile, wave,
// chunk m, j) holds W[row0 + 16 tile + l%16][k .. k + 3] and [k + 4 .. k + 7], k = wave * (K / 8) + 64 m + 16 (l/16) + 8 j;
// rows beyond the workgroup's and indices beyond the wavefront's share are zero.
__global__ __launch_bounds__(256) void group_pack_kernel(const bf16_t *Wo, const bf16_t *W1, const bf16_t *W2, const bf16_t *Wk,
                                                         const bf16_t *Wv, const bf16_t *g_mlp, const bf16_t *g_kv, int KSD, uint4 *dst)
{
    const int per = frags_all(KSD), d = 256 * KSD;
    const long long f_all = ((long long)blockIdx.x * 256 + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (f_all >= (long long)per * kGroupRanks) return;
    const int rank = (int)(f_all / per);
    int f = (int)(f_all - (long long)rank * per);
    const bf16_t *src = nullptr, *gain = nullptr;
    int chunks = chunks_d(KSD), row = 0, rows, K = d;
    bool pairs = false;
    if (f < frags_o(KSD)) {
        rows = 4 * KSD; src = Wo;
    } else if ((f -= frags_o(KSD)) < frags_1(KSD)) {
        rows = 16 * KSD; src = W1; gain = g_mlp;
    } else if ((f -= frags_1(KSD)) < frags_2(KSD)) {
        rows = 4 * KSD; src = W2; chunks = chunks_F(KSD); K = 4 * d;
    } else {
        f -= frags_2(KSD);
        rows = 8 * KSD; gain = g_kv; pairs = true;
    }
    const int j = f & 1, m = (f >> 1) % chunks, w = (f >> 1) / chunks % kPW, tile = (f >> 1) / (chunks * kPW);
    const int kk = 64 * m + 16 * (lane >> 4) + 8 * j;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (tile * 16 + (lane & 15) < rows && kk < K / kPW) {
        row = rank * rows + tile * 16 + (lane & 15);
        if (pairs) { src = row < d ? Wk : Wv; row = row < d ? row : row - d; }
        const int k = w * (K / kPW) + kk;
        v = *reinterpret_cast<const uint4 *>(src + (size_t)row * K + k);
        if (gain) {
            float gg[8], ww[8];
            load8(gain + k, gg);
            load8(reinterpret_cast<const bf16_t *>(&v), ww);
            v.x = pack_bf16(ww[0] * gg[0], ww[1] * gg[1]);
            v.y = pack_bf16(ww[2] * gg[2], ww[3] * gg[3]);
            v.z = pack_bf16(ww[4] * gg[4], ww[5] * gg[5]);
            v.w = pack_bf16(ww[6] * gg[6], ww[7] * gg[7]);
        }
    }
    dst[f_all * 64 + lane] = v;
}

// =============================================================================================
// Host side
// =============================================================================================
// a captured stream must not record memset nodes: words are cleared with a kernel.  The groups' abort words among the first
// counters are kept between the launches of a call: they say that one of its waits expired.
__global__ void group_clear_kernel(unsigned long long *p, size_t n, size_t counters, int keep_abort)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        if (!(keep_abort && i < counters && (i & 15) == 8)) p[i] = 0ULL;
}

typedef void (*group_fn)(GroupArgs);
template <int BM, bool ALIBI, bool HP> static group_fn pick_width(int d)
{
    switch (d) {
    case 256: return group_kernel<1, BM, ALIBI, HP>;
    case 512: return group_kernel<2, BM, ALIBI, HP>;
    case 768: return group_kernel<3, BM, ALIBI, HP>;
    case 1024: return group_kernel<4, BM, ALIBI, HP>;
    default: return nullptr;
    }
}
template <bool ALIBI, bool HP> static group_fn pick_rows(int d, int BM)
{
    return BM == 1 ? pick_width<1, ALIBI, HP>(d) : (BM == 2 ? pick_width<2, ALIBI, HP>(d) : pick_width<4, ALIBI, HP>(d));
}
static group_fn pick_kernel(int d, int BM, bool alibi, bool hp)
{
    if (hp) return alibi ? pick_rows<true, true>(d, BM) : pick_rows<false, true>(d, BM);
    return alibi ? pick_rows<true, false>(d, BM) : pick_rows<false, false>(d, BM);
}
// LDS beyond the default, once per device and kernel: contexts are created often, and the call is not cheap
static bool raise_lds(int device, int d, bool alibi, bool hp)
{
    static std::mutex mu;
    static uint64_t raised[2][2][5] = {};   // a bit per device
    std::lock_guard<std::mutex> lock(mu);
    uint64_t &done = raised[hp][alibi][d / 256];
    const uint64_t bit = 1ULL << (device & 63);
    for (int BM = 1; BM <= kGroupRows && !(done & bit); BM *= 2)
        if (hipFuncSetAttribute((const void *)pick_kernel(d, BM, alibi, hp), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
    done |= bit;
    return true;
}
bool group_stack_kernels(int device, const LayerDims &D) { return raise_lds(device, D.d, D.alibi > 0.f, true); }

size_t group_pack_elements(int d) { return (size_t)kGroupRanks * frags_all(d / 256) * 512; }

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// (the caller has found the device to be one of 256 compute units with cooperative launches: persistent_create)
rt_status group_create(GroupState &P, const rt_config &cfg, const LayerDims &D)
{
    P.available = false;
    if (cfg.dtype != RT_BF16 || (cfg.flags & RT_FLAG_NO_MFMA) || D.F != 4 * D.d || !pick_kernel(D.d, 1, false, false)) return RT_ERR_UNSUPPORTED;
    if (D.p_min != 32) return RT_ERR_UNSUPPORTED;   // a wider window does not fit beside the weights at every width
    P.win_rows = D.p_min;
    P.lds = (size_t)group_lds(D.d / 256, P.win_rows).all;
    if (P.lds > (size_t)160 * 1024) return RT_ERR_UNSUPPORTED;
    if (!raise_lds(cfg.device, D.d, D.alibi > 0.f, false)) return RT_ERR_UNSUPPORTED;
    const int most = kGroups * kGroupRows;
    P.max_batch = cfg.max_batch < most ? cfg.max_batch : most;
    size_t off = 0;
    auto carve = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    const size_t o_bar = carve((size_t)kGroups * 16 * 8);
    P.group_stride = align_up(2 * group_words(D.d, true).all, 32);
    const size_t o_w = carve(P.group_stride * kGroups * 8);
    P.exchange_bytes = off;
    const size_t o_p = carve(group_pack_elements(D.d) * 2);
    const bool want_trace = getenv("RT_PERSIST_TRACE") != nullptr;
    const size_t o_tr = want_trace ? carve((size_t)2 * cfg.max_seq * 16 * 8) : 0;
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
    char *p = (char *)P.slab;
    P.bar = (unsigned long long *)(p + o_bar);
    P.words = (unsigned long long *)(p + o_w);
    P.packed = (bf16_t *)(p + o_p);
    P.trace = want_trace ? (unsigned long long *)(p + o_tr) : nullptr;
    P.trace_rows = want_trace ? cfg.max_seq : 0;
    P.spin.read();
    P.available = true;
    return RT_OK;
}

void group_destroy(GroupState &P)
{
    if (P.slab) (void)hipFree(P.slab);
    P.slab = nullptr;
    P.available = false;
}

size_t group_bytes(const GroupState &P) { return P.slab ? P.slab_bytes : 0; }

bool group_supported(const GroupState &P, const LayerDims &D)
{
    // Laying out the weights (d = 1024: 12 us) takes longer than the groups save on the first positions (us per call, all workgroups /
    // groups, B = 1 .. 16): N = 1 56 - 92 / 58 - 103 at every width; N = 2 d = 256 68 / 65, d = 512 78 / 76, d = 768 91 - 100 / 91 - 100, d = 1024
    // 103 - 111 / 104 - 115; N = 3, d = 1024, B = 16 130 / 129, N = 4 130 / 121
    return P.available && D.B <= P.max_batch && D.N >= (D.d == 1024 ? 3 : 2) && D.N < (1 << 20) - 2;
}

hipError_t group_pack(const LayerDims &D, const Weights &W, bf16_t *packed, bool gains, hipStream_t st)
{
    const int KSD = D.d / 256;
    const long long frags = (long long)frags_all(KSD) * kGroupRanks;
    hipLaunchKernelGGL(group_pack_kernel, dim3((unsigned)((frags + 3) / 4)), dim3(256), 0, st, (const bf16_t *)W.Wo, (const bf16_t *)W.W1,
                       (const bf16_t *)W.W2, (const bf16_t *)W.Wk, (const bf16_t *)W.Wv, gains ? (const bf16_t *)W.g_mlp : nullptr,
                       gains ? (const bf16_t *)W.g_kv : nullptr, KSD, (uint4 *)packed);
    return hipGetLastError();
}

rt_status group_launch(GroupState &P, const LayerDims &D, GroupArgs &A, bool hp, bool first, hipStream_t st, std::string &err)
{
    A.d = D.d; A.H = D.H;
    A.p_min = D.p_min; A.log2_pmin = D.log2_pmin; A.win_rows = P.win_rows;
    A.alpha = D.alpha; A.scale = D.scale; A.eps = D.eps; A.alibi = D.alibi; A.norm_free = D.norm_free;
    A.spin_limit = P.spin.of_launch(); A.bar = P.bar; A.words = P.words; A.group_stride = P.group_stride;
    A.trace_rows = P.trace_rows;
    const char *tw = getenv("RT_PERSIST_TRACE_WG");
    A.trace_rank = tw ? atoi(tw) : kGroupRanks - 1;
    // Waits before the first polls of phases O, 1, 2, KV in units of 4 x 64 clocks (RT_GROUP_SLEEPS, four digits, overrides them).
    // d = 1024, B = 8, N = 2048, ms per call: 0000 17.66, 0010 17.53, 0110 17.50, 0120 17.54, 0011 17.61, 1010 17.85, 1121 17.99
    int sl[4] = {0, 1, 1, 0};
    if (const char *ps = getenv("RT_GROUP_SLEEPS"))
        for (int i = 0; i < 4 && ps[i]; ++i) sl[i] = ps[i] - '0';
    A.sl_o = sl[0]; A.sl_1 = sl[1]; A.sl_2 = sl[2]; A.sl_kv = sl[3];
    int rows = 1;
    for (int g = 0; g < kGroups; ++g) rows = A.w[g].B > rows ? A.w[g].B : rows;
    const int BM = rows > 2 ? 4 : rows;
    // Tags: 1 .. 4094 in turn (fresh buffers hold tag 0).  When the number wraps, words of a call 4094 calls ago (rows of a larger
    // batch) could carry this call's tags: cleared.  A captured launch is replayed with the same number: it has one of its own and
    // clears all words first.
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    hipError_t e = st ? hipStreamIsCapturing(st, &capturing) : hipSuccess;
    if (e != hipSuccess) { err = std::string("hipStreamIsCapturing: ") + hipGetErrorString(e); return RT_ERR_HIP; }
    const bool captured = capturing != hipStreamCaptureStatusNone;
    if (!captured) P.nonce = (P.nonce % 4094u) + 1u;
    A.tag_base = (captured ? 4095u : P.nonce) << 20;
    const bool all = captured || (P.nonce == 1u && P.launched);
    hipLaunchKernelGGL(group_clear_kernel, dim3(all ? 256 : 1), dim3(256), 0, st, P.bar, all ? P.exchange_bytes / 8 : (size_t)kGroups * 16,
                       (size_t)kGroups * 16, first ? 0 : 1);
    e = hipGetLastError();
    if (e != hipSuccess) { err = std::string("group_clear_kernel: ") + hipGetErrorString(e); return RT_ERR_HIP; }
    void *args[] = {&A};
    e = hipLaunchCooperativeKernel((const void *)pick_kernel(D.d, BM, D.alibi > 0.f, hp), dim3(kGroups * kGroupRanks), dim3(kPThreads), args,
                                   (unsigned int)P.lds, st);
    if (e != hipSuccess) { err = std::string("hipLaunchCooperativeKernel: ") + hipGetErrorString(e); return RT_ERR_HIP; }
    P.launched = true;
    return RT_OK;
}

rt_status group_prefill(GroupState &P, const LayerDims &D, const Weights &W, const Scratch &S, const void *x, void *y, void *K, void *V,
                        bool first, hipStream_t st, std::string &err)
{
    hipError_t e = group_pack(D, W, P.packed, !D.norm_free, st);
    if (e != hipSuccess) { err = std::string("group_pack_kernel: ") + hipGetErrorString(e); return RT_ERR_HIP; }
    GroupArgs A = {};
    A.rows = D.N; A.BH = D.B * D.H;
    A.trace = P.trace;
    A.vt_stride = S.vt_stride; A.levels = S.levels; A.slots = S.slots;
    for (int g = 0; g < kGroups; ++g) {
        GroupWork &w = A.w[g];
        w.B = (D.B - g + kGroups - 1) / kGroups;   // sequences g, g + 4, ...
        if (w.B < 0) w.B = 0;
        w.N = D.N;
        w.b0 = g; w.bstep = kGroups;
        w.packed = P.packed;
        w.g_k = (const bf16_t *)W.g_k;
        w.x = (const bf16_t *)x; w.y = (bf16_t *)y; w.K = (bf16_t *)K; w.V = (bf16_t *)V;
        w.Q = (const bf16_t *)S.Q; w.Vt = (const bf16_t *)S.Vt; w.Qf = S.Qf; w.Ktf = S.Ktf; w.Klo = S.Klo; w.Kh = S.Kh; w.VT = S.VT;
        w.pm = S.pm; w.pl = S.pl; w.po = S.po;
        w.far_m = w.far_l = w.far_o = nullptr;
    }
    return group_launch(P, D, A, false, first, st, err);
}

int group_read_trace(GroupState &P, unsigned long long *out, int rows)
{
    if (!P.trace || !out) return 0;
    const int n = rows < 2 * P.trace_rows ? rows : 2 * P.trace_rows;
    if (hipMemcpy(out, P.trace, (size_t)n * 16 * 8, hipMemcpyDeviceToHost) != hipSuccess) return -1;
    return n;
}

int group_wait_expired(GroupState &P)
{
    if (!P.slab || !P.launched) return 0;
    unsigned long long v[kGroups * 16];
    if (hipMemcpy(v, P.bar, sizeof(v), hipMemcpyDeviceToHost) != hipSuccess) return -1;
    for (int g = 0; g < kGroups; ++g)
        if (v[g * 16 + 8] != 0) return 1;
    return 0;
}

}  // namespace rt
