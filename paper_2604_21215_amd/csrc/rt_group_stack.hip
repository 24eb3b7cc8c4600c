// A stack of layers on the grouped engine (rt_group.hip): rt_stack_prefill for up to sixteen sequences.
//
// A layer's queries depend only on its own input, so layer l + 1 can work on a chunk of C positions as soon as layer l has
// finished it.  The four groups of workgroups hold the weights of four layers on chip (or of two layers or of one, for two or four
// shares of the batch) and run one chunk each per step; group_launch is one step.  At a chunk's entry the chunk's queries and temporary pairs
// come from one GEMM over its rows, and one far tile folds all keys before the chunk into its queries (the schedule of
// rt_wavefront.hip: exact, inside the chunk Algorithm 1 as it stands).  When the first layers are through, the groups take the next
// ones: layer l runs on slot l % slots.
//
// Why: the layer-wavefront engine streams every layer's 23 MB (d = 1024) from memory for every position, with five dependent launches
// per position; here a layer's weights are read once per chunk and a position costs five exchanges.
// The vectors are exchanged as bf16 head and remainder (group_kernel's HP form): the arithmetic of the launches, whose products take
// theirs that way.  With one bf16 per value, as rt_layer_prefill has it, the first call below took 130 ms, and its first layer's keys
// and values were 3.0e-3 of their norm from fp64; the launches 1.73e-3, this form 1.73e-3 (storage alone: 1.67e-3).
// Measured (ms per call, launches of rt_wavefront.hip / here): 12 layers, d = 1024, N = 4096, B = 4: 284 / 161; N = 1024, B = 8:
// 112 / 78; N = 128, B = 3: 29.5 / 11.2; 2 layers, N = 1024, B = 2: 33.7 / 13.8.  A position takes 10.9 us in the loop (d = 1024, four
// sequences per group), 1.6 of it for u (128 KB) to arrive.
#include "rt_group.h"
#include "rt_cross_tile.h"
#include "rt_prepass_device.h"

#include <vector>

namespace rt {

constexpr int kStackLevels = 3;    // blocks of 32, 64 and 128 keys inside a chunk
constexpr int kStackSlots = kStackChunk / 2;

// What the launches ahead of a step need of the layers that enter a chunk.
struct StackEntry {
    Weights W;
    const bf16_t *x, *K;
    bf16_t *Q, *Kt, *Vt;
    float *Qf, *Ktf;
    const bf16_t *Kh, *VT;
    float *far_m, *far_l, *far_o;
    int t0, n;                     // first position and length of the chunk
};
struct StackStep {
    StackEntry e[kGroups];
};

template <typename T> __device__ __forceinline__ T *to_global(T *p)
{   // a pointer read out of the arguments by a computed index: global memory
    return (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
}

// grid (ceil(B chunk / 128), ceil(3 H / 2), layers), block 256
__global__ __launch_bounds__(256) void group_stack_prepass_kernel(StackStep S, int B, int rows, int d, int H, float eps, int norm_free)
{
    const StackEntry &E = S.e[blockIdx.z];
    prepass_mfma_body<true>(to_global(E.x), nullptr, to_global((const bf16_t *)E.W.Wq), to_global((const bf16_t *)E.W.Wk),
                            to_global((const bf16_t *)E.W.Wv), to_global((const bf16_t *)E.W.g_attn), to_global((const bf16_t *)E.W.g_q),
                            to_global((const bf16_t *)E.W.g_k), to_global(E.Q), to_global(E.Kt), to_global(E.Vt), to_global(E.Qf),
                            to_global(E.Ktf), B, E.n, (size_t)rows * d, E.t0, d, H, eps, norm_free, blockIdx.x, blockIdx.y);
}

// All keys before the chunk against its queries.  grid (8 * ceil(BH / 8) * ceil(chunk / 128), layers), block 256
template <bool ALIBI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void group_stack_far_kernel(StackStep S, int BH, int nqb, int vt_stride,
                                                                                                         float scale, float alibi, int H)
{
    __shared__ __align__(16) unsigned char lds[2 * cross_tile_lds_bytes<true>()];
    const StackEntry &E = S.e[blockIdx.y];
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int bh = (j / nqb) * 8 + xcd, qb = j % nqb;
    if (bh >= BH || qb * 128 >= E.n) return;   // the whole workgroup leaves together
    // level 30: the slot of a query is its own position; the states of the chunk's first query come first
    const size_t first = (size_t)E.t0 * BH;
    cross_tile_wg<true, 4, 2, ALIBI>(nullptr, to_global(E.Qf), to_global(E.K), to_global(E.Kh), to_global(E.VT), vt_stride,
                                     to_global(E.far_m) - first, to_global(E.far_l) - first, to_global(E.far_o) - first * kHeadDim, BH, bh, E.t0, 0,
                                     0, E.t0, qb * 128 + (int)(threadIdx.x >> 6) * 32, E.n, 30, 0, 0, scale, lds, (int)threadIdx.x,
                                     ALIBI ? alibi_slope(alibi, bh % H, H) : 0.f);
}

__global__ __launch_bounds__(256) void group_stack_poison_kernel(float *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = __uint_as_float(0x7FC00000u);
}

// sequences of one group; groups per layer
static int splits_for(int B, int L)
{
    int s = L >= 3 ? 1 : (L == 2 ? 2 : 4);   // few layers keep the four groups busy with a share of the batch each
    while (s < kGroups && B > s * kGroupRows) s *= 2;
    return s;
}

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

rt_status group_stack_create(GroupStackState &T, const GroupState &P, const LayerDims &D, int device, int max_batch)
{
    if (T.slab || !P.available) return RT_OK;
    if (!group_stack_kernels(device, D)) return RT_ERR_UNSUPPORTED;
    // states of the layers that run at once: at most four sequences of each group
    const int most = kGroups * kGroupRows;
    const size_t BH = (size_t)(4 * max_batch < most ? 4 * max_batch : most) * D.H;
    const size_t far = align_up(BH * kStackChunk * 4, 256), part = align_up(BH * kStackLevels * kStackSlots * 4, 256);
    const size_t pack = align_up(group_pack_elements(D.d) * 2, 256);
    const size_t all = kGroups * pack + (far + part) * (2 + kHeadDim);
    if (hipMalloc(&T.slab, all) != hipSuccess) {
        (void)hipGetLastError();
        T.slab = nullptr;
        return RT_ERR_OOM;
    }
    T.slab_bytes = all;
    char *p = (char *)T.slab;
    for (int g = 0; g < kGroups; ++g, p += pack) T.packed[g] = (bf16_t *)p;
    T.far_m = (float *)p; p += far;
    T.far_l = (float *)p; p += far;
    T.far_o = (float *)p; p += far * kHeadDim;
    T.pm = (float *)p; p += part;
    T.pl = (float *)p; p += part;
    T.po = (float *)p;
    return RT_OK;
}

void group_stack_destroy(GroupStackState &T)
{
    if (T.slab) (void)hipFree(T.slab);
    T.slab = nullptr;
}

bool group_stack_supported(const GroupStackState &T, const GroupState &P, const LayerDims &D, int L)
{
    // ceil(L / slots) N positions here against N + 64 (L - 1) steps of the launches, which carry all layers: a position costs 9 to
    // 12.5 us (d = 256 to 1024), a step 25 us and more (34 with up to three layers), with d = 1024 from 50 us where the ratio of the
    // two counts is large (twelve layers, or nine sequences and more).  Measured, launches / here, by that ratio (134 shapes, B = 1 .. 16,
    // L = 1 .. 24, N = 128 .. 4096):
    //   d < 1024: up to 2.5 1.13 - 3.1 times, 2.6 - 2.8 1.00 - 1.73, 2.8 - 3.1 0.89 - 1.40, 3.3 - 3.7 0.93 - 1.29, 3.9 - 5.6 0.76 - 1.03;
    //             three layers at every ratio (up to 2.8) 1.26 - 2.1
    //   d = 1024: up to 3.6 1.21 - 4.0, 4.4 - 5.2 0.99 - 1.30
    // (0.76: d = 768, B = 5, N = 4096, 12 layers, 208.6 / 275.3 ms; 4.0: one layer, B = 16, N = 2048, 101.9 / 25.4 ms.)
    if (!T.slab || !P.available || D.B > kGroups * kGroupRows || D.N >= (1 << 20) - 2) return false;
    // one layer and one or two positions: 58 - 104 us as launches, 68 - 120 here at N = 1; B = 1, N = 2, d = 1024 129 / 131, but B = 16 187 / 148
    if (L == 1 && D.N < (D.B <= kGroupRows ? 3 : 2)) return false;
    const int slots = kGroups / splits_for(D.B, L);
    const long long here = (long long)((L + slots - 1) / slots) * D.N, steps = D.N + 64LL * (L - 1);
    return L <= 3 || 100 * here <= (D.d == 1024 ? 440 : 275) * steps;
}

rt_status group_stack_prefill(GroupStackState &T, GroupState &P, const LayerDims &D, const WaveLayer *layers, int L, bool poison,
                              hipStream_t st, std::string &err)
{
    const int splits = splits_for(D.B, L), slots = kGroups / splits, BH = D.B * D.H;
    const size_t far_set = (size_t)kStackChunk * BH, part_set = (size_t)kStackLevels * kStackSlots * BH;   // one slot's states
    auto hip_fail = [&](hipError_t e, const char *where) {
        err = std::string(where) + ": " + hipGetErrorString(e);
        return RT_ERR_HIP;
    };
    // A chunk costs a fixed time (launches, weights into LDS and registers, 0.1 ms and more), the last layers wait three chunks for their
    // input: the sum is least near C^2 = (passes over the groups) N * fixed / (3 * time of a position)
    const long long passes = (L + slots - 1) / slots;
    int C = 64;
    while (C < kStackChunk && 2LL * C * C * 10 <= 28 * passes * D.N) C *= 2;
    if (const char *s = getenv("RT_GROUP_CHUNK")) {   // 64, 128 or 256 instead
        const int v = atoi(s);
        if (v == 64 || v == 128 || v == 256) C = v;
    }
    const int nch = (D.N + C - 1) / C;
    if (poison)
        hipLaunchKernelGGL(group_stack_poison_kernel, dim3(1024), dim3(256), 0, st, (float *)T.slab, T.slab_bytes / 4);
    // layer 0: its input is known in full
    hipError_t e = Launch<bf16_t>::prepass(D, layers[0].W, layers[0].S, layers[0].x, D.B, D.N, true, st);
    if (e != hipSuccess) return hip_fail(e, "prepass");

    bool first = true;             // launch of the call
    std::vector<int> done(L, 0);   // chunks of a layer that are finished
    while (done[L - 1] < nch) {
        GroupArgs A = {};
        A.rows = D.N; A.BH = BH;
        A.levels = kStackLevels; A.slots = kStackSlots;
        StackStep pre = {}, far = {};
        int n_pre = 0, n_far = 0, longest = 0;
        int act[kGroups], n_act = 0;
        for (int l = 0; l < L && n_act < slots; ++l)
            if (done[l] < nch && (l == 0 || done[l - 1] > done[l]) && (l < slots || done[l - slots] == nch)) act[n_act++] = l;
        for (int i = 0; i < n_act; ++i) {
            const int l = act[i], slot = l % slots, t0 = done[l] * C;
            const int n = D.N - t0 < C ? D.N - t0 : C;
            const WaveLayer &Y = layers[l];
            if (done[l] == 0 && (e = group_pack(D, Y.W, T.packed[slot], false, st)) != hipSuccess) return hip_fail(e, "group_pack_kernel");
            StackEntry E;
            E.W = Y.W;
            E.x = (const bf16_t *)Y.x; E.K = (const bf16_t *)Y.K;
            E.Q = (bf16_t *)Y.S.Q; E.Kt = (bf16_t *)Y.S.Kt; E.Vt = (bf16_t *)Y.S.Vt; E.Qf = Y.S.Qf; E.Ktf = Y.S.Ktf;
            E.Kh = (const bf16_t *)Y.S.Kh; E.VT = Y.S.VT;
            E.far_m = T.far_m + slot * far_set; E.far_l = T.far_l + slot * far_set; E.far_o = T.far_o + slot * far_set * kHeadDim;
            E.t0 = t0; E.n = n;
            if (slot == 0 && P.trace) A.trace = P.trace + (size_t)t0 * 16;   // rows are positions, of the last layer that group 0 ran
            if (l > 0) pre.e[n_pre++] = E;
            if (t0 > 0) far.e[n_far++] = E;
            longest = n > longest ? n : longest;
            const size_t row = (size_t)t0 * BH * kHeadDim;
            for (int s = 0; s < splits; ++s) {
                GroupWork &w = A.w[slot * splits + s];
                w.B = (D.B - s + splits - 1) / splits;
                w.N = n; w.b0 = s; w.bstep = splits;
                w.packed = T.packed[slot];
                w.g_k = (const bf16_t *)Y.W.g_k;
                A.gains[slot * splits + s][0] = D.norm_free ? nullptr : (const bf16_t *)Y.W.g_mlp;
                A.gains[slot * splits + s][1] = D.norm_free ? nullptr : (const bf16_t *)Y.W.g_kv;
                w.x = (const bf16_t *)Y.x + (size_t)t0 * D.d;
                w.y = (bf16_t *)Y.y + (size_t)t0 * D.d;
                w.K = (bf16_t *)Y.K + row; w.V = (bf16_t *)Y.V + row;
                w.Q = (const bf16_t *)Y.S.Q + row; w.Vt = (const bf16_t *)Y.S.Vt + row;
                w.Qf = Y.S.Qf + row; w.Ktf = Y.S.Ktf + row; w.Klo = Y.S.Klo + row; w.Kh = Y.S.Kh + row;
                w.VT = Y.S.VT + t0;
                w.pm = T.pm + slot * part_set; w.pl = T.pl + slot * part_set; w.po = T.po + slot * part_set * kHeadDim;
                w.far_m = t0 > 0 ? E.far_m : nullptr; w.far_l = E.far_l; w.far_o = E.far_o;
            }
            A.vt_stride = Y.S.vt_stride;
        }
        if (n_pre) {
            hipLaunchKernelGGL(group_stack_prepass_kernel, dim3((unsigned)((D.B * longest + 127) / 128), (unsigned)((3 * D.H + 1) / 2), (unsigned)n_pre),
                               dim3(256), 0, st, pre, D.B, D.N, D.d, D.H, D.eps, D.norm_free);
            if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "group_stack_prepass_kernel");
        }
        if (n_far) {
            const int nqb = (longest + 127) / 128, bh8 = (BH + 7) / 8 * 8;
            const dim3 grid((unsigned)(bh8 * nqb), (unsigned)n_far);
            if (D.alibi > 0.f)
                hipLaunchKernelGGL(group_stack_far_kernel<true>, grid, dim3(256), 0, st, far, BH, nqb, A.vt_stride, D.scale, D.alibi, D.H);
            else
                hipLaunchKernelGGL(group_stack_far_kernel<false>, grid, dim3(256), 0, st, far, BH, nqb, A.vt_stride, D.scale, D.alibi, D.H);
            if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "group_stack_far_kernel");
        }
        const rt_status s = group_launch(P, D, A, true, first, st, err);
        if (s != RT_OK) return s;
        first = false;
        for (int i = 0; i < n_act; ++i) ++done[act[i]];
    }
    return RT_OK;
}

}  // namespace rt
