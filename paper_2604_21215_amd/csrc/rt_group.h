// Interface of the grouped single-launch engine of the sequential loop (rt_group.hip).
#pragma once
#include "../../include/rt.h"
#include "rt_common.h"
#include <string>

namespace rt {

constexpr int kGroups = 4;        // groups of workgroups, two XCDs each
constexpr int kGroupRanks = 64;   // workgroups of a group
constexpr int kGroupRows = 4;     // sequences a group takes at most

// What one group runs: one layer's weights (re-laid by group_pack) and the positions 0 .. N - 1 of the rows
// b0, b0 + bstep, ... of its tensors.  Every pointer is that of position 0.
struct GroupWork {
    int B;                        // sequences (0: the group has no work)
    int N;                        // positions
    int b0, bstep;
    const bf16_t *packed;         // group_pack_elements(d) elements
    const bf16_t *g_k;            // gain of the key normalisation, or null
    const bf16_t *x;
    bf16_t *y, *K, *V;
    const bf16_t *Q, *Vt;
    const float *Qf, *Ktf;
    bf16_t *Klo;
    uint16_t *Kh;
    bf16_t *VT;
    float *pm, *pl, *po;
    const float *far_m, *far_l, *far_o;   // softmax state of the keys before position 0, [N][B H] and [N][B H][64], or null
};

struct GroupArgs {
    int rows;                     // positions between two batch rows of x and y
    int d, H, BH;                 // BH: batch rows times heads of the tensors
    int p_min, log2_pmin, win_rows;
    float alpha, scale, eps, alibi;
    int norm_free;
    int vt_stride, levels, slots;
    unsigned tag_base;
    int sl_o, sl_1, sl_2, sl_kv;  // waits before the first polls, units of 4 x 64 clocks
    long long spin_limit;
    unsigned long long *bar;      // per group 16 words: [0] barrier counter, [8] abort word
    unsigned long long *words;    // exchange words, group_words() per group and parity
    size_t group_stride;          // words between two groups
    // gains of RMS(h) and RMS(z) of each group's layer where they are not in the packed weights, or null (not in GroupWork: two more
    // members there cost the kernels without them 1 %, by other register moves)
    const bf16_t *gains[kGroups][2];
    unsigned long long *trace;    // optional: [2][trace_rows][16] wall-clock stamps
    int trace_rank, trace_rows;
    GroupWork w[kGroups];
};

struct GroupState {
    bool available = false, launched = false;
    void *slab = nullptr;
    size_t slab_bytes = 0, exchange_bytes = 0;
    unsigned long long *bar = nullptr, *words = nullptr;
    bf16_t *packed = nullptr;     // one layer's weights in fragment order
    size_t group_stride = 0;
    SpinLimit spin;
    unsigned nonce = 0;
    int max_batch = 0;            // sequences one launch takes (all groups)
    int win_rows = 0;
    unsigned long long *trace = nullptr;
    int trace_rows = 0;
    size_t lds = 0;
};

size_t group_pack_elements(int d);
rt_status group_create(GroupState &P, const rt_config &cfg, const LayerDims &D);
void group_destroy(GroupState &P);
size_t group_bytes(const GroupState &P);
bool group_supported(const GroupState &P, const LayerDims &D);
// gains: W1 and [Wk; Wv] multiplied by g_mlp and g_kv
hipError_t group_pack(const LayerDims &D, const Weights &W, bf16_t *packed, bool gains, hipStream_t st);
// launches the loop for the work items in A.w (the caller sets them, the tensors' strides and the stamps' place, the rest of A is filled here); hp: the kernels with head and remainder;
// first: the first launch of a call, which alone clears the abort words
rt_status group_launch(GroupState &P, const LayerDims &D, GroupArgs &A, bool hp, bool first, hipStream_t st, std::string &err);
bool group_stack_kernels(int device, const LayerDims &D);   // readies those
rt_status group_prefill(GroupState &P, const LayerDims &D, const Weights &W, const Scratch &S, const void *x, void *y, void *K, void *V,
                        bool first, hipStream_t st, std::string &err);
// A stack of layers on the same kernel (rt_group_stack.hip): the layers run concurrently, one group or two each, a chunk of
// positions apart.
constexpr int kStackChunk = 256;       // positions of a chunk at most
struct GroupStackState {
    void *slab = nullptr;
    size_t slab_bytes = 0;
    bf16_t *packed[kGroups] = {};      // the weights of the layers that are running
    float *far_m = nullptr, *far_l = nullptr, *far_o = nullptr;   // per running layer [kStackChunk][B H] ([64])
    float *pm = nullptr, *pl = nullptr, *po = nullptr;            // and the states of the blocks inside its chunk
};
rt_status group_stack_create(GroupStackState &T, const GroupState &P, const LayerDims &D, int device, int max_batch);
void group_stack_destroy(GroupStackState &T);
bool group_stack_supported(const GroupStackState &T, const GroupState &P, const LayerDims &D, int L);
rt_status group_stack_prefill(GroupStackState &T, GroupState &P, const LayerDims &D, const WaveLayer *layers, int L, bool poison,
                              hipStream_t st, std::string &err);

// fp32 storage, d = 128, 256, 384 (rt_group_f32.hip)
struct GroupF32State {
    bool available = false, launched = false;
    void *slab = nullptr;
    size_t slab_bytes = 0, exchange_bytes = 0, group_stride = 0, lds = 0;
    unsigned long long *bar = nullptr, *words = nullptr;
    void *packed = nullptr;
    long long spin_limit = 0;
    unsigned nonce = 0;
    int groups = 0, max_batch = 0;
};
rt_status group_f32_create(GroupF32State &P, const rt_config &cfg, const LayerDims &D);
void group_f32_destroy(GroupF32State &P);
bool group_f32_supported(const GroupF32State &P, const LayerDims &D);
rt_status group_f32_prefill(GroupF32State &P, const LayerDims &D, const Weights &W, const Scratch &S, const void *x, void *y, void *K, void *V,
                            hipStream_t st, std::string &err);
int group_f32_wait_expired(GroupF32State &P);

int group_read_trace(GroupState &P, unsigned long long *out, int rows);
int group_wait_expired(GroupState &P);

}  // namespace rt
