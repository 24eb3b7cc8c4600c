// Main loop of the bf16 products C[m][n] = sum_k A[m][k] W[n][k] with both operands staged in LDS (the layer's projections of
// Sec. 2.2 when all positions are known: pre-pass, the loop-free layers of Sec. 2.1 / Sec. 6.1, the backward pass's batched
// products; and the products of one position of many sequences).
//
// k-tiles go from global memory straight into a ring of kStages LDS buffers (global_load_lds, 16 bytes per lane: no staging
// registers), kStages - 1 of them in flight while one is used; a wavefront waits for its own loads of the tile it is about to use by
// count, then one workgroup barrier per k-tile says that everybody's loads of it are in and that the buffer about to be refilled
// has been read.  The loads are issued from inline assembly (they write no register): the compiler would wait for ALL loads in
// flight before every read of LDS.  It does not count them, so that its own waits for other loads are never shorter than needed.
//
// A wavefront's load instruction fills 64 consecutive 16-byte slots, so rows cannot be padded; instead slot c of row r holds the
// row's 16-byte piece c ^ swz(r), and fragment reads of eight consecutive rows hit all banks once.
//
// Block tile 64 MT x 64 NT; four wavefronts as 2 x 2, each 32 MT x 32 NT outputs as MT x NT tiles of v_mfma_f32_32x32x16_bf16; KG
// such groups of four share every k-tile's contraction and join their sums at the end.
#pragma once
#include "rt_mfma_device.h"
#include "rt_cross_tile.h"

namespace rt {

template <int MT_, int NT_, int KG_, int KT_, int STAGES_> struct GemmTile {
    static constexpr int MT = MT_, NT = NT_, KG = KG_, KT = KT_, kStages = STAGES_;
    static constexpr int kRows = 64 * MT, kCols = 64 * NT;          // block tile
    static constexpr int kThreads = 256 * KG;
    static constexpr int kPieces = KT / 8;                           // 16-byte pieces per row of a k-tile
    static constexpr int kRowStep = kThreads / kPieces;              // rows one round of loads covers
    static constexpr int kLoadsA = kRows / kRowStep, kLoadsB = kCols / kRowStep;   // per thread and k-tile
    static constexpr int kStageBytes = (kRows + kCols) * KT * 2;
    static constexpr int kLds = kStages * kStageBytes;
    static constexpr int kKs = KT / 16 / KG;                         // 16-index steps of a k-tile per group
    static constexpr int kRegs = 16 / KG;                            // finished registers per tile and wavefront
    static_assert(kRows % kRowStep == 0 && kCols % kRowStep == 0 && kRowStep % 8 == 0 && KT / 16 % KG == 0 && (KG == 1 || KG == 2));
    static_assert((kStages - 2) * (kLoadsA + kLoadsB) < 64, "the load counter has six bits");
    static_assert(KG == 1 || kLds >= 4 * KG * MT * NT * kRegs * 64 * 4, "the join reuses the ring");
    // piece of row r in slot c: c ^ swz(r).  A row of 64 bytes shares its 128 bytes of banks with its neighbour.
    __device__ static int swz(int r) { return kPieces == 4 ? (r >> 1) & 3 : r & 7; }
};
// Many rows: two workgroups per compute unit (72 KB each).  d = 1024, 16384 rows, us: pre-pass / Wo / W2 / W1 176 / 66 / 165 / 255 (W1 is bound by its
// 67 M GELUs and stores), with the tiles staged through registers (staged_mainloop) 181 / 65 / 169 / 258.
using TileMany = GemmTile<4, 2, 1, 32, 3>;
constexpr int kGtRows = TileMany::kRows, kGtCols = TileMany::kCols;

// the sum over the 16 lanes of a row, in every lane of it (rotations within the row: no trip through the LDS crossbar)
__device__ __forceinline__ float sum16(float v)
{
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x128, 0xF, 0xF, false));
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x124, 0xF, 0xF, false));
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x122, 0xF, 0xF, false));
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x121, 0xF, 0xF, false));
    return v;
}

// what a caller hands in need not be aligned to the 16 bytes of a load into LDS: such rows are loaded into registers
inline bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // M0 is reserved: the compiler keeps nothing in it, and is told that it changes
__device__ __forceinline__ void load_to_lds16(uint32_t lds_off, const bf16_t *p)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_off), "v"(p) : "memory", "m0");
}
#pragma clang diagnostic pop
template <int N> __device__ __forceinline__ void wait_loads_and_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// row_a(r), row_b(r): the addresses of k = 0 of row r of the block tile's A and W (16-byte aligned, valid for every r).  K: a
// multiple of the tile's KT.  ring: kLds bytes of LDS.  Register i of acc[mt][nt] afterwards: row 32 MT wm + 32 mt + 8 (i / 4) +
// 4 (lane / 32) + i % 4, column 32 NT wn + 32 nt + lane % 32 of the block tile, wm = wave / 2 % 2, wn = wave % 2; with KG = 2 the
// group g = wave / 4 finishes registers 8 g .. 8 g + 7 and holds their sums in registers 0 .. 7.
// meanwhile(): work of every thread while the first k-tiles are on their way; what it leaves in LDS is visible afterwards.
template <class T, class RowA, class RowB, class Meanwhile>
__device__ __forceinline__ void tiled_mainloop(RowA row_a, RowB row_b, int K, unsigned char *ring, f32x16_t (&acc)[T::MT][T::NT],
                                               Meanwhile meanwhile)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) & 1, wn = wave & 1, kg = wave >> 2;
    const int l32 = lane & 31, hi = lane >> 5;
#pragma unroll
    for (int mt = 0; mt < T::MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < T::NT; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mt][nt][i] = 0.f;

    const int prow = tid / T::kPieces, pc = (tid % T::kPieces) ^ T::swz(prow);
    const bf16_t *ga[T::kLoadsA], *gb[T::kLoadsB];
#pragma unroll
    for (int i = 0; i < T::kLoadsA; ++i) ga[i] = row_a(prow + T::kRowStep * i) + 8 * pc;
#pragma unroll
    for (int i = 0; i < T::kLoadsB; ++i) gb[i] = row_b(prow + T::kRowStep * i) + 8 * pc;
    const uint32_t ring_off = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)ring;
    const int ntiles = K / T::KT;
    int filled = 0;       // k-tiles requested
    uint32_t fill = 0;    // byte offset of the buffer the next one goes to
    auto request = [&]() {
        const uint32_t base = ring_off + fill + 1024u * wave;
#pragma unroll
        for (int i = 0; i < T::kLoadsA; ++i) load_to_lds16(base + 16u * T::kThreads * i, ga[i] + (size_t)filled * T::KT);
#pragma unroll
        for (int i = 0; i < T::kLoadsB; ++i)
            load_to_lds16(base + 16u * T::kThreads * (T::kLoadsA + i), gb[i] + (size_t)filled * T::KT);
        ++filled;
        fill = fill + T::kStageBytes == T::kLds ? 0 : fill + T::kStageBytes;
    };
#pragma unroll
    for (int s = 0; s < T::kStages - 1; ++s)
        if (s < ntiles) request();
    meanwhile();
    // fragment addresses of this lane within a buffer
    const int arow = 32 * T::MT * wm + l32, brow = T::kRows + 32 * T::NT * wn + l32;
    int piece[T::kKs];
#pragma unroll
    for (int ks = 0; ks < T::kKs; ++ks) piece[ks] = 16 * ((2 * (kg * T::kKs + ks) + hi) ^ T::swz(l32));
    uint32_t used = 0;
    for (int t = 0; t < ntiles; ++t) {
        if (t + T::kStages - 2 < ntiles) wait_loads_and_barrier<(T::kStages - 2) * (T::kLoadsA + T::kLoadsB)>();
        else wait_loads_and_barrier<0>();
        if (filled < ntiles) request();
        const unsigned char *buf = ring + used;
#pragma unroll
        for (int ks = 0; ks < T::kKs; ++ks) {
            uint4 fa[T::MT], fb[T::NT];
#pragma unroll
            for (int mt = 0; mt < T::MT; ++mt)
                fa[mt] = *reinterpret_cast<const uint4 *>(buf + (arow + 32 * mt) * (2 * T::KT) + piece[ks]);
#pragma unroll
            for (int nt = 0; nt < T::NT; ++nt)
                fb[nt] = *reinterpret_cast<const uint4 *>(buf + (brow + 32 * nt) * (2 * T::KT) + piece[ks]);
#pragma unroll
            for (int mt = 0; mt < T::MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < T::NT; ++nt) acc[mt][nt] = mfma32u(fa[mt], fb[nt], acc[mt][nt]);
        }
        used = used + T::kStageBytes == T::kLds ? 0 : used + T::kStageBytes;
    }
    if constexpr (T::KG == 2) {   // every wavefront hands the half it does not finish to its partner
        wait_loads_and_barrier<0>();   // the ring has been read
        float *mine = reinterpret_cast<float *>(ring) + (size_t)wave * (T::MT * T::NT * 8 * 64) + lane;
        const float *theirs = reinterpret_cast<const float *>(ring) + (size_t)(wave ^ 4) * (T::MT * T::NT * 8 * 64) + lane;
#pragma unroll
        for (int mt = 0; mt < T::MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < T::NT; ++nt)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float lo = acc[mt][nt][e], up = acc[mt][nt][8 + e];
                    asm("" : "+v"(lo), "+v"(up));   // two values to choose from, not one array with an index (that would go to scratch)
                    mine[((mt * T::NT + nt) * 8 + e) * 64] = kg == 0 ? up : lo;
                    acc[mt][nt][e] = kg == 0 ? lo : up;
                }
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < T::MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < T::NT; ++nt)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[mt][nt][e] += theirs[((mt * T::NT + nt) * 8 + e) * 64];
    }
}

template <class T, class RowA, class RowB>
__device__ __forceinline__ void tiled_mainloop(RowA row_a, RowB row_b, int K, unsigned char *ring, f32x16_t (&acc)[T::MT][T::NT])
{
    tiled_mainloop<T>(row_a, row_b, K, ring, acc, [] {});
}

// The same tile with the next k-tile (64 indices) staged through registers, one tile ahead and two barriers per k-tile, for rows that
// are not aligned to 16 bytes; the sums run in the same order.  Rows of the LDS tiles are 72 elements apart (fragment reads of
// consecutive rows hit distinct banks).
constexpr int kStagedLd = 72;
template <class RowA, class RowB>
__device__ __forceinline__ void staged_mainloop(RowA row_a, RowB row_b, int K, unsigned char *lds, f32x16_t (&acc)[4][2])
{
    bf16_t *As = reinterpret_cast<bf16_t *>(lds), *Bs = As + kGtRows * kStagedLd;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, hi = lane >> 5;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mt][nt][i] = 0.f;
    const int prow = tid >> 3, pc = tid & 7;   // piece pc of rows prow + 32 i
    const bf16_t *ga[8], *gb[4];
#pragma unroll
    for (int i = 0; i < 8; ++i) ga[i] = row_a(prow + 32 * i) + 8 * pc;
#pragma unroll
    for (int i = 0; i < 4; ++i) gb[i] = row_b(prow + 32 * i) + 8 * pc;
    u32x4_t ra[8], rb[4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) ra[i] = *reinterpret_cast<const u32x4_t *>(ga[i] + k0);
#pragma unroll
        for (int i = 0; i < 4; ++i) rb[i] = *reinterpret_cast<const u32x4_t *>(gb[i] + k0);
    };
    auto stage = [&]() {
#pragma unroll
        for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4_t *>(As + (prow + 32 * i) * kStagedLd + 8 * pc) = ra[i];
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4_t *>(Bs + (prow + 32 * i) * kStagedLd + 8 * pc) = rb[i];
        __syncthreads();
    };
    fetch(0);
    stage();
    for (int k0 = 0; k0 < K; k0 += 64) {
        const bool more = k0 + 64 < K;
        if (more) fetch(k0 + 64);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            uint4 fa[4], fb[2];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
                fa[mt] = *reinterpret_cast<const uint4 *>(As + (wm * 128 + mt * 32 + l32) * kStagedLd + ks * 16 + 8 * hi);
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                fb[nt] = *reinterpret_cast<const uint4 *>(Bs + (wn * 64 + nt * 32 + l32) * kStagedLd + ks * 16 + 8 * hi);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) acc[mt][nt] = mfma32u(fa[mt], fb[nt], acc[mt][nt]);
        }
        __syncthreads();   // everyone is done reading the tiles
        if (more) stage();
    }
}

// Many rows, either form.  The ring is the faster one mostly where the row tiles leave a ragged last round of workgroups (rt_layer_recompute,
// us, registers / ring: 3 x 683 rows, d = 768: 254 / 227; 8 x 1000, d = 1024: 536 / 522; 8 x 2048: 991 / 993).
template <bool ALIGNED> constexpr int kManyLds = ALIGNED ? TileMany::kLds : (kGtRows + kGtCols) * kStagedLd * 2;
template <bool ALIGNED, class RowA, class RowB>
__device__ __forceinline__ void many_mainloop(RowA row_a, RowB row_b, int K, unsigned char *lds, f32x16_t (&acc)[4][2])
{
    if constexpr (ALIGNED) tiled_mainloop<TileMany>(row_a, row_b, K, lds, acc);
    else staged_mainloop(row_a, row_b, K, lds, acc);
}

}  // namespace rt
