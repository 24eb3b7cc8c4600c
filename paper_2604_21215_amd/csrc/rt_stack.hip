// The two operations a stack of RT layers needs around the layers themselves: the embedding lookup
// that produces the first layer's input, and the final RMS normalisation followed by the untied
// output projection ("LM head").  Neither is part of the layer recurrence (Sec. 6.1 leaves embedding
// and unembedding out of its cost model); both are bandwidth-bound single passes.
#include "rt_mfma_device.h"

namespace rt {

// x[b][n][:] = table[ids[b * ids_stride + first + n]][:]; one wavefront per row, 16-byte pieces.
template <typename T>
__global__ __launch_bounds__(256) void embed_rows_kernel(const T *__restrict__ table, const int32_t *__restrict__ ids,
                                                         T *__restrict__ x, int B, int N, int d, int vocab,
                                                         long long ids_stride, int first)
{
    const int lane = threadIdx.x & 63;
    const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= (long long)B * N) return;
    const int b = (int)(row / N), n = (int)(row % N);
    int id = ids[b * ids_stride + first + n];
    id = min(max(id, 0), vocab - 1);  // ids outside the table are clamped, never dereferenced
    constexpr int per = 16 / (int)sizeof(T);
    const uint4 *src = reinterpret_cast<const uint4 *>(table + (size_t)id * d);
    uint4 *dst = reinterpret_cast<uint4 *>(x + (size_t)row * d);
    for (int c = lane; c < d / per; c += 64) dst[c] = src[c];
}

// logits[b][v] = sum_k W[v][k] * (g[k] z[b][k] / rms(z[b])), fp32 out.  A workgroup first builds the
// normalised rows of one batch tile in LDS, then each of its wavefronts walks over vocabulary rows.
constexpr int kHeadLdsFloats = 12288;

template <typename T>
__global__ __launch_bounds__(256) void lm_head_kernel(const T *__restrict__ W, const T *__restrict__ g,
                                                      const T *__restrict__ z, long long z_stride, float *__restrict__ logits,
                                                      int B, int d, int vocab, float eps, int norm_free, int bt)
{
    __shared__ float zs[kHeadLdsFloats];
    __shared__ float red[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int b0 = 0; b0 < B; b0 += bt) {
        const int nb = min(bt, B - b0);
        __syncthreads();
        for (int b = 0; b < nb; ++b) {
            const T *zr = z + (size_t)(b0 + b) * z_stride;
            float ss = 0.f;
            for (int k = threadIdx.x; k < d; k += 256) {
                const float v = to_f32(zr[k]);
                zs[b * d + k] = v;
                ss = fmaf(v, v, ss);
            }
            ss = wave_sum(ss);
            if (lane == 0) red[wave] = ss;
            __syncthreads();
            const float tot = red[0] + red[1] + red[2] + red[3];
            const float rinv = norm_free ? 1.f : rsqrtf(tot / (float)d + eps);
            for (int k = threadIdx.x; k < d; k += 256) {
                const float gg = (g && !norm_free) ? to_f32(g[k]) : 1.f;
                zs[b * d + k] *= rinv * gg;
            }
            __syncthreads();
        }
        for (int v = blockIdx.x * 4 + wave; v < vocab; v += gridDim.x * 4) {
            const T *wr = W + (size_t)v * d;
            float acc[8];
#pragma unroll
            for (int b = 0; b < 8; ++b) acc[b] = 0.f;
            for (int k = lane * 8; k < d; k += 512) {
                float w[8];
                load8(wr + k, w);
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    if (b < nb) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) acc[b] = fmaf(w[e], zs[b * d + k + e], acc[b]);
                    }
                }
            }
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                if (b < nb) {
                    const float s = wave_sum(acc[b]);
                    if (lane == 0) logits[(size_t)(b0 + b) * vocab + v] = s;
                }
            }
        }
    }
}

// The same on the matrix cores (bf16 storage): D[16 vocabulary rows][16 batch columns] += W[16][32] z^T[32][16].  The
// normalised rows are not rounded: each element is staged as three bf16 parts whose sum holds all 24 bits of the fp32 value,
// and every weight fragment feeds three instructions (the chip has ten times the matrix rate that this needs at the memory
// rate).  The heads' sums of 32 products are added up in four partial sums on the vector ALUs: one accumulator that runs through
// all 3 d / 32 instructions rounds at every one of them (distance from fp64 at d = 1024 / 4096: 3.4e-7 / 6.9e-7 of the norm; this
// form 0.9e-7 / 1.3e-7, the plain-ALU form 1.2e-7 / 1.7e-7; the times are the same, while with eight partial sums a second workgroup
// of a compute unit no longer has registers: 256 batch rows, d = 512: 104 -> 161 us).
// Bound: the matrix, read once per 16 batch rows.  The plain-ALU form above reads 32 KB of LDS and issues 8192 adds
// per weight row at 8 batch rows: 153 us for 67 MB (d = 1024, 32768 rows, 8 batch rows) = 0.44 TB/s; here 22 us = 3.0 TB/s.
// A wavefront takes 16 vocabulary rows at a time; the contraction index of a step pair is assigned so that a lane's two
// loads are 32 contiguous bytes (four lanes cover a row's 128), kHeadAhead pairs are in flight, the first of them requested
// before the rows are normalised.
// grid (<= row tiles / 8, batch tiles of bt), block 512, LDS 3 bt (d + 8) bf16.  d a multiple of 256.
constexpr int kHeadAhead = 4;
__global__ __launch_bounds__(512) void lm_head_mfma_kernel(const bf16_t *__restrict__ W, const bf16_t *__restrict__ g,
                                                           const bf16_t *__restrict__ z, long long z_stride,
                                                           float *__restrict__ logits, int B, int d, int vocab, float eps,
                                                           int norm_free, int bt, int wide_stores)
{
    extern __shared__ __align__(16) unsigned char head_smem[];
    bf16_t *zs = reinterpret_cast<bf16_t *>(head_smem);   // [3][bt][d + 8]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 15, gk = lane >> 4;
    const int b0 = blockIdx.y * bt, nb = min(bt, B - b0), ld = d + 8;
    const int tiles = (vocab + 15) / 16, tstep = gridDim.x * 8;
    int tile = blockIdx.x * 8 + wave;
    uint4 w[2 * kHeadAhead];
    const bf16_t *wr = W + (size_t)min(tile * 16 + col, vocab - 1) * d + 16 * gk;
#pragma unroll
    for (int j = 0; j < kHeadAhead; ++j) {
        w[2 * j] = *reinterpret_cast<const uint4 *>(wr + 64 * j);
        w[2 * j + 1] = *reinterpret_cast<const uint4 *>(wr + 64 * j + 8);
    }
    for (int b = wave; b < nb; b += 8) {
        const bf16_t *zr = z + (long long)(b0 + b) * z_stride;
        float ss = 0.f;
#pragma unroll 4
        for (int k = lane; k < d; k += 64) { const float v = bf16_to_f32(zr[k]); ss = fmaf(v, v, ss); }
        ss = wave_sum(ss);
        const float rinv = norm_free ? 1.f : rsqrtf(ss / (float)d + eps);
#pragma unroll 4
        for (int k = lane; k < d; k += 64) {
            const float v = bf16_to_f32(zr[k]) * (rinv * ((g && !norm_free) ? bf16_to_f32(g[k]) : 1.f));
            // by truncation, as a value beyond the largest bf16 has a finite head then; every difference is exact
            const uint32_t p0 = __float_as_uint(v) & 0xFFFF0000u;
            const float r1 = (p0 & 0x7F800000u) == 0x7F800000u ? 0.f : v - __uint_as_float(p0);   // an infinity has no remainder
            const uint32_t p1 = __float_as_uint(r1) & 0xFFFF0000u;
            const uint32_t p2 = __float_as_uint(r1 - __uint_as_float(p1));
            zs[(size_t)b * ld + k] = (bf16_t)(p0 >> 16);
            zs[(size_t)(bt + b) * ld + k] = (bf16_t)(p1 >> 16);
            zs[(size_t)(2 * bt + b) * ld + k] = (bf16_t)(p2 >> 16);
        }
    }
    __syncthreads();
    const int cb = min(col, nb - 1);   // columns beyond the batch repeat its last row (their results are dropped)
    const bf16_t *zh = zs + (size_t)cb * ld + 16 * gk, *zm = zh + (size_t)bt * ld, *zl = zm + (size_t)bt * ld;
    for (; tile < tiles; tile += tstep) {   // no barrier below
        const bf16_t *wn = W + (size_t)min((tile + tstep) * 16 + col, vocab - 1) * d + 16 * gk;   // the next tile's rows
        constexpr f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
        f32x4_t low = zero, head[kHeadAhead];   // middle and tail parts: 2^-8 of the sum, in one chain
#pragma unroll
        for (int j = 0; j < kHeadAhead; ++j) head[j] = zero;
        for (int k0 = 0; k0 < d; k0 += 64 * kHeadAhead) {
            const bool last = k0 + 64 * kHeadAhead >= d;
            const bf16_t *src = last ? wn : wr + k0 + 64 * kHeadAhead;
#pragma unroll
            for (int j = 0; j < kHeadAhead; ++j) {
                Frag a0, a1, x;
                a0.u = w[2 * j];
                a1.u = w[2 * j + 1];
                if (!last || tile + tstep < tiles) {
                    w[2 * j] = *reinterpret_cast<const uint4 *>(src + 64 * j);
                    w[2 * j + 1] = *reinterpret_cast<const uint4 *>(src + 64 * j + 8);
                }
                const int k = k0 + 64 * j;
                x.u = *reinterpret_cast<const uint4 *>(zl + k); low = mfma16(a0, x, low);
                x.u = *reinterpret_cast<const uint4 *>(zl + k + 8); low = mfma16(a1, x, low);
                x.u = *reinterpret_cast<const uint4 *>(zm + k); low = mfma16(a0, x, low);
                x.u = *reinterpret_cast<const uint4 *>(zm + k + 8); low = mfma16(a1, x, low);
                x.u = *reinterpret_cast<const uint4 *>(zh + k); head[j] += mfma16(a0, x, zero);
                x.u = *reinterpret_cast<const uint4 *>(zh + k + 8); head[j] += mfma16(a1, x, zero);
            }
        }
        static_assert(kHeadAhead == 4, "four partial sums");
        const f32x4_t top = (head[0] + head[1]) + (head[2] + head[3]);
        f32x4_t acc = top + low;
        // an infinite weight times the other parts, zero or of the other sign, is no part of the sum: the head's product stands
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = acc[r] == acc[r] ? acc[r] : top[r];
        wr = wn;
        if (col < nb) {   // lane: four consecutive vocabulary rows of batch row b0 + col
            const int v0 = tile * 16 + 4 * gk;
            float *out = logits + (size_t)(b0 + col) * vocab + v0;
            if (wide_stores) {
                if (v0 < vocab) *reinterpret_cast<float4 *>(out) = make_float4(acc[0], acc[1], acc[2], acc[3]);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (v0 + r < vocab) out[r] = acc[r];
            }
        }
    }
}
constexpr size_t kHeadMfmaMaxLds = 152 * 1024;

// Up to how many batch rows the plain-ALU form is the faster one: few vocabulary rows leave the other with a handful of wavefronts,
// each with the whole contraction as one chain of loads, where this one has a wavefront per vocabulary row; its time grows with the
// batch rows, the other's does not.  us, plain / matrix cores, at d = 1024: 2000 rows, B = 1: 4.6 / 12.7, 5: 12.5 / 13.2, 6: 15.1 / 13.1;
// 4000 rows, B = 2: 11.9 / 12.9, 3: 16.0 / 13.1; 8000, B = 1: 10.0 / 12.8, 2: 17.8 / 12.9; 16000, B = 1: 13.6 / 15.6; 20000, B = 1:
// 17.3 / 16.5.  d = 256, 1000 rows, B = 2: 4.6 / 5.2, 3: 5.2 / 5.0; d = 512, B = 4: 7.2 / 7.9, 5: 8.3 / 8.0; d = 4096, B = 6: 36.7 / 44.4,
// 8: 49 / 45 (8000 rows, B = 2: 48.8 / 57.3, 3: 68.8 / 58.2).
static int head_plain_rows(int d, int vocab)
{
    const int wide = d >= 2048 && d <= 8192 ? 1 : 0;
    if (vocab <= 2048) return d < 512 ? 2 : (d < 1024 ? 4 : 5 + wide);
    if (vocab <= 4096) return d < 512 ? 1 : 2 + wide;
    if (vocab <= 8192) return d < 512 ? 0 : 1 + wide;
    return vocab <= 16384 && d >= 1024 ? 1 : 0;
}

template <typename T>
hipError_t embed_rows_launch(const void *table, const int32_t *ids, void *x, int B, int N, int d, int vocab,
                             long long ids_stride, int first, hipStream_t st)
{
    const long long rows = (long long)B * N;
    hipLaunchKernelGGL(embed_rows_kernel<T>, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, (const T *)table, ids, (T *)x,
                       B, N, d, vocab, ids_stride, first);
    return hipGetLastError();
}

template <typename T>
hipError_t lm_head_launch(const void *W, const void *g, const void *z, long long z_stride, float *logits, int B, int d,
                          int vocab, float eps, int norm_free, hipStream_t st)
{
    // bf16 rows of whole 256-index blocks: the matrix-core kernel (32768 rows, d = 1024, B = 8: 22 us against 153 of the
    // plain-ALU form, which keeps the other types and widths, and few rows of both kinds)
    if (sizeof(T) == 2 && d % (64 * kHeadAhead) == 0 && B > head_plain_rows(d, vocab) && (size_t)3 * (d + 8) * 2 <= kHeadMfmaMaxLds) {
        int bt = (int)(kHeadMfmaMaxLds / ((size_t)3 * (d + 8) * 2));
        bt = bt > 16 ? 16 : bt;
        bt = bt > B ? B : bt;
        const size_t lds = (size_t)3 * bt * (d + 8) * 2;
        hipError_t e = hipFuncSetAttribute((const void *)lm_head_mfma_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kHeadMfmaMaxLds);
        if (e != hipSuccess) return e;
        const int tiles = (vocab + 15) / 16, want = (tiles + 7) / 8;
        const int fit = (int)((size_t)160 * 1024 / lds), resident = 256 * (fit > 3 ? 3 : fit);   // workgroups on the chip at once
        const int wide = vocab % 4 == 0 && ((uintptr_t)logits & 15) == 0;
        hipLaunchKernelGGL(lm_head_mfma_kernel, dim3(want < resident ? want : resident, (B + bt - 1) / bt), dim3(512), lds, st,
                           (const bf16_t *)W, (const bf16_t *)g, (const bf16_t *)z, z_stride, logits, B, d, vocab, eps, norm_free, bt,
                           wide);
        return hipGetLastError();
    }
    int bt = kHeadLdsFloats / d;
    if (bt > 8) bt = 8;
    int blocks = (vocab + 3) / 4;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(lm_head_kernel<T>, dim3(blocks), dim3(256), 0, st, (const T *)W, (const T *)g, (const T *)z, z_stride,
                       logits, B, d, vocab, eps, norm_free, bt);
    return hipGetLastError();
}

template hipError_t embed_rows_launch<float>(const void *, const int32_t *, void *, int, int, int, int, long long, int,
                                             hipStream_t);
template hipError_t embed_rows_launch<bf16_t>(const void *, const int32_t *, void *, int, int, int, int, long long, int,
                                              hipStream_t);
template hipError_t lm_head_launch<float>(const void *, const void *, const void *, long long, float *, int, int, int, float,
                                          int, hipStream_t);
template hipError_t lm_head_launch<bf16_t>(const void *, const void *, const void *, long long, float *, int, int, int, float,
                                           int, hipStream_t);

}  // namespace rt
