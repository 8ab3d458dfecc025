// What the shared-tile attention kernels and the launch that runs the second sweep beside the projection have in common:
// arguments, key tiles, and the second sweep itself.
#pragma once

#include <float.h>

#include "common.hpp"

namespace ckv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int AM_DH = 128;
constexpr int AM_TILE_KEYS = 64;
constexpr int AM_TILE_BYTES = AM_TILE_KEYS * AM_DH * 2; // 16 KiB
constexpr int AM_MAX_WAVES = 16;                       // pass 1: waves per workgroup, one per (head, 32-row block)
constexpr int AM_COLSUM_WAVES = 8;                     // pass 2: waves per workgroup, one per head
constexpr float AM_LOG2E = 1.4426950408889634f;
constexpr float AM_NEG = -1.0e30f;

#define LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))
#define GLOBAL_PTR(p) ((const __attribute__((address_space(1))) void *)(p))

struct AttnArgs {
    const bf16_t *q;
    const bf16_t *k;
    int H, G, n, W, chunks;
    int chunk_keys; // keys per workgroup, a multiple of the tile
    int qbs;        // 32-row blocks of the window: a wave owns one (query head, row block)
    int wpw;        // (head, row block) pairs per workgroup: a multiple of qbs, so a head's blocks share a workgroup
    int causal; // window row w sees keys <= n - W + w only
    int merge;  // the chunks' pairs lie [head][chunk][row] and pass 2 merges them, else [head][row][chunk] for a launch between
    float post; // log2 W for the window mean, 0 for the sum
    float c; // scale * log2(e)
    int64_t ks0, ks1, ks2;
};

// Q fragments of one head: block qb covers window rows (qb0+qb)*32 .. +31 (zero past W).
template <int QB>
__device__ __forceinline__ void load_q_frags(const AttnArgs &A, int bi, int head, int qb0, int l32, int half,
                                             bf16x8 (&qf)[QB][8])
{
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int w = (qb0 + qb) * 32 + l32;
        const bf16_t *p = A.q + (((size_t)bi * A.H + head) * A.W + min(w, A.W - 1)) * AM_DH + half * 8;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            bf16x8 x = *reinterpret_cast<const bf16x8 *>(p + s * 16);
            if (w >= A.W) x = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
            qf[qb][s] = x;
        }
    }
}

// Direct global->LDS load of one 64-key tile, shared among the nw waves of the workgroup.
// Instruction j fills LDS KiB j = keys 4j .. 4j+3; lane i writes slot i % 16 of key 4j + i / 16 and
// fetches 16-byte chunk (i % 16) ^ (key & 15) of that key row.  Rows past n-1 re-read row n-1.
// The loads are buffer loads (not flat/global ones) so that the compiler keeps exact LDS wait counts.
__device__ __forceinline__ void load_k_tile(__amdgpu_buffer_rsrc_t krsrc, int64_t ks2, int key0, int n, char *buf,
                                            int wave, int nw, int lane)
{
    for (int j = wave; j < AM_TILE_BYTES / 1024; j += nw) {
        const int key_in_tile = 4 * j + (lane >> 4);
        const int key = min(key0 + key_in_tile, n - 1);
        const uint32_t voff = (uint32_t)(((int64_t)key * ks2 + (((lane & 15) ^ (key_in_tile & 15)) * 8)) * 2);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(krsrc, LDS_PTR(buf + j * 1024), 16, voff, 0, 0, 0);
    }
}

// Buffer descriptor over one kv head's keys (token stride ks2 elements; the host checks n * ks2 * 2 < 2 GiB).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_k_rsrc(const bf16_t *kbase, int64_t ks2, int n)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)kbase, 0, (int)(((int64_t)(n - 1) * ks2 + AM_DH) * 2), 0x00020000);
}

__device__ __forceinline__ void read_k_frags(const char *tile, int kb, int l32, int half, bf16x8 (&kf)[8])
{
    const char *row = tile + (kb * 32 + l32) * (AM_DH * 2);
#pragma unroll
    for (int s = 0; s < 8; ++s) kf[s] = *reinterpret_cast<const bf16x8 *>(row + (((2 * s + half) ^ (l32 & 15)) * 16));
}

__device__ __forceinline__ f32x16 zero16()
{
    return f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
}

// ---- pass 2 ---------------------------------------------------------------------------------------
// LDS of a workgroup: two key tiles and, per wave, the rows' E (when the wave merges them)
template <int QB> constexpr int attn_colsum_lds() { return 2 * AM_TILE_BYTES + AM_COLSUM_WAVES * QB * 32 * (int)sizeof(float); }

// One workgroup's share: chunk `chunk` of (batch item, kv head) pair `bg`, query heads h0 .. h0 + (waves) - 1 of the group.
// stats: the rows' E, or (A.merge) the chunks' pairs, which every wave then merges for its own head's rows.
template <int QB>
__device__ __forceinline__ void attn_colsum_body(const AttnArgs &A, const float *__restrict__ stats, float *__restrict__ a_raw,
                                                 char *lds, int chunk, int bg, int h0)
{
    const int bi = bg / (A.H / A.G), g = bg % (A.H / A.G);
    const int nw = blockDim.x >> 6;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int head = g * A.G + h0 + wave;
    const bool head_ok = h0 + wave < A.G;
    const bf16_t *kbase = A.k + bi * A.ks0 + g * A.ks1;
    const __amdgpu_buffer_rsrc_t krsrc = make_k_rsrc(kbase, A.ks2, A.n);
    const int key_begin = chunk * A.chunk_keys;
    const int key_end = min(key_begin + A.chunk_keys, A.n);
    const int tiles = (key_end - key_begin + AM_TILE_KEYS - 1) / AM_TILE_KEYS;

    load_k_tile(krsrc, A.ks2, key_begin, A.n, lds, wave, nw, lane);
    bf16x8 qf[QB][8];
    load_q_frags<QB>(A, bi, head_ok ? head : g * A.G, 0, l32, half, qf);
    // E of the 16 window rows a lane's accumulators belong to (+inf past W: weight 0)
    float e[QB][16];
    const size_t bh = (size_t)bi * A.H + (head_ok ? head : g * A.G);
    if (A.merge) { // uniform over the launch
        // lane (row l32, half) takes the chunks of its half's parity, then the two halves merge
        float *mine = reinterpret_cast<float *>(lds + 2 * AM_TILE_BYTES) + wave * QB * 32;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int w = qb * 32 + l32;
            const float2 *pairs = reinterpret_cast<const float2 *>(stats) + bh * A.chunks * A.W + min(w, A.W - 1);
            float m = AM_NEG, l = 0.f;
            for (int c0 = half; c0 < A.chunks; c0 += 16) {
                float2 x[8]; // requested together; chunks past the last repeat it with weight 0
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = pairs[(size_t)min(c0 + 2 * u, A.chunks - 1) * A.W];
                float mn = m;
#pragma unroll
                for (int u = 0; u < 8; ++u) mn = fmaxf(mn, x[u].x);
                l *= __builtin_amdgcn_exp2f(m - mn);
#pragma unroll
                for (int u = 0; u < 8; ++u) l += (c0 + 2 * u < A.chunks ? x[u].y : 0.f) * __builtin_amdgcn_exp2f(x[u].x - mn);
                m = mn;
            }
            const float mo = __shfl_xor(m, 32), lo = __shfl_xor(l, 32), mt = fmaxf(m, mo);
            l = l * __builtin_amdgcn_exp2f(m - mt) + lo * __builtin_amdgcn_exp2f(mo - mt);
            if (half == 0) mine[w] = head_ok && w < A.W ? mt + log2f(l) + A.post : INFINITY;
        }
        // (read by the wave that wrote them: program order and the LDS counter keep them coherent)
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int j = 0; j < 16; ++j) e[qb][j] = mine[qb * 32 + 8 * (j / 4) + 4 * half + (j % 4)];
    } else {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int w = qb * 32 + 8 * (j / 4) + 4 * half + (j % 4);
                e[qb][j] = (head_ok && w < A.W) ? stats[(bh * A.W + w) * 2] : INFINITY;
            }
    }
    float *out = a_raw + bh * (size_t)A.n;
    __syncthreads();
    for (int t = 0; t < tiles; ++t) {
        const char *cur = lds + (t & 1) * AM_TILE_BYTES;
        if (t + 1 < tiles)
            load_k_tile(krsrc, A.ks2, key_begin + (t + 1) * AM_TILE_KEYS, A.n, lds + ((t + 1) & 1) * AM_TILE_BYTES, wave,
                        nw, lane);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const int key0 = key_begin + t * AM_TILE_KEYS + kb * 32;
            if (key0 >= key_end) break;
            bf16x8 kf[8];
            read_k_frags(cur, kb, l32, half, kf);
            float colsum = 0.f;
            const bool tail = A.causal && key0 + 31 > A.n - A.W; // some window rows do not see these keys
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                f32x16 acc = zero16();
#pragma unroll
                for (int s = 0; s < 8; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[qb][s], kf[s], acc, 0, 0, 0);
                // acc[j]: window row qb*32 + 8*(j/4) + 4*half + j%4, key key0 + l32
                if (tail) {
#pragma unroll
                    for (int j = 0; j < 16; ++j)
                        if (key0 + l32 > A.n - A.W + qb * 32 + 8 * (j / 4) + 4 * half + (j % 4)) acc[j] = -INFINITY;
                }
#pragma unroll
                for (int j = 0; j < 16; ++j) colsum += __builtin_amdgcn_exp2f(fmaf(acc[j], A.c, -e[qb][j]));
            }
            colsum += __shfl_xor(colsum, 32);
            const int key = key0 + l32;
            if (head_ok && half == 0 && key < A.n) out[key] = colsum;
        }
        __syncthreads();
    }
}

// the arguments both sweeps of a layer are launched with
AttnArgs attn_mfma_args(const Dims &d, const void *q, const void *k);

} // namespace ckv
