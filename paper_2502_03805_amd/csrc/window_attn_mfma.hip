// Observation-window attention on the matrix cores, bf16, d_h = 128 (Algorithm 2, lines 2-3; eq. (2)).
//
// a^h_i = reduce_w softmax_i(scale * q_w . k_i) needs every window row's max and sum over all n keys
// before any weight can be summed over the window, so the keys are swept twice and the tiny logits
// (G*W rows per kv head) are recomputed on the MFMA units instead of being stored:
//   pass 1 (stats)   per key chunk: row max m and l = sum_i 2^(t_i - m) of t = logit * log2(e)
//   reduce           per row: E = log2(sum_i 2^t_i) (+ log2 W for the window mean)
//   pass 2 (colsum)  a^h_i = sum_w 2^(t_wi - E_w)
//
// Work split: one workgroup per (key chunk, kv head).  Pass 1: one WAVE per (query head of the group, block
// of 32 window rows), holding those queries as MFMA fragments in registers (rows past W are zero and masked):
// a window of more than 32 rows is spread over several waves (more waves in flight, fewer registers each; the
// row statistics need no exchange).  Pass 2: one wave per query head with all its row blocks, because a key's
// window sum runs over all of them (splitting it and adding the shares through LDS was measured slower).  Key tiles of 64 rows stream once per workgroup through LDS (direct global->LDS
// loads, double buffered, 16-byte chunks XOR-swizzled against bank conflicts) and are read by every wave.
//
// v_mfma_f32_32x32x16_bf16 operand layout: a lane holds 8 consecutive k of row (A) / column (B)
// lane % 32 at k offset 8 * (lane / 32); accumulator j is row 8*(j/4) + 4*(lane/32) + j%4, column lane%32.
//   pass 1 computes K . Q^T (lane = one query row, registers = 16 keys): row statistics stay lane-local;
//   pass 2 computes Q . K^T (lane = one key, registers = 16 query rows): the window sum is lane-local.
#include "window_attn_mfma.hpp"

namespace ckv {

// ---- pass 1 ---------------------------------------------------------------------------------------
template <int QB>
__global__ __launch_bounds__(64 * AM_MAX_WAVES) void attn_stats_mfma_kernel(AttnArgs A, float *__restrict__ part)
{
    __shared__ __attribute__((aligned(1024))) char lds[2 * AM_TILE_BYTES];
    const int chunk = blockIdx.x, bi = blockIdx.y / (A.H / A.G), g = blockIdx.y % (A.H / A.G);
    const int nw = blockDim.x >> 6;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int vw = blockIdx.z * A.wpw + wave;               // (query head, 32-row block of the window) of this wave
    const bool head_ok = wave < A.wpw && vw < A.G * A.qbs;
    const int head = g * A.G + (head_ok ? vw / A.qbs : 0);
    const int qb0 = head_ok ? vw % A.qbs : 0;
    const bf16_t *kbase = A.k + bi * A.ks0 + g * A.ks1;
    const __amdgpu_buffer_rsrc_t krsrc = make_k_rsrc(kbase, A.ks2, A.n);
    const int key_begin = chunk * A.chunk_keys;
    const int key_end = min(key_begin + A.chunk_keys, A.n);
    const int tiles = (key_end - key_begin + AM_TILE_KEYS - 1) / AM_TILE_KEYS;

    bf16x8 qf[QB][8];
    load_q_frags<QB>(A, bi, head, qb0, l32, half, qf);
    float m[QB], l[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) { m[qb] = AM_NEG; l[qb] = 0.f; }

    load_k_tile(krsrc, A.ks2, key_begin, A.n, lds, wave, nw, lane);
    __syncthreads();
    for (int t = 0; t < tiles; ++t) {
        const char *cur = lds + (t & 1) * AM_TILE_BYTES;
        if (t + 1 < tiles)
            load_k_tile(krsrc, A.ks2, key_begin + (t + 1) * AM_TILE_KEYS, A.n, lds + ((t + 1) & 1) * AM_TILE_BYTES, wave,
                        nw, lane);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const int key0 = key_begin + t * AM_TILE_KEYS + kb * 32; // first key of this 32-key block
            if (key0 >= key_end) break;
            bf16x8 kf[8];
            read_k_frags(cur, kb, l32, half, kf);
            // blocks past the end of the keys, or (causal tail) reaching into the last W keys, need masking
            const bool ragged = key0 + 32 > A.n || (A.causal && key0 + 31 > A.n - A.W);
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                f32x16 acc = zero16();
#pragma unroll
                for (int s = 0; s < 8; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[qb][s], acc, 0, 0, 0);
                // acc[j]: key key0 + 8*(j/4) + 4*half + j%4, query row l32
                // t = acc * c with c > 0, so the block maximum of t is c * max(acc); 2^(t - m) = 2^fma(acc, c, -m)
                if (ragged) {
                    const int last_seen = A.causal ? A.n - A.W + (qb0 + qb) * 32 + l32 : A.n - 1; // last key this row sees
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        const int key = key0 + 8 * (j / 4) + 4 * half + (j % 4);
                        if (key >= A.n || key > last_seen) acc[j] = -INFINITY;
                    }
                }
                float amax = fmaxf(fmaxf(acc[0], acc[1]), acc[2]);
#pragma unroll
                for (int j = 3; j < 15; j += 2) amax = fmaxf(fmaxf(amax, acc[j]), acc[j + 1]);
                amax = fmaxf(amax, acc[15]);
                const float mn = fmaxf(m[qb], amax * A.c);
                float add = 0.f;
#pragma unroll
                for (int j = 0; j < 16; ++j) add += __builtin_amdgcn_exp2f(fmaf(acc[j], A.c, -mn));
                l[qb] = l[qb] * __builtin_amdgcn_exp2f(m[qb] - mn) + add;
                m[qb] = mn;
            }
        }
        __syncthreads();
    }
    // merge the two lanes that hold the same query row, then one (m, l) pair per row and chunk
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float mo = __shfl_xor(m[qb], 32), lo = __shfl_xor(l[qb], 32);
        const float mt = fmaxf(m[qb], mo);
        const float lt = l[qb] * __builtin_amdgcn_exp2f(m[qb] - mt) + lo * __builtin_amdgcn_exp2f(mo - mt);
        const int w = (qb0 + qb) * 32 + l32;
        if (head_ok && half == 0 && w < A.W) {
            const size_t bh = (size_t)bi * A.H + head;
            const size_t at = A.merge ? (bh * A.chunks + chunk) * A.W + w : (bh * A.W + w) * A.chunks + chunk;
            reinterpret_cast<float2 *>(part)[at] = make_float2(mt, lt);
        }
    }
}

// One wave per window row: E = log2(sum_i 2^t_i) (+ log2 W for the mean), stored at stats[row*2].
__global__ __launch_bounds__(64) void attn_stats_reduce_log2_kernel(const float *__restrict__ part,
                                                                    float *__restrict__ stats, int chunks, float post)
{
    const size_t row = blockIdx.x;
    const float *p = part + row * (size_t)chunks * 2;
    float m = AM_NEG;
    for (int c = threadIdx.x; c < chunks; c += 64) m = fmaxf(m, p[2 * c]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    float l = 0.f;
    for (int c = threadIdx.x; c < chunks; c += 64) l += p[2 * c + 1] * exp2f(p[2 * c] - m);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o);
    if (threadIdx.x == 0) {
        stats[row * 2] = m + log2f(l) + post;
        stats[row * 2 + 1] = 0.f;
    }
}

template <int QB>
__global__ __launch_bounds__(64 * AM_COLSUM_WAVES) void attn_colsum_mfma_kernel(AttnArgs A, const float *__restrict__ stats,
                                                                             float *__restrict__ a_raw)
{
    __shared__ __attribute__((aligned(1024))) char lds[attn_colsum_lds<QB>()];
    attn_colsum_body<QB>(A, stats, a_raw, lds, blockIdx.x, blockIdx.y, blockIdx.z * AM_COLSUM_WAVES);
}

bool attn_mfma_supported(const Dims &d)
{
    return d.dh == AM_DH && d.W <= 96 && ((int64_t)(d.n - 1) * d.ks[2] + AM_DH) * 2 < ((int64_t)1 << 31);
}
// Keys per workgroup.  Longer chunks spread the fixed cost of a workgroup (its query fragments, the first tile's
// latency) over more keys; measured, 1024 keys win as long as the launch still has two workgroups per CU
// (Qwen 128K: both sweeps 20 % faster than with 256), 512 at Llama 32K, 256 below.
// Short contexts leave CUs idle instead, and a sweep is as long as one workgroup's chain of tiles: 128 or 64 keys (one tile)
// while that makes no more workgroups than there are CUs.  Attention-only call, 32 heads over 8, us, 256 keys / this: 200
// tokens 18.4 / 13.0, 1024 18.9 / 13.2, 2048 18.9 / 14.0, 3072 19.2 / 15.9, 4096 19.3 / 16.2; 4 over 1, 16384 tokens 20.2 / 16.6.
// With a second workgroup on a CU there is nothing to gain (6000 tokens, 128 keys: 20.0 / 20.4).
static int attn_chunk_keys(const Dims &d)
{
    const int qbs = (d.W + 31) / 32, wpw = (AM_MAX_WAVES / qbs) * qbs;
    const long long per_chunk_row = (long long)d.batch * d.Hkv * ((d.G * qbs + wpw - 1) / wpw);
    const auto wgs = [&](int keys) { return per_chunk_row * ((d.n + keys - 1) / keys); };
    int keys = 1024;
    while (keys > 256 && wgs(keys) < 512) keys >>= 1;
    if (keys == 256)
        while (keys > ATTN_SHORT_CHUNK && wgs(keys / 2) <= ATTN_SHORT_WGS) keys >>= 1;
    return keys;
}
int mfma_attn_chunks(const Dims &d) { const int keys = attn_chunk_keys(d); return (d.n + keys - 1) / keys; }

// Short contexts: the waves of pass 2 merge the chunks' pairs themselves (a few KiB out of L2 under the first key tile's
// latency) instead of a launch of their own between the sweeps.  Attention-only call, 32 heads over 8, us,
// launch between / merged: 12 chunks 20.8 / 18.5, 32 22.2 / 20.0, 47 25.7 / 24.7, 64 27.7 / 27.4 (256 keys each), 41.0 / 40.5 (512),
// 94 36.0 / 37.1, 128 115.5 / 120.6 (1024): up to 64.  The short chunks of few heads make more of them (4 heads over 1: 110 chunks
// 15.7 / 16.1, 256 16.6 / 20.2), merged all the same where that puts pass 2 beside the projection (157 chunks 35.8 / 29.7, 256
// 41.7 / 36.6, and 20000 tokens, 157 of 128 keys, 48.6 / 42.1).
constexpr int AM_MERGE_CHUNKS = 64;
bool attn_mfma_merges(const Dims &d)
{
    return mfma_attn_chunks(d) <= AM_MERGE_CHUNKS || (attn_chunk_keys(d) < 256 && vproj_colsum_room(d));
}

AttnArgs attn_mfma_args(const Dims &d, const void *q, const void *k)
{
    AttnArgs A;
    A.q = (const bf16_t *)q; A.k = (const bf16_t *)k;
    A.H = d.H; A.G = d.G; A.n = d.n; A.W = d.W; A.chunks = mfma_attn_chunks(d); A.causal = d.causal;
    A.merge = attn_mfma_merges(d);
    A.post = d.window_sum ? 0.0f : log2f((float)d.W);
    A.chunk_keys = attn_chunk_keys(d);
    A.qbs = (d.W + 31) / 32;
    A.wpw = (AM_MAX_WAVES / A.qbs) * A.qbs;
    A.c = d.scale * AM_LOG2E;
    A.ks0 = d.ks[0]; A.ks1 = d.ks[1]; A.ks2 = d.ks[2];
    return A;
}

hipError_t launch_attn_stats_mfma(const Dims &d, const void *q, const void *k, float *part, hipStream_t s)
{
    const AttnArgs A = attn_mfma_args(d, q, k);
    const int pairs = d.G * A.qbs, nw = pairs < A.wpw ? pairs : A.wpw;
    dim3 grid(A.chunks, d.batch * d.Hkv, (pairs + A.wpw - 1) / A.wpw), block(64 * nw);
    hipLaunchKernelGGL(attn_stats_mfma_kernel<1>, grid, block, 0, s, A, part);
    return hipGetLastError();
}

hipError_t launch_attn_stats_reduce_log2(const Dims &d, const float *part, int chunks, float *stats, hipStream_t s)
{
    const size_t rows = (size_t)d.batch * d.H * d.W;
    const float post = d.window_sum ? 0.0f : log2f((float)d.W);
    hipLaunchKernelGGL(attn_stats_reduce_log2_kernel, dim3((unsigned)rows), dim3(64), 0, s, part, stats, chunks, post);
    return hipGetLastError();
}

hipError_t launch_attn_colsum_mfma(const Dims &d, const void *q, const void *k, const float *stats, float *a_raw,
                                   hipStream_t s)
{
    const AttnArgs A = attn_mfma_args(d, q, k);
    const int nw = d.G < AM_COLSUM_WAVES ? d.G : AM_COLSUM_WAVES;
    dim3 grid(A.chunks, d.batch * d.Hkv, (d.G + AM_COLSUM_WAVES - 1) / AM_COLSUM_WAVES), block(64 * nw);
    const int qb = (d.W + 31) / 32;
    if (qb == 1) hipLaunchKernelGGL(attn_colsum_mfma_kernel<1>, grid, block, 0, s, A, stats, a_raw);
    else if (qb == 2) hipLaunchKernelGGL(attn_colsum_mfma_kernel<2>, grid, block, 0, s, A, stats, a_raw);
    else hipLaunchKernelGGL(attn_colsum_mfma_kernel<3>, grid, block, 0, s, A, stats, a_raw);
    return hipGetLastError();
}

} // namespace ckv
