// The fp32 key sweeps' bodies, shared by their own launches and those that run them beside the magnitudes' kernels.
#pragma once

#include <float.h>

#include "common.hpp"

namespace ckv {

typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int AF_WAVES = 4;
constexpr int AF_KEYS = 32;       // keys per block
constexpr int AF_ROWS = 32;       // window rows per block
constexpr int AF_MAX_RANGES = 64; // key ranges per head that every wave of pass 2 merges by itself
constexpr int AF_SIMDS = 1024;    // of the chip
constexpr int AF_CHAINS = 2;      // accumulators per block of logits
constexpr double AF_LOG2E = 1.4426950408889634;
constexpr float AF_NEG = -1.0e30f;

struct AttnF32Args {
    const float *q, *k;
    int H, G, n, W;
    int ranges; // wave r of a row block takes key blocks r, r + ranges, ...
    int merged; // pairs lie [head][row][range] and a launch of their own merges them, else [head][range][row]
    int qbs;    // row blocks of a window
    int waves;  // in all
    int causal;
    float post;    // 1 / W for the window mean, 1 for the sum
    float c, c_lo; // scale * log2(e), and what its rounding left out
    int64_t ks0, ks1, ks2;
};

// Which rows and keys a wave works on.  pass 1: one wave per (kv head, range, query head of the group, row block);
// pass 2: one per (kv head, range, query head), which runs over the window's row blocks.
struct F32Job {
    int bi, g, head, qb, range;
};
__device__ __forceinline__ bool f32_job(const AttnF32Args &A, int wg, int per_range, int qbs, F32Job &J)
{
    const int w = wg * AF_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w >= A.waves) return false;
    const int Hkv = A.H / A.G, in_range = w % per_range, r = w / per_range;
    J.range = r % A.ranges;
    const int bh = r / A.ranges;
    J.bi = bh / Hkv;
    J.g = bh % Hkv;
    J.head = J.g * A.G + in_range / qbs;
    J.qb = in_range % qbs;
    return true;
}

// Operand fragments of 32 rows (this lane's row at p): chunk i holds k = 8i + 4 * half .. + 3.  Requested in this order, the
// one in which `logits` uses and refills them: its waits then count the loads behind a chunk, and not all of them.
template <int DH>
__device__ __forceinline__ void load_rows(const float *p, int half, float4 (&f)[DH / 8])
{
#pragma unroll
    for (int i = 0; i < DH / 8; ++i) {
        f[i] = *reinterpret_cast<const float4 *>(p + 8 * i + 4 * half);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// 2^(logit * c - m), 0 for a masked logit.  c's rounding would be a relative error of up to 2^-24 |t| that all of a row's
// weights share in sign; the second fma takes it out.
__device__ __forceinline__ float weight(float logit, float m, const AttnF32Args &A)
{
    const float t = fmaf(logit, A.c_lo, fmaf(logit, A.c, -m));
    return logit == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(t);
}

// One block of logits: a (rows of the result) times b; after its use each chunk of `refill` takes the next block's.
template <int DH, bool KEYS_ARE_ROWS, int CHAINS>
__device__ __forceinline__ f32x16 logits(float4 (&key)[DH / 8], const float4 (&query)[DH / 8], const float *next, int half)
{
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 acc[CHAINS];
#pragma unroll
    for (int i = 0; i < DH / 8; ++i) {
        const float kx[4] = {key[i].x, key[i].y, key[i].z, key[i].w}, qx[4] = {query[i].x, query[i].y, query[i].z, query[i].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            f32x16 &to = acc[e % CHAINS];
            const f32x16 from = i == 0 && e < CHAINS ? zero : to; // (zero is an operand of the instruction)
            to = KEYS_ARE_ROWS ? __builtin_amdgcn_mfma_f32_32x32x2f32(kx[e], qx[e], from, 0, 0, 0)
                               : __builtin_amdgcn_mfma_f32_32x32x2f32(qx[e], kx[e], from, 0, 0, 0);
        }
        key[i] = *reinterpret_cast<const float4 *>(next + 8 * i + 4 * half);
        __builtin_amdgcn_sched_barrier(0); // (left alone, the loads gather at the block's end and nothing covers them)
    }
#pragma unroll
    for (int c = CHAINS / 2; c > 0; c >>= 1)
#pragma unroll
        for (int x = 0; x < c; ++x)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[x][j] += acc[x + c][j];
    return acc[0];
}

template <int DH, int CHAINS>
__device__ __forceinline__ void attn_stats_f32_body(const AttnF32Args &A, float *__restrict__ part, int wg)
{
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    F32Job J;
    if (!f32_job(A, wg, A.G * A.qbs, A.qbs, J)) return; // no barrier in this kernel
    const float *kbase = A.k + J.bi * A.ks0 + J.g * A.ks1;
    const int blocks = (A.n + AF_KEYS - 1) / AF_KEYS;
    auto key_row = [&](int block) { return kbase + (int64_t)min(block * AF_KEYS + l32, A.n - 1) * A.ks2; };
    const int row = J.qb * AF_ROWS + l32; // this lane's window row (rows past W repeat the last and are not stored)
    float4 qf[DH / 8], kf[DH / 8];
    load_rows<DH>(A.q + (((size_t)J.bi * A.H + J.head) * A.W + min(row, A.W - 1)) * DH, half, qf);
    load_rows<DH>(key_row(J.range), half, kf);
    float m = AF_NEG, l = 0.f;
    const int last_seen = A.causal ? A.n - A.W + row : A.n - 1; // last key this lane's row sees
    const int clean_end = A.causal ? A.n - A.W + 1 : A.n;       // keys before this one are seen by every row
    for (int b = J.range; b < blocks; b += A.ranges) {
        f32x16 acc = logits<DH, true, CHAINS>(kf, qf, key_row(min(b + A.ranges, blocks - 1)), half);
        // acc[j]: key b * 32 + 8*(j/4) + 4*half + j%4, window row l32
        if (b * AF_KEYS + AF_KEYS > clean_end) { // uniform
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int key = b * AF_KEYS + 8 * (j / 4) + 4 * half + (j % 4);
                if (key >= A.n || key > last_seen) acc[j] = -INFINITY;
            }
        }
        float amax = fmaxf(fmaxf(acc[0], acc[1]), acc[2]);
#pragma unroll
        for (int j = 3; j < 15; j += 2) amax = fmaxf(fmaxf(amax, acc[j]), acc[j + 1]);
        amax = fmaxf(amax, acc[15]);
        const float mn = fmaxf(m, amax * A.c);
        float add = 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) add += weight(acc[j], mn, A);
        l = l * __builtin_amdgcn_exp2f(m - mn) + add;
        m = mn;
    }
    // the two lanes that hold the same window row
    const float mo = __shfl_xor(m, 32), lo = __shfl_xor(l, 32);
    const float mt = fmaxf(m, mo);
    const float lt = l * __builtin_amdgcn_exp2f(m - mt) + lo * __builtin_amdgcn_exp2f(mo - mt);
    if (half == 0 && row < A.W) {
        const size_t head = (size_t)J.bi * A.H + J.head;
        const size_t at = A.merged ? (head * A.W + row) * A.ranges + J.range : (head * A.ranges + J.range) * A.W + row;
        reinterpret_cast<float2 *>(part)[at] = make_float2(mt, lt);
    }
}

// stat: per wave the 32 rows' (M, weight), ordered [half][16] as a lane's accumulators are
typedef float2 F32RowStat[2][16];
template <int DH, int CHAINS>
__device__ __forceinline__ void attn_colsum_f32_body(const AttnF32Args &A, const float *__restrict__ part,
                                                     float *__restrict__ a_raw, F32RowStat *stat, int wg)
{
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    F32Job J;
    if (!f32_job(A, wg, A.G, 1, J)) return; // no barrier in this kernel
    const float *kbase = A.k + J.bi * A.ks0 + J.g * A.ks1;
    const int blocks = (A.n + AF_KEYS - 1) / AF_KEYS;
    auto key_row = [&](int block) { return kbase + (int64_t)min(block * AF_KEYS + l32, A.n - 1) * A.ks2; };
    float *out = a_raw + ((size_t)J.bi * A.H + J.head) * (size_t)A.n;
    const int pair_ranges = A.merged ? 1 : A.ranges; // (merged: `part` is the merged rows' (M, weight))
    const float2 *pairs = reinterpret_cast<const float2 *>(part) + ((size_t)J.bi * A.H + J.head) * pair_ranges * (size_t)A.W;
    const int clean_end = A.causal ? A.n - A.W + 1 : A.n;
    for (int qb = 0; qb < A.qbs; ++qb) {
        const int row = qb * AF_ROWS + l32, rc = min(row, A.W - 1);
        float4 qf[DH / 8], kf[DH / 8];
        load_rows<DH>(A.q + (((size_t)J.bi * A.H + J.head) * A.W + rc) * DH, half, qf);
        load_rows<DH>(key_row(J.range), half, kf);
        float M, wt;
        if (A.merged) { // uniform over the launch
            const float2 x = pairs[rc];
            M = x.x;
            wt = x.y;
        } else {
            // the row's pairs over the ranges: this lane takes those of its half's parity, then the two halves merge
            float m = AF_NEG, l = 0.f;
            for (int r0 = half; r0 < A.ranges; r0 += 16) {
                float2 x[8]; // requested together; ranges past the last repeat it with weight 0
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = pairs[(size_t)min(r0 + 2 * u, A.ranges - 1) * A.W + rc];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const float mn = fmaxf(m, x[u].x);
                    l = l * __builtin_amdgcn_exp2f(m - mn) + (r0 + 2 * u < A.ranges ? x[u].y : 0.f) * __builtin_amdgcn_exp2f(x[u].x - mn);
                    m = mn;
                }
            }
            const float mo = __shfl_xor(m, 32), lo = __shfl_xor(l, 32);
            M = fmaxf(m, mo);
            wt = A.post / (l * __builtin_amdgcn_exp2f(m - M) + lo * __builtin_amdgcn_exp2f(mo - M));
        }
        // row l32 = 8*(j/4) + 4*hf + j%4 of the block belongs to accumulator j of the lanes of half hf
        if (half == 0) stat[wave][(l32 >> 2) & 1][(l32 >> 3) * 4 + (l32 & 3)] = make_float2(M, row < A.W ? wt : 0.f);
        float me[16], we[16]; // (read by the wave that wrote them: program order and the LDS counter keep them coherent)
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const float2 x = stat[wave][half][j];
            me[j] = x.x;
            we[j] = x.y;
        }
        __builtin_amdgcn_s_waitcnt(0x0F70); // vmcnt(0): from here on the loop's own loads are all that is in flight
        for (int b = J.range; b < blocks; b += A.ranges) {
            f32x16 acc = logits<DH, false, CHAINS>(kf, qf, key_row(min(b + A.ranges, blocks - 1)), half);
            // acc[j]: window row qb*32 + 8*(j/4) + 4*half + j%4, key b * 32 + l32
            const int key = b * AF_KEYS + l32;
            if (b * AF_KEYS + AF_KEYS > clean_end && A.causal) { // uniform: some window rows do not see these keys
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (key > A.n - A.W + qb * AF_ROWS + 8 * (j / 4) + 4 * half + (j % 4)) acc[j] = -INFINITY;
            }
            float s = 0.f;
#pragma unroll
            for (int j = 0; j < 16; ++j) s = fmaf(weight(acc[j], me[j], A), we[j], s);
            s += __shfl_xor(s, 32);
            if (half == 0 && key < A.n) out[key] = qb == 0 ? s : out[key] + s; // (this lane's own earlier store)
        }
    }
}

// The arguments of pass 1 (else pass 2) of a layer; part_floats as launch_attn_f32 has it.
AttnF32Args attn_f32_args(const Dims &d, const void *q, const void *k, size_t part_floats, bool pass1);
inline int attn_f32_wgs(const AttnF32Args &A) { return (A.waves + AF_WAVES - 1) / AF_WAVES; }
hipError_t launch_attn_f32_merge(const Dims &d, const AttnF32Args &A, const float *part, float *stats, hipStream_t s);

} // namespace ckv
