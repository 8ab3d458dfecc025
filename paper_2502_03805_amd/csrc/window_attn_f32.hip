// Observation-window attention for fp32 layers on the fp32 matrix instruction, d_h = 64 or 128, any window
// (Algorithm 2, lines 2-3; eq. (2)).  The two sweeps of the bf16 kernels:
//   pass 1   per (32 window rows of a query head, key range): row max m and l = sum_i 2^(t_i - m), t = logit * log2(e)
//   pass 2   a^h_i = sum_w 2^(t_wi - M_w) * weight_w, with (M_w, weight_w = 1 / sum [/ W]) of the row merged from the
//            ranges' pairs by every wave that needs them, or by a launch between where a head has more than 64 ranges
//
// v_mfma_f32_32x32x2_f32: a lane holds row (A) / column (B) lane % 32 at k = lane / 32; accumulator j is row
// 8*(j/4) + 4*(lane/32) + j%4, column lane%32.  It adds its two products one after the other in fp32, as a scalar fmaf
// chain does.  A logit is the sum of two chains of half of d_h each: its rounding, which all of a heavy entry's weights
// share, is most of the result's error.  Against 64 bits (2-norm, means over 100 layers of the tiny shape and 30 of the
// larger one below): the vector kernel 3.6e-7 / 2.4e-7, one chain 3.6e-7 / 2.3e-7, two 2.0e-7 / 1.5e-7, four 1.6e-7 /
// 1.1e-7; two cost 1 %, four 2 - 4 (the sums' additions, which nothing covers where a SIMD has one wave).
// Which k an instruction takes is free as long as both operands agree: instruction 4i + e takes k = 8i + 4 * (lane / 32)
// + e, so that a lane's operands of four instructions are one 16-byte load from global memory; no LDS.
//
// Work split: a wave owns one block of 32 window rows of one query head (its queries in registers for its whole life)
// and every ranges-th block of 32 keys; a key fragment's register is refilled with the wave's next block as soon as its
// four instructions are issued (held there: gathered at the block's end, as the compiler would have them, the loads are
// covered by nothing, and both sweeps take 860 instead of 607 us at 32 heads over 8 kv heads, d_h 128, 131072 tokens).
// Neighbouring waves take the same keys for the group's other row blocks (the second reader finds them in L1).  Bound by
// the fp32 matrix rate, 64 flop per cycle and SIMD.
// 16 heads over 4 kv heads, d_h 128, 8192 tokens, W 32: 122 us on the vector ALUs, 36 like this; 4 heads, d_h 64, 1024
// tokens, W 8: 24 and 13 us (2 x 1.07 GFLOP are 2 x 7 us at the larger one).
#include <float.h>
#include <type_traits>

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
    float c, c_lo; // scale * log2(e), and what its rounding left out
    int64_t ks0, ks1, ks2;
};

// Which rows and keys a wave works on.  pass 1: one wave per (kv head, range, query head of the group, row block);
// pass 2: one per (kv head, range, query head), which runs over the window's row blocks.
struct F32Job {
    int bi, g, head, qb, range;
};
__device__ __forceinline__ bool f32_job(const AttnF32Args &A, int per_range, int qbs, F32Job &J)
{
    const int w = blockIdx.x * AF_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
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
template <int DH, bool KEYS_ARE_ROWS>
__device__ __forceinline__ f32x16 logits(float4 (&key)[DH / 8], const float4 (&query)[DH / 8], const float *next, int half)
{
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 acc[AF_CHAINS];
#pragma unroll
    for (int i = 0; i < DH / 8; ++i) {
        const float kx[4] = {key[i].x, key[i].y, key[i].z, key[i].w}, qx[4] = {query[i].x, query[i].y, query[i].z, query[i].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            f32x16 &to = acc[e % AF_CHAINS];
            const f32x16 from = i == 0 && e < AF_CHAINS ? zero : to; // (zero is an operand of the instruction)
            to = KEYS_ARE_ROWS ? __builtin_amdgcn_mfma_f32_32x32x2f32(kx[e], qx[e], from, 0, 0, 0)
                               : __builtin_amdgcn_mfma_f32_32x32x2f32(qx[e], kx[e], from, 0, 0, 0);
        }
        key[i] = *reinterpret_cast<const float4 *>(next + 8 * i + 4 * half);
        __builtin_amdgcn_sched_barrier(0); // (left alone, the loads gather at the block's end and nothing covers them)
    }
#pragma unroll
    for (int c = AF_CHAINS / 2; c > 0; c >>= 1)
#pragma unroll
        for (int x = 0; x < c; ++x)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[x][j] += acc[x + c][j];
    return acc[0];
}

template <int DH>
__global__ __launch_bounds__(64 * AF_WAVES, 2) void attn_stats_f32_kernel(AttnF32Args A, float *__restrict__ part)
{
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    F32Job J;
    if (!f32_job(A, A.G * A.qbs, A.qbs, J)) return; // no barrier in this kernel
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
        f32x16 acc = logits<DH, true>(kf, qf, key_row(min(b + A.ranges, blocks - 1)), half);
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

// One wave per window row: the ranges' pairs -> (M, weight).
__global__ __launch_bounds__(64) void attn_merge_f32_kernel(const float *__restrict__ part, float *__restrict__ stats,
                                                            int ranges, float post)
{
    const float2 *p = reinterpret_cast<const float2 *>(part) + (size_t)blockIdx.x * ranges;
    float m = AF_NEG, l = 0.f;
    for (int r0 = 0; r0 < ranges; r0 += 512) {
        float2 x[8]; // requested together; ranges past the last repeat it with weight 0
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = p[min(r0 + 64 * u + (int)threadIdx.x, ranges - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float mn = fmaxf(m, x[u].x);
            l = l * __builtin_amdgcn_exp2f(m - mn) +
                (r0 + 64 * u + (int)threadIdx.x < ranges ? x[u].y : 0.f) * __builtin_amdgcn_exp2f(x[u].x - mn);
            m = mn;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const float mo = __shfl_xor(m, o), lo = __shfl_xor(l, o), mt = fmaxf(m, mo);
        l = l * __builtin_amdgcn_exp2f(m - mt) + lo * __builtin_amdgcn_exp2f(mo - mt);
        m = mt;
    }
    if (threadIdx.x == 0) reinterpret_cast<float2 *>(stats)[blockIdx.x] = make_float2(m, post / l);
}

template <int DH>
__global__ __launch_bounds__(64 * AF_WAVES, 2) void attn_colsum_f32_kernel(AttnF32Args A, const float *__restrict__ part,
                                                                           float *__restrict__ a_raw, float post)
{
    // per wave: the 32 rows' (M, weight), ordered [half][16] as a lane's accumulators are
    __shared__ __attribute__((aligned(16))) float2 stat[AF_WAVES][2][16];
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    F32Job J;
    if (!f32_job(A, A.G, 1, J)) return; // no barrier in this kernel
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
            wt = post / (l * __builtin_amdgcn_exp2f(m - M) + lo * __builtin_amdgcn_exp2f(mo - M));
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
            f32x16 acc = logits<DH, false>(kf, qf, key_row(min(b + A.ranges, blocks - 1)), half);
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

static int f32_blocks(const Dims &d) { return (d.n + AF_KEYS - 1) / AF_KEYS; }

// Key ranges per head.  64, as every wave of pass 2 merges all of its rows' ranges; a launch of few heads does not fill the
// chip with them (1024 SIMDs) and takes as many as give a wave per SIMD, two where each then still has eight blocks, with
// the merge in a launch of its own.  Both sweeps and the combine, W 32, us, 64 ranges / like this / vector kernel: 1 head,
// d_h 64: 16384 tokens 33 / 18 / 62, 131072 178 / 27 / 74; 4 heads, d_h 128, 131072: 338 / 102 / 385; 16 heads, d_h 64,
// 131072: 190 / 174 / 610.
static int f32_ranges(const Dims &d, size_t part_floats)
{
    const size_t fits = part_floats / ((size_t)d.batch * d.H * d.W * 2);
    const int blocks = f32_blocks(d);
    for (int per_simd = 2; per_simd > 0; --per_simd) {
        int most = per_simd * AF_SIMDS / (d.batch * d.H);
        if ((size_t)most > fits) most = (int)fits;
        if (most <= AF_MAX_RANGES || blocks <= AF_MAX_RANGES) continue;
        const int each = (blocks + most - 1) / most, r = (blocks + each - 1) / each;
        if (r > AF_MAX_RANGES && (per_simd == 1 || each >= 8)) return r;
    }
    int r = blocks < AF_MAX_RANGES ? blocks : AF_MAX_RANGES;
    if ((size_t)r > fits) r = (int)fits;
    return r;
}

// A block of window rows costs the matrix instruction the same whether one row of it or all 32 are used; the vector
// kernel's time goes with W * d_h.  At W * d_h of 256 and less it is the faster one once the launch is long enough to be
// bound by that and not by its latencies.  us, vector / this one: W 1: 32 heads, 4096 tokens, d_h 64 19.1 / 24.7, d_h 128
// 27.9 / 36.6; 1 head, 40000, d_h 64 15.5 / 17.1, 4096 14.2 / 13.6.  32 heads, 16384 tokens: W 2 46 / 54 and 80 / 88, W 4
// 49 / 54 and 92 / 89 (d_h 64 and 128); W 2, 8 heads, 9000 tokens, d_h 128: 30.5 / 28.5.
static bool vector_is_faster(const Dims &d)
{
    return d.W * d.dh <= 256 && (long long)d.batch * d.H * d.n >= (d.W == 1 ? 32768 + 1 : 131072);
}

bool attn_f32_taken(const Dims &d, size_t part_floats)
{
    return (d.dh == 64 || d.dh == 128) && !vector_is_faster(d) && f32_ranges(d, part_floats) >= 1 &&
           (long long)d.batch * d.H * ((d.W + AF_ROWS - 1) / AF_ROWS) * (2 * AF_SIMDS) < (1ll << 31);
}

template <int DH>
static void launch_attn_f32_dh(const AttnF32Args &base, const Dims &d, float *part, float *stats, float *a_raw, bool pass1,
                               hipStream_t s)
{
    AttnF32Args A = base;
    const dim3 block(64 * AF_WAVES);
    const float post = d.window_sum ? 1.0f : 1.0f / (float)d.W;
    if (pass1) {
        A.waves = d.batch * d.H * A.qbs * A.ranges;
        hipLaunchKernelGGL(attn_stats_f32_kernel<DH>, dim3((A.waves + AF_WAVES - 1) / AF_WAVES), block, 0, s, A, part);
        if (A.merged)
            hipLaunchKernelGGL(attn_merge_f32_kernel, dim3(d.batch * d.H * d.W), dim3(64), 0, s, part, stats, A.ranges, post);
    } else {
        A.waves = d.batch * d.H * A.ranges;
        hipLaunchKernelGGL(attn_colsum_f32_kernel<DH>, dim3((A.waves + AF_WAVES - 1) / AF_WAVES), block, 0, s, A,
                           A.merged ? stats : part, a_raw, post);
    }
}

hipError_t launch_attn_f32(const Dims &d, const void *q, const void *k, float *part, size_t part_floats, float *stats,
                           float *a_raw, bool pass1, hipStream_t s)
{
    AttnF32Args A;
    A.q = (const float *)q; A.k = (const float *)k;
    A.H = d.H; A.G = d.G; A.n = d.n; A.W = d.W; A.causal = d.causal;
    A.qbs = (d.W + AF_ROWS - 1) / AF_ROWS;
    A.ranges = f32_ranges(d, part_floats);
    A.merged = A.ranges > AF_MAX_RANGES;
    A.waves = 0;
    const double c = (double)d.scale * AF_LOG2E;
    A.c = (float)c;
    A.c_lo = (float)(c - (double)A.c);
    A.ks0 = d.ks[0]; A.ks1 = d.ks[1]; A.ks2 = d.ks[2];
    if (d.dh == 64) launch_attn_f32_dh<64>(A, d, part, stats, a_raw, pass1, s);
    else launch_attn_f32_dh<128>(A, d, part, stats, a_raw, pass1, s);
    return hipGetLastError();
}

} // namespace ckv
