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
// 1.1e-7; two cost 1 %, four 2 - 4 (the sums' additions, which nothing covers where a SIMD has one wave; at d_h 64, with the
// registers they take, 10).  Two here; four where the sweeps share their launches, and nothing is seen of the cost.
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
#include "window_attn_f32.hpp"

namespace ckv {

template <int DH>
__global__ __launch_bounds__(64 * AF_WAVES, 2) void attn_stats_f32_kernel(AttnF32Args A, float *__restrict__ part)
{
    attn_stats_f32_body<DH, AF_CHAINS>(A, part, blockIdx.x);
}

template <int DH>
__global__ __launch_bounds__(64 * AF_WAVES, DH == 64 ? 3 : 2) void attn_colsum_f32_kernel(AttnF32Args A, const float *__restrict__ part,
                                                                           float *__restrict__ a_raw)
{
    __shared__ __attribute__((aligned(16))) F32RowStat stat[AF_WAVES];
    attn_colsum_f32_body<DH, AF_CHAINS>(A, part, a_raw, stat, blockIdx.x);
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

AttnF32Args attn_f32_args(const Dims &d, const void *q, const void *k, size_t part_floats, bool pass1)
{
    AttnF32Args A;
    A.q = (const float *)q; A.k = (const float *)k;
    A.H = d.H; A.G = d.G; A.n = d.n; A.W = d.W; A.causal = d.causal;
    A.qbs = (d.W + AF_ROWS - 1) / AF_ROWS;
    A.ranges = f32_ranges(d, part_floats);
    A.merged = A.ranges > AF_MAX_RANGES;
    A.waves = d.batch * d.H * A.ranges * (pass1 ? A.qbs : 1);
    A.post = d.window_sum ? 1.0f : 1.0f / (float)d.W;
    const double c = (double)d.scale * AF_LOG2E;
    A.c = (float)c;
    A.c_lo = (float)(c - (double)A.c);
    A.ks0 = d.ks[0]; A.ks1 = d.ks[1]; A.ks2 = d.ks[2];
    return A;
}

hipError_t launch_attn_f32_merge(const Dims &d, const AttnF32Args &A, const float *part, float *stats, hipStream_t s)
{
    if (!A.merged) return hipSuccess;
    hipLaunchKernelGGL(attn_merge_f32_kernel, dim3(d.batch * d.H * d.W), dim3(64), 0, s, part, stats, A.ranges, A.post);
    return hipGetLastError();
}

hipError_t launch_attn_f32(const Dims &d, const void *q, const void *k, float *part, size_t part_floats, float *stats,
                           float *a_raw, bool pass1, hipStream_t s)
{
    const AttnF32Args A = attn_f32_args(d, q, k, part_floats, pass1);
    const dim3 grid(attn_f32_wgs(A)), block(64 * AF_WAVES);
    if (pass1) {
        if (d.dh == 64) hipLaunchKernelGGL(attn_stats_f32_kernel<64>, grid, block, 0, s, A, part);
        else hipLaunchKernelGGL(attn_stats_f32_kernel<128>, grid, block, 0, s, A, part);
        return launch_attn_f32_merge(d, A, part, stats, s);
    }
    const float *rows = A.merged ? stats : part;
    if (d.dh == 64) hipLaunchKernelGGL(attn_colsum_f32_kernel<64>, grid, block, 0, s, A, rows, a_raw);
    else hipLaunchKernelGGL(attn_colsum_f32_kernel<128>, grid, block, 0, s, A, rows, a_raw);
    return hipGetLastError();
}

} // namespace ckv
