// Per-entry L1 (or L2) magnitude of the projected value for fp32 layers, on the f16 matrix cores
// (Theorem 3.3; Algorithm 1, lines 2-3):  N^h_i = sum_c | sum_t V^g[i,t] * W_O^h[t,c] |.
//
// An fp32 number is the sum of two f16 numbers once a power of two has brought it into f16's range:
//   x * s = hi + lo,  hi = f16(x * s), lo = f16(x * s - hi), the difference exact.
// A token's row of V and a tile of W_O (d_h rows by 32 columns of a head) have a scale each that takes their largest
// entry to [2^14, 2^15).  The two parts hold 23 of fp32's 24 bits at least: a quarter of the values lose their last one
// (2^-23 of x; rms 2^-24), and a subnormal lo rounds by 2^-40 of the row's or tile's largest entry (the instruction takes
// subnormal operands as they are).  Of the four products of v * w the one that is left out, lo * lo, is at most 2^-22 of it
// (rms 2^-24.6); the three others are exact in the MFMA's fp32 accumulators and are added smallest first.  In all 9e-8 of a
// product (rms), random in sign: over the d_model columns of a magnitude that is far below the rounding of its sums, and the
// last of these, which were most of the error, are in 64 bits.
//
//   split     W_O once per call into [head][d_model][2 parts][d_h] (and from the canonical layout to output-major), with
//             a factor per tile that undoes its scale
//   project   the tiling of the bf16 kernel: a wave keeps RB blocks of 16 token rows (both parts) as MFMA fragments, the
//             head's parts stream through LDS in tiles of 32 columns (16 KiB at d_h 128, double buffered, direct
//             buffer->LDS loads, 16-byte chunks swizzled), three MFMAs per (k-step, row block), the previous column
//             block's |acc| times the tile's factor added up under them.  Rows whose operands do not fit the scheme are
//             computed again from the fp32 operands (exact_rows): those that meet an infinity, a NaN or a row or tile
//             whose largest entry lies outside 2^-60 .. 2^60 (they come out as NaN), and those whose result is so small
//             against their operands' largest entries that the error of the small entries might show (VS_SMALL).
//
// What bounds it: the matrix cores, at three f16 MFMAs per fp32 product, 5 times the rate of the fp32 MFMA (157 TFLOP/s
// nominal).  (Three bf16 parts per operand and six products, which need no scales, took twice the matrix work.)
// Measured, score call at 16 query heads over 4 kv heads, d_h 128, d_model 2048, 8192 tokens: 2.57 ms on the vector ALUs
// (27 TFLOP/s), 0.287 with the six bf16 products, 0.174 like this (the project kernel 240 -> 139 us).  The magnitudes' error
// against 64 bits (2-norm, means over 9 and 30 layers): d_model 2048 6.7e-7 / 5.7e-8 / 4.9e-8, d_model 256 and d_h 64
// 2.4e-7 / 4.2e-8 / 3.3e-8 (vector / six bf16 products / this, whose last additions are in 64 bits).
#include "vproj_split_f32.hpp"

namespace ckv {

template <int DH, bool OUT_IN>
__global__ __launch_bounds__(VS_THREADS) void split_wo_kernel(const float *__restrict__ w, f16_t *__restrict__ out,
                                                              float *__restrict__ factor, int H, int dm)
{
    split_wo_body<DH, OUT_IN>(w, out, factor, H, dm, blockIdx.x, blockIdx.y);
}

template <int DH, int RB, bool L2>
__global__ __launch_bounds__(VS_THREADS, 2) void vproj_split_kernel(SplitArgs P)
{
    __shared__ __attribute__((aligned(1024))) char lds[2 * SGeo<DH>::TILE_BYTES];
    vproj_split_body<DH, RB, L2>(P, lds, blockIdx.x);
}

SplitArgs vproj_split_args(const Dims &d, int row_blocks, int out_in, const void *v, const void *w_o, void *scratch, float *vnorm,
                           unsigned *wgs)
{
    SplitArgs P;
    P.v = (const float *)v; P.w_o = (const float *)w_o;
    P.parts = (const f16_t *)scratch;
    P.factors = (const float *)(P.parts + (size_t)d.H * d.dh * d.dm * VS_PARTS);
    P.vnorm = vnorm;
    P.out_in = out_in; P.H = d.H; P.G = d.G; P.n = d.n; P.dm = d.dm;
    P.vs0 = d.vs[0]; P.vs1 = d.vs[1]; P.vs2 = d.vs[2];
    const int rows_per_wg = VS_WAVES * row_blocks * 16;
    P.row_tiles = (d.n + rows_per_wg - 1) / rows_per_wg;
    P.heads = d.batch * d.H;
    *wgs = (unsigned)(8ll * (((long long)P.heads * P.row_tiles + 7) / 8));
    return P;
}

// The parts (4 bytes per entry) and a factor per tile; 6 bytes per entry are what callers size the workspace by.
size_t vproj_split_bytes(const Dims &d) { return (size_t)d.H * d.dh * d.dm * 6; }

bool vproj_split_supported(const Dims &d)
{
    return (d.dh == 64 || d.dh == 128) && d.dm % VS_TN == 0 && (size_t)d.dm * VS_PARTS * d.dh * 2 < ((size_t)1 << 31) &&
           ((long long)d.batch * d.H + 8) * (d.n / 64 + 2) < (1ll << 31) && d.H < 65536;
}

// Row blocks per wave, by the cost of the launch's rounds: an XCD holds 64 workgroups (two per CU); a round's time is
// proportional to RB + c2 with two workgroups on every CU and to 0.48 RB + c1 with one.  Over 512 .. 16384 tokens, 16 heads,
// every choice timed, the rule's is within 1 % of the best (3.5 % at one length).  The stage's time with 1 / 2 / 3 / 4 blocks,
// us: d_h 128, d_model 2048: n 1024 49 / 52 / 63 / 72, 4096 96 / 87 / 102 / 82, 6144 136 / 121 / 116 / 129, 16384 334 / 294 /
// 300 / 272; d_h 64, d_model 1024, 1 / 2 / 4 / 6 blocks: 2048 24 / 24 / 29 / 35, 8192 52 / 47 / 45 / 56, 12288 72 / 66 / 62 / 62.
int vproj_split_row_blocks(const Dims &d)
{
    const int choices[] = {6, 5, 4, 3, 2, 1}; // (the registers hold four blocks at d_h 128)
    return d.dh == 64 ? cheapest_rounds(d, VS_WAVES * 16, 0.55, 0.55, choices, 6)
                      : cheapest_rounds(d, VS_WAVES * 16, 0.40, 0.38, choices + 2, 4);
}

template <int DH>
static void launch_split(const Dims &d, int out_in, const SplitArgs &P, hipStream_t s)
{
    const dim3 grid(d.dm / VS_TN, d.H), block(VS_THREADS);
    f16_t *parts = (f16_t *)P.parts;
    float *factors = (float *)P.factors;
    if (out_in) hipLaunchKernelGGL((split_wo_kernel<DH, true>), grid, block, 0, s, P.w_o, parts, factors, d.H, d.dm);
    else hipLaunchKernelGGL((split_wo_kernel<DH, false>), grid, block, 0, s, P.w_o, parts, factors, d.H, d.dm);
}

template <int DH, int RB>
static void launch_project(const Dims &d, const SplitArgs &P, unsigned wgs, hipStream_t s)
{
    if (d.norm == CKV_NORM_L2) hipLaunchKernelGGL((vproj_split_kernel<DH, RB, true>), dim3(wgs), dim3(VS_THREADS), 0, s, P);
    else hipLaunchKernelGGL((vproj_split_kernel<DH, RB, false>), dim3(wgs), dim3(VS_THREADS), 0, s, P);
}

hipError_t launch_vproj_split(const Dims &d, int out_in, const void *v, const void *w_o, void *scratch, float *vnorm, hipStream_t s)
{
    const int rb = vproj_split_row_blocks(d);
    unsigned wgs;
    const SplitArgs P = vproj_split_args(d, rb, out_in, v, w_o, scratch, vnorm, &wgs);
    if (d.dh == 64) {
        launch_split<64>(d, out_in, P, s);
        switch (rb) {
        case 6: launch_project<64, 6>(d, P, wgs, s); break;
        case 5: launch_project<64, 5>(d, P, wgs, s); break;
        case 4: launch_project<64, 4>(d, P, wgs, s); break;
        case 3: launch_project<64, 3>(d, P, wgs, s); break;
        case 2: launch_project<64, 2>(d, P, wgs, s); break;
        default: launch_project<64, 1>(d, P, wgs, s); break;
        }
    } else {
        launch_split<128>(d, out_in, P, s);
        switch (rb) {
        case 4: launch_project<128, 4>(d, P, wgs, s); break;
        case 3: launch_project<128, 3>(d, P, wgs, s); break;
        case 2: launch_project<128, 2>(d, P, wgs, s); break;
        default: launch_project<128, 1>(d, P, wgs, s); break;
        }
    }
    return hipGetLastError();
}

} // namespace ckv
