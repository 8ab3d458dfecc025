// Launches of short contexts: the second key sweep beside the projection, in one launch (bf16, d_h = 128, windows of up to
// 32 rows, up to four query heads per kv head).
//
// The projection of a context of up to about 3500 tokens (32 heads) puts one workgroup on a CU and is bound by the matrix
// cores; the sweep's workgroups, a few hundred at most, take the slots that are left and wait for memory and for each other's
// tiles there.  By itself the sweep is a launch of 7 us that fills an eighth of the chip.  Score call, 32 heads over 8,
// d_model 4096, causal, us, apart and with a launch that reduces the rows / together and merged: 600 tokens 48.1 / 38.3, 1024
// 51.8 / 43.2, 2048 69.3 / 60.4, 3072 89.0 / 79.4, 3500 96.7 / 88.2; from two workgroups per CU on there is no room beside the
// projection and nothing to gain (3700 tokens: 105.0 / 103.4, by the merge alone).  (256 keys per workgroup of the
// sweeps; with the 64 or 128 of short contexts, together: 600 tokens 37.0, 1024 41.0, 2048 57.7, 3072 78.3.)
//
// fp32 layers (below): the split of W_O beside the first sweep, and the project kernel beside the second one.
#include "vproj_mfma.hpp"
#include "vproj_split_f32.hpp"
#include "window_attn_f32.hpp"
#include "window_attn_mfma.hpp"

namespace ckv {

template <int RB>
__global__ __launch_bounds__(VM_THREADS, 2) void vproj_colsum_kernel(VprojArgs P, int vproj_wgs, AttnArgs A,
                                                                     const float *__restrict__ stats, float *__restrict__ a_raw)
{
    static_assert(attn_colsum_lds<1>() <= VM_LDS, "one buffer for either");
    __shared__ __attribute__((aligned(1024))) char lds[VM_LDS];
    const int wg = (int)blockIdx.x - vproj_wgs; // (uniform) the projection's workgroups come first
    if (wg < 0) vproj_mfma_body<AM_DH, RB>(P, lds, blockIdx.x);
    else attn_colsum_body<1>(A, stats, a_raw, lds, wg % A.chunks, wg / A.chunks, 0);
}

// One workgroup of the projection per CU at most: the other half of the chip's slots is the sweep's.
bool vproj_colsum_room(const Dims &d)
{
    if (d.attn_only || d.norm != CKV_NORM_L1 || d.dh != AM_DH || d.W > 32 || d.G > VM_WAVES || !vproj_mfma_supported(d)) return false;
    unsigned wgs;
    (void)vproj_mfma_args(d, vproj_mfma_row_blocks(d), nullptr, nullptr, nullptr, &wgs);
    return wgs <= 256;
}
bool vproj_colsum_taken(const Dims &d) { return vproj_colsum_room(d) && attn_mfma_merges(d); }

hipError_t launch_vproj_colsum(const Dims &d, const void *q, const void *k, const void *v, const void *w_t, const float *part,
                               float *a_raw, float *vnorm, hipStream_t s)
{
    const int rb = vproj_mfma_row_blocks(d);
    unsigned wgs;
    const VprojArgs P = vproj_mfma_args(d, rb, v, w_t, vnorm, &wgs);
    const AttnArgs A = attn_mfma_args(d, q, k);
    const dim3 grid(wgs + A.chunks * d.batch * d.Hkv), block(VM_THREADS);
    switch (rb) {
    case 7: hipLaunchKernelGGL(vproj_colsum_kernel<7>, grid, block, 0, s, P, (int)wgs, A, part, a_raw); break;
    case 6: hipLaunchKernelGGL(vproj_colsum_kernel<6>, grid, block, 0, s, P, (int)wgs, A, part, a_raw); break;
    case 5: hipLaunchKernelGGL(vproj_colsum_kernel<5>, grid, block, 0, s, P, (int)wgs, A, part, a_raw); break;
    case 4: hipLaunchKernelGGL(vproj_colsum_kernel<4>, grid, block, 0, s, P, (int)wgs, A, part, a_raw); break;
    case 3: hipLaunchKernelGGL(vproj_colsum_kernel<3>, grid, block, 0, s, P, (int)wgs, A, part, a_raw); break;
    default: hipLaunchKernelGGL(vproj_colsum_kernel<2>, grid, block, 0, s, P, (int)wgs, A, part, a_raw); break;
    }
    return hipGetLastError();
}

// ---- fp32 ------------------------------------------------------------------------------------------------------------
// Two pairs of kernels that do not depend on each other: of four launches in a chain, two are left.  Score call, us,
// four launches / two: 4 heads, d_h 64, d_model 256, 512 tokens 19.9 / 13.2, 1024 20.8 / 13.4, 4096 22.5 / 16.8 (a third one merges
// the rows' pairs there); 16 heads over 4, d_h 128, d_model 2048, 1024 tokens 63.9 / 62.4, 2048 76.6 / 74.5, 4096 105.5 / 105.8 (both
// want the matrix cores there).  With two workgroups of the project kernel per CU there is no room beside it.
template <int DH, bool OUT_IN>
__global__ __launch_bounds__(VS_THREADS, 2) void split_stats_kernel(SplitArgs P, int split_wgs, AttnF32Args A, float *__restrict__ part)
{
    static_assert(VS_THREADS == 64 * AF_WAVES, "workgroups of either kind");
    const int wg = (int)blockIdx.x - split_wgs, tiles = P.dm / VS_TN; // (uniform)
    if (wg < 0) split_wo_body<DH, OUT_IN>(P.w_o, (f16_t *)P.parts, (float *)P.factors, P.H, P.dm, blockIdx.x % tiles, blockIdx.x / tiles);
    else attn_stats_f32_body<DH, 4>(A, part, wg);
}

template <int DH, int RB>
__global__ __launch_bounds__(VS_THREADS, 2) void split_colsum_kernel(SplitArgs P, int vproj_wgs, AttnF32Args A,
                                                                     const float *__restrict__ rows, float *__restrict__ a_raw)
{
    static_assert(sizeof(F32RowStat) * AF_WAVES <= 2 * SGeo<DH>::TILE_BYTES, "one buffer for either");
    __shared__ __attribute__((aligned(1024))) char lds[2 * SGeo<DH>::TILE_BYTES];
    const int wg = (int)blockIdx.x - vproj_wgs; // (uniform) the project kernel's workgroups come first
    if (wg < 0) vproj_split_body<DH, RB, false>(P, lds, blockIdx.x);
    else attn_colsum_f32_body<DH, 4>(A, rows, a_raw, reinterpret_cast<F32RowStat *>(lds), wg);
}

bool split_colsum_taken(const Dims &d)
{
    if (d.norm != CKV_NORM_L1) return false;
    unsigned wgs;
    (void)vproj_split_args(d, vproj_split_row_blocks(d), 0, nullptr, nullptr, nullptr, nullptr, &wgs);
    return wgs <= 256;
}

template <int DH>
static void launch_split_stats(const SplitArgs &P, const AttnF32Args &A, float *part, hipStream_t s)
{
    const int split_wgs = P.dm / VS_TN * P.H;
    const dim3 grid(split_wgs + attn_f32_wgs(A)), block(VS_THREADS);
    if (P.out_in) hipLaunchKernelGGL((split_stats_kernel<DH, true>), grid, block, 0, s, P, split_wgs, A, part);
    else hipLaunchKernelGGL((split_stats_kernel<DH, false>), grid, block, 0, s, P, split_wgs, A, part);
}

template <int DH, int RB>
static void launch_split_colsum(const SplitArgs &P, unsigned wgs, const AttnF32Args &A, const float *rows, float *a_raw, hipStream_t s)
{
    hipLaunchKernelGGL((split_colsum_kernel<DH, RB>), dim3(wgs + attn_f32_wgs(A)), dim3(VS_THREADS), 0, s, P, (int)wgs, A, rows, a_raw);
}

hipError_t launch_score_f32_short(const Dims &d, int out_in, const void *q, const void *k, const void *v, const void *w_o,
                                  void *scratch, float *part, size_t part_floats, float *stats, float *a_raw, float *vnorm,
                                  hipStream_t s)
{
    const int rb = vproj_split_row_blocks(d);
    unsigned wgs;
    const SplitArgs P = vproj_split_args(d, rb, out_in, v, w_o, scratch, vnorm, &wgs);
    const AttnF32Args A1 = attn_f32_args(d, q, k, part_floats, true), A2 = attn_f32_args(d, q, k, part_floats, false);
    if (d.dh == 64) launch_split_stats<64>(P, A1, part, s);
    else launch_split_stats<128>(P, A1, part, s);
    hipError_t e = launch_attn_f32_merge(d, A1, part, stats, s);
    if (e != hipSuccess) return e;
    const float *rows = A1.merged ? stats : part;
    if (d.dh == 64) {
        switch (rb) {
        case 6: launch_split_colsum<64, 6>(P, wgs, A2, rows, a_raw, s); break;
        case 5: launch_split_colsum<64, 5>(P, wgs, A2, rows, a_raw, s); break;
        case 4: launch_split_colsum<64, 4>(P, wgs, A2, rows, a_raw, s); break;
        case 3: launch_split_colsum<64, 3>(P, wgs, A2, rows, a_raw, s); break;
        case 2: launch_split_colsum<64, 2>(P, wgs, A2, rows, a_raw, s); break;
        default: launch_split_colsum<64, 1>(P, wgs, A2, rows, a_raw, s); break;
        }
    } else {
        switch (rb) {
        case 4: launch_split_colsum<128, 4>(P, wgs, A2, rows, a_raw, s); break;
        case 3: launch_split_colsum<128, 3>(P, wgs, A2, rows, a_raw, s); break;
        case 2: launch_split_colsum<128, 2>(P, wgs, A2, rows, a_raw, s); break;
        default: launch_split_colsum<128, 1>(P, wgs, A2, rows, a_raw, s); break;
        }
    }
    return hipGetLastError();
}

} // namespace ckv
