// Launches of short contexts: the second key sweep beside the projection, in one launch (bf16, d_h = 128, windows of up to
// 32 rows, up to four query heads per kv head).
//
// The projection of a context of up to about 3500 tokens (32 heads) puts one workgroup on a CU and is bound by the matrix
// cores; the sweep's workgroups, a few hundred at most, take the slots that are left and wait for memory and for each other's
// tiles there.  By itself the sweep is a launch of 7 us that fills an eighth of the chip.  Score call, 32 heads over 8,
// d_model 4096, causal, us, apart and with a launch that reduces the rows / together and merged: 600 tokens 48.1 / 38.3, 1024
// 51.8 / 43.2, 2048 69.3 / 60.4, 3072 89.0 / 79.4, 3500 96.7 / 88.2; from two workgroups per CU on there is no room beside the
// projection and nothing to gain (3700 tokens: 105.0 / 103.4, by the merge alone).
#include "vproj_mfma.hpp"
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
bool vproj_colsum_taken(const Dims &d)
{
    if (d.norm != CKV_NORM_L1 || d.dh != AM_DH || d.W > 32 || d.G > VM_WAVES || !attn_mfma_merges(d)) return false;
    unsigned wgs;
    (void)vproj_mfma_args(d, vproj_mfma_row_blocks(d), nullptr, nullptr, nullptr, &wgs);
    return wgs <= 256;
}

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

} // namespace ckv
