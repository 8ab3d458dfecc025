// Per-entry L1 magnitude of the projected value on the matrix cores (bf16 in, fp32 accumulate)
// (Theorem 3.3; Algorithm 1, lines 2-3):  N^h_i = sum_c | sum_t V^g[i,t] * W_O^h[t,c] |.
//
// This is a dense n x d_h by d_h x d_model contraction per query head whose n x d_model result is
// only needed as a row-wise sum of magnitudes, so the products live in MFMA accumulators, are
// folded into per-row partial sums by the epilogue and never reach memory.
//
// Tiling (written for d_h = 128; d_h = 64 runs the same kernel with two k-steps per chain and 256-column tiles):
//   * workgroup = 4 waves, two workgroups per CU; wave w owns RB blocks of 16 token rows whose V
//     fragments (4 k-steps of 32) stay in registers for the whole kernel: V is read once per
//     workgroup.  The product is taken transposed, (W_O^h)^T V^T: the streamed W_O fragment is the
//     MFMA A operand, shared by RB consecutive MFMAs, and the resident V fragments are B operands
//     (measured 1.3 % faster than the other way round; the fragment layouts are the same).
//   * the head's W_O slice, stored output-major ([d_model][H*d_h]: the 128 inner-dimension values
//     of an output column are contiguous), streams through LDS in tiles of TN columns, double
//     buffered, with direct buffer->LDS loads (no staging registers).  A wave-level direct load
//     fills 1 KiB of consecutive LDS, so the tile is unpadded [TN][256 B]; bank conflicts of the
//     fragment reads are avoided by storing 16-byte chunk q of column c at slot q ^ (c & 15).
//   * v_mfma_f32_16x16x32_bf16: a lane holds 8 consecutive k of row (A) / column (B) lane % 16 at
//     k offset 8 * (lane / 16); accumulator register v of a lane is row 4*(lane/16) + v, column
//     lane % 16, i.e. here output column 4*(lane/16) + v of token lane % 16.  This shape sustains a markedly higher rate than 32x32x16 on this part when the
//     operands are real (toggling) data, i.e. when the chip is power limited.
//   * software pipeline per 16-column block: 4 k-steps x RB row blocks of MFMAs into one accumulator
//     set while the previous block's set is drained with sum += |acc| (abs is a source modifier:
//     one VALU op per product, one per MFMA) and the next block's W_O fragments are fetched from LDS.
//     sched_barrier fences keep this order through the compiler's scheduler.
#include "vproj_mfma.hpp"

namespace ckv {

bool vproj_mfma_supported(const Dims &d)
{
    return (d.dh == 128 || d.dh == 64) && d.dm % (VM_TILE_BYTES / (d.dh * 2)) == 0 &&
           (size_t)d.dm * d.H * d.dh * 2 < ((size_t)1 << 31) &&
           ((long long)d.batch * d.H + 8) * (d.n / 64 + 2) < (1ll << 31);
}

VprojArgs vproj_mfma_args(const Dims &d, int row_blocks, const void *v, const void *w_t, float *vnorm, unsigned *wgs)
{
    VprojArgs P;
    P.v = (const bf16_t *)v; P.w_t = (const bf16_t *)w_t; P.vnorm = vnorm;
    P.H = d.H; P.G = d.G; P.n = d.n; P.dm = d.dm;
    P.vs0 = d.vs[0]; P.vs1 = d.vs[1]; P.vs2 = d.vs[2];
    const int rows_per_wg = VM_WAVES * row_blocks * 16;
    P.row_tiles = (d.n + rows_per_wg - 1) / rows_per_wg;
    P.heads = d.batch * d.H;
    P.pair = (size_t)2 * d.dh * d.dm * 2 <= ((size_t)2 << 20) ? 1 : 0; // two slices within 2 MiB
    *wgs = (unsigned)(8ll * (((long long)P.heads * P.row_tiles + 7) / 8)); // an eighth of the (head, row tile) items per XCD
    return P;
}

template <int DH, int RB>
__global__ __launch_bounds__(VM_THREADS, 2) void vproj_mfma_kernel(VprojArgs P)
{
    __shared__ __attribute__((aligned(1024))) char lds[VM_LDS];
    vproj_mfma_body<DH, RB>(P, lds, blockIdx.x);
}

template <int DH, int RB>
static void launch_rb(const Dims &d, const void *v, const void *w_t, float *vnorm, hipStream_t s)
{
    unsigned wgs;
    const VprojArgs P = vproj_mfma_args(d, RB, v, w_t, vnorm, &wgs);
    hipLaunchKernelGGL((vproj_mfma_kernel<DH, RB>), dim3(wgs), dim3(VM_THREADS), 0, s, P);
}

int cheapest_rounds(const Dims &d, int rows_per_block, double c2, double c1, const int *choices, int count)
{
    const long long heads = (long long)d.batch * d.H;
    int best = choices[0];
    double least = 0.0;
    for (int i = 0; i < count; ++i) {
        const int rb = choices[i], rows = rows_per_block * rb;
        const long long wgs = (heads * ((d.n + rows - 1) / rows) + 7) / 8, rest = wgs % 64;
        const double cost = (double)(wgs / 64) * (rb + c2) + (rest > 32 ? rb + c2 : rest > 0 ? 0.48 * rb + c1 : 0.0);
        if (i == 0 || cost < least) { least = cost; best = rb; }
    }
    return best;
}

// Row blocks per wave.  Many blocks stream W_O less often; few cut a short launch into enough workgroups to fill the
// chip (an XCD holds 64: two per CU), and the last round of workgroups is paid for whole.  A round's time was measured
// (d_model 4096, 2 .. 7 blocks; the ratios hold at 2048 and 5120) as proportional to RB + c when every CU holds two
// workgroups and to 0.48 RB + c1 when it holds one, with c = 1.07, c1 = 0.90 at d_h 128 and c = 1.84, c1 = 1.83 at
// d_h 64; the choice is the RB whose rounds cost least.  Against the fixed 6 (7 for the longest launches) that this
// replaces, 32 heads, us: n 1024 57.5 -> 34.4 (2 blocks), 2048 60.2 -> 50.7 (4), 4096 112.4 -> 91.6 (4), 8192
// 178.3 -> 176.0 (4); 6 and 7 as before from 12288 on.  d_h 64, d_model 2048: n 1024 20.6 -> 13.8, 8192 53.2 -> 48.6 (8
// blocks), 4 x 30000 646 -> 611 (10).
int vproj_mfma_row_blocks(const Dims &d)
{
    const int choices64[] = {10, 8, 6, 4, 3, 2}, choices128[] = {7, 6, 5, 4, 3, 2}; // (12 and 8 blocks spill)
    return d.dh == 64 ? cheapest_rounds(d, VM_WAVES * 16, 1.84, 1.83, choices64, 6)
                      : cheapest_rounds(d, VM_WAVES * 16, 1.07, 0.90, choices128, 6);
}

hipError_t launch_vproj_mfma(const Dims &d, const void *v, const void *w_t, float *vnorm, hipStream_t s)
{
    const int rb = vproj_mfma_row_blocks(d);
    if (d.dh == 64) {
        switch (rb) {
        case 10: launch_rb<64, 10>(d, v, w_t, vnorm, s); break;
        case 8: launch_rb<64, 8>(d, v, w_t, vnorm, s); break;
        case 6: launch_rb<64, 6>(d, v, w_t, vnorm, s); break;
        case 4: launch_rb<64, 4>(d, v, w_t, vnorm, s); break;
        case 3: launch_rb<64, 3>(d, v, w_t, vnorm, s); break;
        default: launch_rb<64, 2>(d, v, w_t, vnorm, s); break;
        }
    } else {
        switch (rb) {
        case 7: launch_rb<128, 7>(d, v, w_t, vnorm, s); break;
        case 6: launch_rb<128, 6>(d, v, w_t, vnorm, s); break;
        case 5: launch_rb<128, 5>(d, v, w_t, vnorm, s); break;
        case 4: launch_rb<128, 4>(d, v, w_t, vnorm, s); break;
        case 3: launch_rb<128, 3>(d, v, w_t, vnorm, s); break;
        default: launch_rb<128, 2>(d, v, w_t, vnorm, s); break;
        }
    }
    return hipGetLastError();
}

} // namespace ckv
