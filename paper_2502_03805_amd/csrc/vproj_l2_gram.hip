// L2 magnitude of the projected value through the Gram matrix (bf16, d_h = 128)
// (the L2 variant of the distance the paper mentions beside its L1 default; Theorem 3.3's row norm with
// the 2-norm):   N^h_i = || v_i W_O^h ||_2 = sqrt( v_i G^h v_i^T ),   G^h = W_O^h W_O^h^T  (d_h x d_h).
//
// The shortcut is exact for the 2-norm only (for L1 the n x d_model products are needed).  It replaces the
// n x d_h x d_model contraction by n x d_h x d_h: 32 times less MFMA work at d_model = 4096.
//
//   gram_partial  G^h over a slice of the d_model columns on the matrix cores, from the canonical W_O (exact products,
//                 fp32 sums; W_O is a weight: this is a per-layer constant, a few GFLOP)
//   gram_finish   sums the slices, folds the symmetric G onto its lower block triangle (32 x 32 blocks: those
//                 below the diagonal doubled, those above dropped -- the quadratic form is unchanged and
//                 12 of the 32 block products fall away) and splits it into two bf16 matrices G_hi + G_lo
//                 (error ~2^-17 relative), stored [head][u][t]
//   l2 kernel     one workgroup per (query head, range of rows) with the head's two G matrices (64 KiB) resident in
//                 LDS; V rows stream through registers as MFMA B fragments,  Y^T = G V^T  is accumulated with
//                 v_mfma_f32_16x16x32_bf16 over G_hi and G_lo, and the epilogue multiplies by v again:
//                 N^2_i = sum_u Y[i,u] v[i,u].
#include <type_traits>

#include "common.hpp"

namespace ckv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int GL_DH = 128;
constexpr int GL_SLICES = 4;          // d_model slices of the Gram partial sums
constexpr int GL_G_BYTES = GL_DH * GL_DH * 2; // one bf16 Gram matrix: 32 KiB

#define LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

__device__ __forceinline__ bf16_t f32_to_bf16_rne(float x)
{
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

// partial[head][slice][u][t] = sum over the slice's columns c of W_O[h*128+u][c] * W_O[h*128+t][c], for the 32 x 32 blocks
// on and below the diagonal (G is symmetric).
//
// v_mfma_f32_16x16x4_f32: a lane holds row (A) / column (B) lane % 16 at k = lane / 16; accumulator v is row
// 4 * (lane / 16) + v, column lane % 16.  The products of bf16 values are exact in fp32 and the instruction adds its four
// products one after the other, so a chain over ascending columns has the bits of a scalar fmaf loop (checked against
// one).  The bf16 form of the instruction would be faster still, but it sums in another order, and every value of G that
// lies near a tie of G_hi's rounding would then move between the two parts of the stored constant.
//
// Work split: a chain runs over a whole slice, so the blocks are what is dealt out: 40 blocks of 16 x 16 per (head,
// slice), 20 per workgroup, runs of two or three per wave (one accumulator chain each).  The workgroup's tile, 128 rows x 64
// columns of the canonical W_O (rows contiguous along d_model), sits in LDS with each row's even words before its odd ones,
// so that a lane's values of 16 columns are one 16-byte read, at a pitch of 36 words (the 16 rows of a read start on 16
// different bank groups); the next two tiles are in registers meanwhile.
// Bound by the fp32 matrix rate (157 TFLOP/s nominal; 2.7 GFLOP at 32 heads and d_model 4096 are 17 us) and the operand
// reads under it: 28 us in a chain of calls, 33 under the kernel trace.  Before, on the way here: fp32 products on the vector ALUs from the output-major layout 229 us
// and a layout change of 21 us before it; single words instead of 16-byte reads 56; five blocks per wave, one wave per
// SIMD, 47; two per wave, ten waves (six blocks on the fullest SIMD, an A read per block) 34.
constexpr int GP_CHUNK = 64;                   // columns per LDS tile
constexpr int GP_HALF = GP_CHUNK / 4;          // words of a row that lanes with k = 0, 1 read (the others read the rest)
constexpr int GP_PITCH = 2 * GP_HALF + 4;      // words per row
constexpr int GP_WAVES = 8;                    // waves per workgroup; the threads move two 16-byte pieces of a tile each
constexpr int GP_BLOCKS = 3;                   // 16 x 16 blocks per wave at most

// Runs of blocks in one block row i (16 rows of G; it has (i | 1) + 1 blocks, up to the end of its 32 x 32 diagonal block):
// eight runs of three and eight of two make up the 40.  A workgroup takes four of each, its waves 0-3 the runs of three
// and 4-7 those of two: waves w and w + 4 share a SIMD, which so gets five blocks.  A run reads its A operand once.
struct GramRun { int8_t i, j; };
__device__ constexpr GramRun GP_RUNS[2][GP_WAVES] = {
    {{4, 0}, {4, 3}, {5, 0}, {5, 3}, {0, 0}, {1, 0}, {2, 0}, {2, 2}},
    {{6, 0}, {6, 3}, {7, 0}, {7, 3}, {3, 0}, {3, 2}, {6, 6}, {7, 6}},
};

__global__ __launch_bounds__(64 * GP_WAVES) void gram_partial_kernel(const bf16_t *__restrict__ w_o, float *__restrict__ partial, int dm)
{
    __shared__ __attribute__((aligned(16))) uint32_t tile[2][GL_DH * GP_PITCH];
    const int h = blockIdx.x, slice = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const int cols = dm / GL_SLICES; // host guarantees dm % (GL_SLICES * GP_CHUNK) == 0
    const int bi = GP_RUNS[blockIdx.z][wave].i, bj = GP_RUNS[blockIdx.z][wave].j;
    const bool three = wave < GP_WAVES / 2; // uniform over the wave
    // word of this lane's row inside the tile, for k = lane / 16 of the first four columns; the run's blocks follow each other
    const int aoff = (bi * 16 + l16) * GP_PITCH + (kg >> 1) * GP_HALF;
    const int boff = (bj * 16 + l16) * GP_PITCH + (kg >> 1) * GP_HALF;
    // odd columns are the upper halves of their words; a bf16 value is the upper half of its fp32
    const uint32_t pick = (kg & 1) ? 0x07060C0Cu : 0x05040C0Cu;
    auto value = [&](uint32_t w) { return __uint_as_float(__builtin_amdgcn_perm(w, 0u, pick)); };

    // staging: 8 pieces per row; two tiles are in flight in registers while a third is worked on
    const bf16_t *src = w_o + ((size_t)h * GL_DH + (threadIdx.x >> 3)) * dm + slice * cols + (threadIdx.x & 7) * 8;
    const int tiles = cols / GP_CHUNK; // even: d_model is a multiple of 512
    auto fetch = [&](int t, uint4 (&piece)[2]) __attribute__((always_inline)) {
        const int c0 = min(t, tiles - 1) * GP_CHUNK;
#pragma unroll
        for (int j = 0; j < 2; ++j) piece[j] = *reinterpret_cast<const uint4 *>(src + (size_t)j * (GL_DH / 2) * dm + c0);
    };
    auto stash = [&](uint32_t *to, const uint4 (&piece)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            uint32_t *p = to + (j * (GL_DH / 2) + (threadIdx.x >> 3)) * GP_PITCH + (threadIdx.x & 7) * 2;
            *reinterpret_cast<uint2 *>(p) = make_uint2(piece[j].x, piece[j].z);
            *reinterpret_cast<uint2 *>(p + GP_HALF) = make_uint2(piece[j].y, piece[j].w);
        }
    };
    f32x4 acc[GP_BLOCKS];
#pragma unroll
    for (int x = 0; x < GP_BLOCKS; ++x) acc[x] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto run = [&](auto blocks_c, const uint32_t *cur) __attribute__((always_inline)) {
        constexpr int BLOCKS = decltype(blocks_c)::value;
#pragma unroll
        for (int q = 0; q < GP_HALF / 4; ++q) { // 16 columns: four words per lane and operand, four steps of the chains
            const uint4 a = *reinterpret_cast<const uint4 *>(cur + aoff + 4 * q);
            uint4 b[BLOCKS];
#pragma unroll
            for (int x = 0; x < BLOCKS; ++x) b[x] = *reinterpret_cast<const uint4 *>(cur + boff + x * 16 * GP_PITCH + 4 * q);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float av = value(k == 0 ? a.x : k == 1 ? a.y : k == 2 ? a.z : a.w);
#pragma unroll
                for (int x = 0; x < BLOCKS; ++x) {
                    const uint32_t wb = k == 0 ? b[x].x : k == 1 ? b[x].y : k == 2 ? b[x].z : b[x].w;
                    acc[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, value(wb), acc[x], 0, 0, 0);
                }
            }
        }
    };
    auto work = [&](const uint32_t *cur) __attribute__((always_inline)) {
        if (three) run(std::integral_constant<int, 3>{}, cur);
        else run(std::integral_constant<int, 2>{}, cur);
    };
    uint4 even[2], odd[2]; // pieces of the next even and odd tile
    fetch(0, even);
    fetch(1, odd);
    stash(tile[0], even);
    __syncthreads();
    for (int t = 0; t < tiles; t += 2) {
        fetch(t + 2, even);
        work(tile[0]);
        stash(tile[1], odd); // (read last before the previous barrier)
        __syncthreads();
        fetch(t + 3, odd);
        work(tile[1]);
        stash(tile[0], even);
        __syncthreads();
    }
    float *dst = partial + ((size_t)h * GL_SLICES + slice) * GL_DH * GL_DH;
#pragma unroll
    for (int x = 0; x < GP_BLOCKS; ++x) {
        if (x < 2 || three)
#pragma unroll
            for (int v = 0; v < 4; ++v) dst[(bi * 16 + 4 * kg + v) * GL_DH + (bj + x) * 16 + l16] = acc[x][v];
    }
}

// G = sum of the slices (fixed order), folded onto its lower block triangle, split into hi + lo bf16;
// gram[head][0 = hi, 1 = lo][u][t].  One element per thread, 64 workgroups per head (a single workgroup per head: 22 us).
__global__ __launch_bounds__(256) void gram_finish_kernel(const float *__restrict__ partial, bf16_t *__restrict__ gram)
{
    const int h = blockIdx.y, e = blockIdx.x * 256 + threadIdx.x; // e = u * 128 + t
    const int bu = e >> 12, bt = (e & (GL_DH - 1)) >> 5;
    float g = 0.f;
    if (bt <= bu) { // (the other blocks hold nothing)
#pragma unroll
        for (int s = 0; s < GL_SLICES; ++s) g += partial[((size_t)h * GL_SLICES + s) * GL_DH * GL_DH + e];
    }
    // v G v^T = sum over the 32 x 32 blocks (bu, bt) on and below the diagonal, the ones below it counted twice: the
    // kernel reads those blocks only (20 of the 32 block products)
    g = bt < bu ? 2.f * g : g;
    const bf16_t hi = f32_to_bf16_rne(g);
    const bf16_t lo = f32_to_bf16_rne(g - bf16_to_f32(hi));
    gram[((size_t)h * 2 + 0) * GL_DH * GL_DH + e] = hi;
    gram[((size_t)h * 2 + 1) * GL_DH * GL_DH + e] = lo;
}

// N^h_i for HEADS query heads of a kv group and one range of rows, with the heads' Gram matrices resident in LDS.
//
// One workgroup of 4 * HEADS waves per (HEADS query heads, range of rows): two 4-wave workgroups per CU with one
// head each, or one 8-wave workgroup with two.  The heads' G_hi | G_lo (64 KiB each) are fetched once, at the
// start; after the one barrier that follows, every wave is on its own: it walks its blocks of GR_RB x 16 rows,
// requests the next block's V fragments (global -> registers) before it starts on the current one, and runs the
// block through the workgroup's heads, reading the Gram fragments it needs from LDS.  No barrier and no Gram
// traffic in the loop.  V is read once per workgroup of a kv group; the workgroups that work on the same rows are
// neighbours in launch order on one XCD (workgroup L of a 1-D grid runs on XCD L % 8), so the later readers of a
// row find it in that XCD's L2.  Two heads per workgroup halve the V traffic (6 % faster with four heads per
// group); with an odd number of heads the workgroup that is left with one head would idle half of the time
// (measured 6 % slower with five), so such groups take one head per workgroup.
constexpr int GR_RB = 4;
constexpr int GR_BLOCK_ROWS = GR_RB * 16;
constexpr int GR_AHEAD = 3;           // vproj_l2_long_kernel: k-chunks of V held twice
constexpr int GR_LONG_BLOCKS = 4;     // blocks per wave from which it is taken

template <int HEADS>
__global__ __launch_bounds__(HEADS * 256, HEADS == 1 ? 2 : 1) void vproj_l2_resident_kernel(const bf16_t *__restrict__ v,
                                                                             const bf16_t *__restrict__ gram,
                                                                             float *__restrict__ vnorm, int H, int G, int n,
                                                                             int64_t vs0, int64_t vs1, int64_t vs2, int pairs,
                                                                             int ranges, int rows_per_range)
{
    constexpr int GR_HEADS = HEADS, GR_WAVES = 4 * HEADS;
    __shared__ __attribute__((aligned(1024))) char lds[GR_HEADS * 2 * GL_G_BYTES]; // per head: G_hi | G_lo, XOR-swizzled
    const int Hkv = H / G, hgroups = G / GR_HEADS; // (the launcher takes HEADS = 2 for even G only)
    // an XCD takes an eighth of the (kv head, range of rows) items; the workgroups of a kv group that share one are
    // neighbours in launch order
    const int items = pairs * ranges, per_xcd = (items + 7) >> 3;
    const int hl = ((int)blockIdx.x >> 3) % hgroups * GR_HEADS; // first head of this workgroup inside its kv group
    const int k_in_xcd = ((int)blockIdx.x >> 3) / hgroups, item = ((int)blockIdx.x & 7) * per_xcd + k_in_xcd;
    if (k_in_xcd >= per_xcd || item >= items) return; // uniform over the workgroup
    const int range = item % ranges, pair = item / ranges;
    const int bi = pair / Hkv, g = pair % Hkv, h = g * G + hl;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kc = lane >> 4;
    const int row_begin = range * rows_per_range;            // a multiple of GR_BLOCK_ROWS
    const int row_end = min(n, row_begin + rows_per_range);
    if (row_begin >= row_end) return;                        // uniform over the workgroup
    const int nblk = (row_end - row_begin + GR_BLOCK_ROWS - 1) / GR_BLOCK_ROWS;
    const bf16_t *vbase = v + bi * vs0 + g * vs1;

    for (int hh = 0; hh < GR_HEADS; ++hh) {   // a head's 64 KiB: 64 direct loads of 1 KiB; row u of a matrix is 256 B = 16 chunks;
        // chunk q sits at slot q ^ f(u), f(u) = 4 * ((u / 8) % 4) + u % 4: the 16 rows that one MFMA A operand reads
        // together (see below) have 16 different f, so their 16-byte reads fall on different banks
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(gram + (size_t)(h + hh) * 2 * GL_DH * GL_DH), 0, 2 * GL_G_BYTES, 0x00020000);
#pragma unroll
        for (int j = 0; j < 64 / GR_WAVES; ++j) {
            const int kib = j * GR_WAVES + wave;
            const int urow = (kib * 4 + (lane >> 4)) & (GL_DH - 1);
            const int f = ((urow >> 3) & 3) * 4 + (urow & 3);
            const uint32_t voff = (uint32_t)(kib * 1024 + (lane >> 4) * 256 + (((lane & 15) ^ f) * 16));
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, LDS_PTR(lds + hh * 2 * GL_G_BYTES + kib * 1024), 16, voff, 0, 0, 0);
        }
    }
    // V rows through a buffer descriptor over this kv head's rows (the host checks that they span less than 2 GiB, so
    // 32-bit byte offsets do).  Rows past n - 1 re-read row n - 1 (never stored): the clamp is in the lane's
    // offset, because the descriptor's range check does not see the scalar offset.
    const __amdgpu_buffer_rsrc_t vrsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)vbase, 0, (int)(((int64_t)(n - 1) * vs2 + GL_DH) * 2), 0x00020000);
    const uint32_t row_bytes = (uint32_t)(vs2 * 2);
    // a block's V fragments in two halves: k-chunks 0-1 (the row's first 128 bytes) and 2-3 (its second)
    auto load_v_half = [&](int blk, int hf, bf16x8 (&dst)[GR_RB][2]) {
        const int row0 = row_begin + blk * GR_BLOCK_ROWS;
#pragma unroll
        for (int rb = 0; rb < GR_RB; ++rb) {
            const uint32_t voff = (uint32_t)min(row0 + rb * 16 + l16, n - 1) * row_bytes + (uint32_t)(kc * 16 + hf * 128);
#pragma unroll
            for (int s = 0; s < 2; ++s)
                dst[rb][s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(vrsrc, voff + s * 64, 0, 0));
        }
    };
    // Registers: the first halves of two blocks (the current one and the wave's next, requested a block ahead) and
    // the second half of the current block only, requested when the block starts: the block-lower-triangular
    // Gram matrix needs k-chunks 2-3 from its fifth 16-row slab on, 48 MFMAs into the block.
    bf16x8 va[2][GR_RB][2], vb[GR_RB][2];
    if (wave < nblk) load_v_half(wave, 0, va[0]);
    __syncthreads(); // the Gram matrices have landed (every wave waits for its own loads first)
    if (wave >= nblk) return; // after the only barrier

    // The 16 rows u of G that one MFMA takes as its A operand are chosen so that the product's epilogue factor
    // v[i][u] is already in the lane's registers: accumulator value j of lane (i, kc) belongs to A row
    // m = 4 * kc + j, and that row is u(m) = 32 * sp + 8 * (m / 4) + 4 * half + m % 4 = 32 * sp + 8 * kc + 4 * half + j,
    // i.e. element 4 * half + j of the lane's own V fragment of k-chunk sp.  (sp, half) = (ub / 2, ub % 2) covers all rows.
    const int a_row = 8 * (l16 >> 2) + (l16 & 3);          // + 32 * sp + 4 * half
    const int a_f = 4 * (l16 >> 2) + (l16 & 3);            // f(u) of that row: bits 3-4 and 0-1 of u
    float *out = vnorm + ((size_t)bi * H + h) * (size_t)n;

    // One block of rows from register set CUR; the other set receives the wave's next block meanwhile.
    auto block_step = [&](auto cur_c, int blk) {
        constexpr int CUR = decltype(cur_c)::value;
        load_v_half(blk, 1, vb);
        load_v_half(blk + GR_WAVES, 0, va[CUR ^ 1]); // unconditional (clamped rows): the wait counts stay exact
        // the block's fragments serve every head of the workgroup, one after the other
#pragma unroll 1
        for (int hh = 0; hh < GR_HEADS; ++hh) {
        const char *gl = lds + hh * 2 * GL_G_BYTES;
        float nsq[GR_RB];
#pragma unroll
        for (int rb = 0; rb < GR_RB; ++rb) nsq[rb] = 0.f;
        // fragments of 16 rows of G_hi (0-3) and G_lo (4-7) for one ub; the next ub's are requested into the same
        // registers as soon as this ub's MFMAs are issued and arrive under its epilogue and the other wave's work
        bf16x8 gf[8];
        auto read_g = [&](int ub) {
            const char *rowp = gl + (32 * (ub >> 1) + 4 * (ub & 1) + a_row) * 256;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (s > (ub >> 1)) continue; // (rows of block sp meet the k-chunks s <= sp only)
                const int slot = ((4 * s + kc) ^ a_f) * 16;
                gf[s] = *reinterpret_cast<const bf16x8 *>(rowp + slot);
                gf[4 + s] = *reinterpret_cast<const bf16x8 *>(rowp + GL_G_BYTES + slot);
            }
        };
        read_g(0);
#pragma unroll
        for (int ub = 0; ub < GL_DH / 16; ++ub) {
            const int sp = ub >> 1, half = ub & 1;
            f32x4 acc[GR_RB];
#pragma unroll
            for (int rb = 0; rb < GR_RB; ++rb) acc[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s <= sp; ++s) {
#pragma unroll
                for (int rb = 0; rb < GR_RB; ++rb)
                    acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gf[4 + s], s < 2 ? va[CUR][rb][s] : vb[rb][s - 2], acc[rb], 0, 0, 0);
#pragma unroll
                for (int rb = 0; rb < GR_RB; ++rb)
                    acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gf[s], s < 2 ? va[CUR][rb][s] : vb[rb][s - 2], acc[rb], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (ub + 1 < GL_DH / 16) read_g(ub + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int rb = 0; rb < GR_RB; ++rb) {
                const u32x4 w = __builtin_bit_cast(u32x4, sp < 2 ? va[CUR][rb][sp] : vb[rb][sp - 2]);
                const uint32_t w0 = w[2 * half], w1 = w[2 * half + 1];
                nsq[rb] = fmaf(acc[rb][0], __uint_as_float(w0 << 16), nsq[rb]);
                nsq[rb] = fmaf(acc[rb][1], __uint_as_float(w0 & 0xFFFF0000u), nsq[rb]);
                nsq[rb] = fmaf(acc[rb][2], __uint_as_float(w1 << 16), nsq[rb]);
                nsq[rb] = fmaf(acc[rb][3], __uint_as_float(w1 & 0xFFFF0000u), nsq[rb]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        const int row0 = row_begin + blk * GR_BLOCK_ROWS;
#pragma unroll
        for (int rb = 0; rb < GR_RB; ++rb) {
            float x = nsq[rb];
            x += __shfl_xor(x, 16);
            x += __shfl_xor(x, 32);
            const int row = row0 + rb * 16 + l16;
            if (kc == 0 && row < row_end) out[(size_t)hh * n + row] = sqrtf(fmaxf(x, 0.f));
        }
        }
    };
    for (int blk = wave; blk < nblk; blk += 2 * GR_WAVES) {
        block_step(std::integral_constant<int, 0>{}, blk);
        if (blk + GR_WAVES < nblk) block_step(std::integral_constant<int, 1>{}, blk + GR_WAVES);
    }
}

// The same for two heads per workgroup and long ranges (GR_LONG_BLOCKS blocks per wave and more).  In the kernel above a
// wave runs matrix and vector work in turns, waits for half of a block's V rows at its start, and the older of a SIMD's two
// waves, which is served first, ends early.  Here
//   * a slab's epilogue runs under the next slab's MFMAs (two accumulator sets), and each Gram fragment's registers are
//     refilled as soon as its MFMAs are issued
//   * the longest slabs come first, both heads inside: a block's last k-chunk of V is needed by the first slabs only, so its
//     registers take the next block's half a block ahead, the other three are held twice
//   * the blocks of a range go to the workgroup's waves as they ask
// Score call at 32 heads over 8, us, the kernel above / equal shares / this: 131072 tokens 267 / 259 / 257, 4 x 20011 182 / 177 /
// 174; MFMA busy 60 -> 72 % of a CU's cycles.  The code of a block is a straight line over both heads (10 KiB, twice), which a
// wave with one or two blocks only fetches: 8192 tokens 35.5 / 36.2, 30011 (3.75 blocks per wave) 78.0 / 77.5; one head per
// workgroup (five heads per group, 131072 tokens): 464 / 466.
__global__ __launch_bounds__(512, 1) void vproj_l2_long_kernel(const bf16_t *__restrict__ v, const bf16_t *__restrict__ gram,
                                                               float *__restrict__ vnorm, int H, int G, int n, int64_t vs0,
                                                               int64_t vs1, int64_t vs2, int pairs, int ranges, int rows_per_range)
{
    constexpr int GR_HEADS = 2, GR_WAVES = 8;
    __shared__ __attribute__((aligned(1024))) char lds[GR_HEADS * 2 * GL_G_BYTES]; // per head: G_hi | G_lo, XOR-swizzled
    __shared__ int next_block;
    const int Hkv = H / G, hgroups = G / GR_HEADS; // (G is even)
    // (work items, the Gram matrices' place in LDS and the choice of an MFMA's 16 rows of G as in the kernel above)
    const int items = pairs * ranges, per_xcd = (items + 7) >> 3;
    const int hl = ((int)blockIdx.x >> 3) % hgroups * GR_HEADS; // first head of this workgroup inside its kv group
    const int k_in_xcd = ((int)blockIdx.x >> 3) / hgroups, item = ((int)blockIdx.x & 7) * per_xcd + k_in_xcd;
    if (k_in_xcd >= per_xcd || item >= items) return; // uniform over the workgroup
    const int range = item % ranges, pair = item / ranges;
    const int bi = pair / Hkv, g = pair % Hkv, h = g * G + hl;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kc = lane >> 4;
    const int row_begin = range * rows_per_range;            // a multiple of GR_BLOCK_ROWS
    const int row_end = min(n, row_begin + rows_per_range);
    if (row_begin >= row_end) return;                        // uniform over the workgroup
    const int nblk = (row_end - row_begin + GR_BLOCK_ROWS - 1) / GR_BLOCK_ROWS;
    const bf16_t *vbase = v + bi * vs0 + g * vs1;

    for (int hh = 0; hh < GR_HEADS; ++hh) {
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(gram + (size_t)(h + hh) * 2 * GL_DH * GL_DH), 0, 2 * GL_G_BYTES, 0x00020000);
#pragma unroll
        for (int j = 0; j < 64 / GR_WAVES; ++j) {
            const int kib = j * GR_WAVES + wave;
            const int urow = (kib * 4 + (lane >> 4)) & (GL_DH - 1);
            const int f = ((urow >> 3) & 3) * 4 + (urow & 3);
            const uint32_t voff = (uint32_t)(kib * 1024 + (lane >> 4) * 256 + (((lane & 15) ^ f) * 16));
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, LDS_PTR(lds + hh * 2 * GL_G_BYTES + kib * 1024), 16, voff, 0, 0, 0);
        }
    }
    const __amdgpu_buffer_rsrc_t vrsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)vbase, 0, (int)(((int64_t)(n - 1) * vs2 + GL_DH) * 2), 0x00020000);
    const uint32_t row_bytes = (uint32_t)(vs2 * 2);
    // 64 bytes of each row of a block (k-chunk s) as B fragments
    auto load_v = [&](int blk, int s, bf16x8 (&dst)[GR_RB]) {
        const int row0 = row_begin + blk * GR_BLOCK_ROWS;
#pragma unroll
        for (int rb = 0; rb < GR_RB; ++rb) {
            const uint32_t voff = (uint32_t)min(row0 + rb * 16 + l16, n - 1) * row_bytes + (uint32_t)(kc * 16);
            dst[rb] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(vrsrc, voff + s * 64, 0, 0));
        }
    };
    bf16x8 va[2][GR_AHEAD][GR_RB], vb[GR_RB];
    if (wave < nblk) {
#pragma unroll
        for (int s = 0; s < GR_AHEAD; ++s) load_v(wave, s, va[0][s]);
        load_v(wave, GR_AHEAD, vb);
    }
    if (threadIdx.x == 0) next_block = 2 * GR_WAVES;
    __syncthreads(); // the Gram matrices have landed (every wave waits for its own loads first)
    if (wave >= nblk) return; // after the only barrier

    const int a_row = 8 * (l16 >> 2) + (l16 & 3);          // + 32 * sp + 4 * half
    const int a_f = 4 * (l16 >> 2) + (l16 & 3);            // f(u) of that row: bits 3-4 and 0-1 of u
    float *out = vnorm + ((size_t)bi * H + h) * (size_t)n;

    // A unit of work is 16 rows of one head's G (a slab): 2 * (sp + 1) fragments of four MFMAs each.  The units of a block run
    // from the longest slabs to the shortest, the heads inside, so that a V chunk's last use comes early.
    constexpr int UNITS = 8 * GR_HEADS;
    auto unit_sp = [](int u) { return 3 - u / (2 * GR_HEADS); };
    auto unit_half = [](int u) { return u / GR_HEADS % 2; };
    auto unit_head = [](int u) { return u % GR_HEADS; };
    bf16x8 gf[4][2]; // fragments of k-chunk s: G_lo, G_hi
    int ga[4]; // LDS offset of this lane's row at chunk s, slab 0 of the first head
#pragma unroll
    for (int s = 0; s < 4; ++s) ga[s] = a_row * 256 + ((4 * s + kc) ^ a_f) * 16;
    auto read_g = [&](int u, int s, int p) {
        gf[s][p] = *reinterpret_cast<const bf16x8 *>(lds + ga[s] + unit_head(u) * 2 * GL_G_BYTES + (1 - p) * GL_G_BYTES +
                                                      (32 * unit_sp(u) + 4 * unit_half(u)) * 256);
    };
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int p = 0; p < 2; ++p) read_g(0, s, p);

    // One block of rows from register set CUR; the other set receives the wave's next block meanwhile.
    auto block_step = [&](auto cur_c, int blk, int nxt) __attribute__((always_inline)) {
        constexpr int CUR = decltype(cur_c)::value;
        // (opaque, or the compiler lifts the reads of what never changes out of the loop and spills them)
#pragma unroll
        for (int s = 0; s < 4; ++s) asm volatile("" : "+v"(ga[s]));
        auto chunk = [&](int s, int rb) -> bf16x8 & { return s < GR_AHEAD ? va[CUR][s][rb] : vb[rb]; };
#pragma unroll
        for (int s = 0; s < GR_AHEAD; ++s) load_v(nxt, s, va[CUR ^ 1][s]); // unconditional (clamped rows)
        float nsq[GR_HEADS][GR_RB];
#pragma unroll
        for (int hh = 0; hh < GR_HEADS; ++hh)
#pragma unroll
            for (int rb = 0; rb < GR_RB; ++rb) nsq[hh][rb] = 0.f;
        f32x4 acc[2][GR_RB];
        // one of the 16 products of a finished unit's epilogue: N^2 += Y[u] v[u]
        auto epilogue = [&](int u, int item) __attribute__((always_inline)) {
            const int rb = item % GR_RB, j = item / GR_RB;
            const uint32_t w = __builtin_bit_cast(u32x4, chunk(unit_sp(u), rb))[2 * unit_half(u) + (j >> 1)];
            float &to = nsq[unit_head(u)][rb];
            to = fmaf(acc[u & 1][rb][j], __uint_as_float(j & 1 ? w & 0xFFFF0000u : w << 16), to);
        };
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            const int sp = unit_sp(u), next = (u + 1) % UNITS, sp_next = unit_sp(next), groups = 2 * (sp + 1);
#pragma unroll
            for (int s = 0; s <= sp; ++s)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const int g = 2 * s + p;
#pragma unroll
                    for (int rb = 0; rb < GR_RB; ++rb)
                        acc[u & 1][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gf[s][p], chunk(s, rb), g == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[u & 1][rb], 0, 0, 0);
                    // the fragment's slot takes the next unit's; the block's last unit also fetches those that it has no use for
                    if (s <= sp_next) read_g(next, s, p);
                    if (sp < sp_next) {
#pragma unroll
                        for (int x = 1 + s; x < 4; x += sp + 1) read_g(next, x, p);
                    }
                    // the unit before: its epilogue under these MFMAs
                    if (u > 0) {
#pragma unroll
                        for (int i = g * 4 * GR_RB / groups; i < (g + 1) * 4 * GR_RB / groups; ++i) epilogue(u - 1, i);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            if (u == 2 * GR_HEADS) load_v(nxt, GR_AHEAD, vb); // (the slabs that meet chunk 3 are through)
        }
#pragma unroll
        for (int i = 0; i < 4 * GR_RB; ++i) epilogue(UNITS - 1, i);
        // (pinned here: the epilogues of a row block would otherwise sink behind the branch around the store before its own,
        // and their accumulators would have to be kept until then)
#pragma unroll
        for (int hh = 0; hh < GR_HEADS; ++hh)
#pragma unroll
            for (int rb = 0; rb < GR_RB; ++rb) asm volatile("" : "+v"(nsq[hh][rb]));
        const int row0 = row_begin + blk * GR_BLOCK_ROWS;
#pragma unroll
        for (int hh = 0; hh < GR_HEADS; ++hh)
#pragma unroll
            for (int rb = 0; rb < GR_RB; ++rb) {
                float x = nsq[hh][rb];
                x += __shfl_xor(x, 16);
                x += __shfl_xor(x, 32);
                const int row = row0 + rb * 16 + l16;
                if (kc == 0 && row < row_end) out[(size_t)hh * n + row] = sqrtf(fmaxf(x, 0.f));
            }
    };
    // A wave's first two blocks are its own, the others go to whoever asks next: of the two waves of a SIMD the older one is
    // served first, and with equal shares the other would run the last sixth of its blocks alone.
    auto take = [&]() __attribute__((always_inline)) {
        int t = 0;
        if (lane == 0) t = atomicAdd(&next_block, 1);
        return t;
    };
    int blk = wave, nxt = wave + GR_WAVES;
    while (blk < nblk) {
        int t = take();
        block_step(std::integral_constant<int, 0>{}, blk, nxt);
        blk = nxt;
        nxt = __builtin_amdgcn_readfirstlane(t);
        if (blk >= nblk) break;
        t = take();
        block_step(std::integral_constant<int, 1>{}, blk, nxt);
        blk = nxt;
        nxt = __builtin_amdgcn_readfirstlane(t);
    }
}

bool vproj_l2_mfma_supported(const Dims &d)
{
    // (the V rows of one kv head are addressed through a buffer descriptor with 32-bit byte offsets)
    return d.dh == GL_DH && d.dm % 512 == 0 &&
           (((int64_t)(d.n - 1) * d.vs[2] + GL_DH) * 2) < ((int64_t)1 << 31);
}

size_t vproj_l2_gram_bytes(const Dims &d) { return (size_t)d.H * 2 * GL_DH * GL_DH * 2; }

// partial sums of the Gram slices, followed by room for the Gram matrices themselves
size_t vproj_l2_workspace_bytes(const Dims &d)
{
    return (size_t)d.H * GL_SLICES * GL_DH * GL_DH * 4 + vproj_l2_gram_bytes(d);
}

hipError_t launch_gram(const Dims &d, const void *w_o, void *gram_out, void *partial_scratch, hipStream_t s)
{
    float *partial = (float *)partial_scratch;
    hipLaunchKernelGGL(gram_partial_kernel, dim3(d.H, GL_SLICES, 2), dim3(64 * GP_WAVES), 0, s, (const bf16_t *)w_o, partial, d.dm);
    hipLaunchKernelGGL(gram_finish_kernel, dim3(GL_DH * GL_DH / 256, d.H), dim3(256), 0, s, partial, (bf16_t *)gram_out);
    return hipGetLastError();
}

hipError_t launch_vproj_l2_mfma(const Dims &d, const void *v, const void *gram, float *vnorm, hipStream_t s)
{
    // heads per workgroup: two where the group's heads pair up, else one
    const int heads = d.G % 2 == 0 ? 2 : 1, waves = 4 * heads;
    // ranges of rows per workgroup of heads: eight waves per CU over the whole launch where the context allows it,
    // so that every workgroup is resident from the start (a kv group's workgroups then walk the same rows side by side)
    const int pairs = d.batch * d.Hkv;
    // (dealing whole kv heads to the XCDs used four of the eight with 4 kv heads: 28 query heads, 32768 tokens 75 us, now 42)
    const int per_range = pairs * (d.G / heads);
    int ranges = (512 / heads) / per_range;
    const int most = (d.n + waves * GR_BLOCK_ROWS - 1) / (waves * GR_BLOCK_ROWS); // a block per wave at least
    ranges = ranges > most ? most : ranges;
    ranges = ranges < 1 ? 1 : ranges;
    int rows_per_range = (d.n + ranges - 1) / ranges;
    rows_per_range = (rows_per_range + GR_BLOCK_ROWS - 1) / GR_BLOCK_ROWS * GR_BLOCK_ROWS;
    const dim3 grid((unsigned)(8 * ((pairs * ranges + 7) / 8) * (d.G / heads))), block(waves * 64);
    if (heads == 2 && rows_per_range >= GR_LONG_BLOCKS * waves * GR_BLOCK_ROWS)
        hipLaunchKernelGGL(vproj_l2_long_kernel, grid, block, 0, s, (const bf16_t *)v, (const bf16_t *)gram, vnorm, d.H, d.G,
                           d.n, d.vs[0], d.vs[1], d.vs[2], pairs, ranges, rows_per_range);
    else if (heads == 2)
        hipLaunchKernelGGL(vproj_l2_resident_kernel<2>, grid, block, 0, s, (const bf16_t *)v, (const bf16_t *)gram, vnorm,
                           d.H, d.G, d.n, d.vs[0], d.vs[1], d.vs[2], pairs, ranges, rows_per_range);
    else
        hipLaunchKernelGGL(vproj_l2_resident_kernel<1>, grid, block, 0, s, (const bf16_t *)v, (const bf16_t *)gram, vnorm,
                           d.H, d.G, d.n, d.vs[0], d.vs[1], d.vs[2], pairs, ranges, rows_per_range);
    return hipGetLastError();
}

} // namespace ckv
