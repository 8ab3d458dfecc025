// Per-entry L1 (or L2) magnitude of the projected value for fp32 layers, on the bf16 matrix cores
// (Theorem 3.3; Algorithm 1, lines 2-3):  N^h_i = sum_c | sum_t V^g[i,t] * W_O^h[t,c] |.
//
// An fp32 number (of magnitude 2^-60 to 2^60, or zero) is the sum of three bf16 numbers (3 x 8 significant bits):
//   x = x0 + x1 + x2,  x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1), both differences exact.
// With round-to-nearest |x1| <= 2^-9 |x0| and |x2| <= 2^-18 |x0|, so of the nine products of v * w the three that are
// left out (v1 w2, v2 w1, v2 w2) are below 2^-26 of it, under half an ulp of the fp32 product; the six others are exact
// in the MFMA's fp32 accumulators and are added smallest first.  Nothing is held in 16 bits that was held in 32: the
// three parts together are the number.
//
//   split     W_O once per call into [head][d_model][3 parts][d_h] (and from the canonical layout to output-major)
//   project   the tiling of the bf16 kernel: a wave keeps RB blocks of 16 token rows (all three parts) as MFMA
//             fragments, the head's parts stream through LDS in tiles of 32 columns (24 KiB at d_h 128, double
//             buffered, direct buffer->LDS loads, 16-byte chunks swizzled), six MFMAs per (k-step, row block), the
//             previous column block's |acc| drained under them.  Rows that meet an entry outside that range are computed
//             again from the fp32 operands (exact_rows), so that they get what fp32 products give.
//
// What bounds it: the matrix cores; six bf16 MFMAs per fp32 product still leave 2.7 times the rate of the fp32 MFMA
// (157 TFLOP/s nominal).  Measured at 16 query heads over 4 kv heads, d_h 128, d_model 2048, 8192 tokens: the score call
// 2.57 ms with the vector kernel (27 TFLOP/s), 0.293 ms with this one; 4 heads, d_h 64, d_model 256, 1024 tokens: 119 and
// 21 us.  One product may be off by 9.8e-8 of itself (an fp32 fma: 6.0e-8; rms 2.60e-8 and 2.53e-8), but the sums run in
// 16 accumulators instead of one: the magnitudes' error against 64 bits (2-norm) is 5.7e-8 where the vector kernel has
// 6.7e-7 (d_model 2048), and 4.2e-8 where it has 2.4e-7 (d_model 256).
#include <type_traits>

#include "common.hpp"

namespace ckv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int VS_THREADS = 256;
constexpr int VS_WAVES = 4;
constexpr int VS_TN = 32;   // output columns per LDS tile (every supported d_model is a multiple)
constexpr int VS_PARTS = 3;

#define LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

// The three bf16 parts of x.  They are x itself, and every product of two parts is exact, for zero and for magnitudes from
// 2^-60 up to 2^60: no part and no product lies below fp32's smallest subnormal (below 2^-110 the third part would fall
// under bf16's), no sum of products overflows.  Any other x (infinity and NaN among them) becomes a NaN, and the project
// kernel computes the rows that come out as NaN again, in fp32.  Random values of order one or 1e-2 are never that small.
__device__ __forceinline__ void split3(float x, uint32_t &p0, uint32_t &p1, uint32_t &p2)
{
    const uint32_t u = __float_as_uint(x);
    const bool has_parts = ((u >> 23) & 0xFFu) - (127u - 60u) < 120u || (u << 1) == 0u;
    p0 = has_parts ? (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16 : 0x7FC0u;
    const float r = x - __uint_as_float(p0 << 16);
    const uint32_t ur = __float_as_uint(r);
    p1 = (ur + 0x7FFFu + ((ur >> 16) & 1u)) >> 16;
    const float r2 = r - __uint_as_float(p1 << 16);
    p2 = __float_as_uint(r2) >> 16; // at most 8 significant bits are left: exact
}

// Eight consecutive values as three fragments.
__device__ __forceinline__ void split8(const float4 &a, const float4 &b, bf16x8 (&f)[VS_PARTS])
{
    const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t w[VS_PARTS][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t lo[VS_PARTS], hi[VS_PARTS];
        split3(x[2 * e], lo[0], lo[1], lo[2]);
        split3(x[2 * e + 1], hi[0], hi[1], hi[2]);
#pragma unroll
        for (int p = 0; p < VS_PARTS; ++p) w[p][e] = lo[p] | (hi[p] << 16);
    }
#pragma unroll
    for (int p = 0; p < VS_PARTS; ++p) f[p] = __builtin_bit_cast(bf16x8, make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]));
}

// ---- split of W_O -----------------------------------------------------------------------------------
// Output-major source [d_model][H * d_h]: a thread takes 8 neighbouring values of one output column.
__global__ __launch_bounds__(256) void split_wo_kernel(const float *__restrict__ w, bf16_t *__restrict__ out, int H, int dh,
                                                       int dm)
{
    const int per_col = H * dh / 8;
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= (size_t)dm * per_col) return;
    const int c = (int)(t / per_col), e = (int)(t % per_col) * 8, h = e / dh, d = e % dh;
    const float4 *src = reinterpret_cast<const float4 *>(w + (size_t)c * H * dh + e);
    bf16x8 f[VS_PARTS];
    split8(src[0], src[1], f);
    bf16_t *dst = out + ((size_t)h * dm + c) * VS_PARTS * dh + d;
#pragma unroll
    for (int p = 0; p < VS_PARTS; ++p) *reinterpret_cast<bf16x8 *>(dst + (size_t)p * dh) = f[p];
}

// Canonical source [H * d_h][d_model]: a 64 x 32 block (d_h by columns) is turned in LDS on the way.
__global__ __launch_bounds__(256) void split_wo_turn_kernel(const float *__restrict__ w, bf16_t *__restrict__ out, int dh,
                                                            int dm)
{
    __shared__ float tile[64][33];
    const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 64; // d_model is a multiple of 32, H * d_h one of 64
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
    for (int j = 0; j < 8; ++j) tile[ty + 8 * j][tx] = w[(size_t)(r0 + ty + 8 * j) * dm + c0 + tx];
    __syncthreads();
    const int c = threadIdx.x >> 3, e = (threadIdx.x & 7) * 8;
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = tile[e + j][c];
    bf16x8 f[VS_PARTS];
    split8(make_float4(x[0], x[1], x[2], x[3]), make_float4(x[4], x[5], x[6], x[7]), f);
    const int h = r0 / dh, d = r0 % dh + e;
    bf16_t *dst = out + ((size_t)h * dm + c0 + c) * VS_PARTS * dh + d;
#pragma unroll
    for (int p = 0; p < VS_PARTS; ++p) *reinterpret_cast<bf16x8 *>(dst + (size_t)p * dh) = f[p];
}

// ---- projection -------------------------------------------------------------------------------------
template <int DH>
struct SGeo {
    static constexpr int KS = DH / 32;                     // k-steps of one 16x16x32 MFMA chain
    static constexpr int ROW_BYTES = DH * 2;               // one part of one column: 16 or 8 chunks of 16 bytes
    static constexpr int CPR = ROW_BYTES / 16;
    static constexpr int COL_BYTES = VS_PARTS * ROW_BYTES; // the three parts of a column are neighbours
    static constexpr int TILE_BYTES = VS_TN * COL_BYTES;   // 24 or 12 KiB
    static constexpr int LOADS = TILE_BYTES / 1024 / VS_WAVES; // direct loads per wave per tile
    // chunk q of a row of column c sits at slot q ^ swz(c): the 16 columns of a fragment read then fall on
    // different banks (d_h 64: two columns share the 256 bytes of a bank row, so neighbours take the same key)
    __host__ __device__ static constexpr int swz(int c) { return DH == 128 ? (c & 15) : ((c >> 1) & 7); }
};

template <bool L2> __device__ __forceinline__ void drain(float &to, float x) { to = L2 ? fmaf(x, x, to) : to + fabsf(x); }

// The magnitudes of VS_EXACT neighbouring rows from the fp32 operands themselves, by one wave: a lane takes every 64th
// column, one fma chain over d_h per row.  For rows with an operand that has no three parts: rare, so all that is asked of
// it is the rate of the vector kernel.  The score call at 16 heads over 4 kv heads, d_model 2048, 8192 tokens: 2.55 ms with
// the vector kernel; 0.30 here, 0.44 - 0.51 with one such row, 2.05 with one in every row.
constexpr int VS_EXACT = 8;
template <int DH, bool L2, bool OUT_IN>
__device__ __forceinline__ void exact_rows(const float *vbase, int64_t vs2, int row, int n, const float *w, int64_t ldw, int dm,
                                           float (&out)[VS_EXACT])
{
    const int lane = threadIdx.x & 63;
    const float *v[VS_EXACT];
#pragma unroll
    for (int j = 0; j < VS_EXACT; ++j) {
        v[j] = vbase + (int64_t)min(row + j, n - 1) * vs2;
        out[j] = 0.f;
    }
    for (int c = lane; c < dm; c += 64) { // (d_model is a multiple of 32: half of the lanes may skip the last round)
        float p[VS_EXACT];
#pragma unroll
        for (int j = 0; j < VS_EXACT; ++j) p[j] = 0.f;
#pragma unroll 2
        for (int t = 0; t < DH; t += 4) {
            float x[4];
            if (OUT_IN) { // [d_model][H * d_h]: this lane's column is contiguous
                const float4 four = *reinterpret_cast<const float4 *>(w + c * ldw + t);
                x[0] = four.x; x[1] = four.y; x[2] = four.z; x[3] = four.w;
            } else {      // [H * d_h][d_model]: the lanes' columns are
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = w[(t + e) * ldw + c];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < VS_EXACT; ++j) p[j] = fmaf(v[j][t + e], x[e], p[j]);
        }
#pragma unroll
        for (int j = 0; j < VS_EXACT; ++j) drain<L2>(out[j], p[j]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int j = 0; j < VS_EXACT; ++j) out[j] += __shfl_xor(out[j], o);
}

template <int DH, int RB, bool L2>
__global__ __launch_bounds__(VS_THREADS, 2) void vproj_split_kernel(const float *__restrict__ v, const float *__restrict__ w_o,
                                                                    int out_in, const bf16_t *__restrict__ w3,
                                                                    float *__restrict__ vnorm, int H, int G, int n, int dm,
                                                                    int64_t vs0, int64_t vs1, int64_t vs2, int row_tiles,
                                                                    int heads)
{
    using geo = SGeo<DH>;
    constexpr int KS = geo::KS, CB = VS_TN / 16;
    __shared__ __attribute__((aligned(1024))) char lds[2 * geo::TILE_BYTES];
    // workgroup L runs on XCD L % 8; an XCD takes an eighth of the (head, row tile) pairs in head order, so that the
    // workgroups resident on it stream the same head's parts out of its L2, whatever the number of heads
    const int total = heads * row_tiles, per_xcd = (total + 7) >> 3;
    const int k_in_xcd = blockIdx.x >> 3, item = (blockIdx.x & 7) * per_xcd + k_in_xcd;
    if (k_in_xcd >= per_xcd || item >= total) return;                 // uniform over the workgroup
    const int hb = item / row_tiles, tile_x = item % row_tiles;       // batch * H + head
    const int h = hb % H, bi = hb / H, g = h / G;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kc = lane >> 4;
    const int row0 = (tile_x * VS_WAVES + wave) * (RB * 16);

    // one head's parts: d_model * COL_BYTES (the host checks that this stays below 2 GiB)
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(w3 + (size_t)h * dm * VS_PARTS * DH), 0, dm * geo::COL_BYTES, 0x00020000);
    // load j of this wave fills KiB m = j * 4 + wave of the tile; a lane's 16 bytes belong to column col, part row p
    auto issue_load = [&](int tile, int j, char *buf) {
        const int kib = j * VS_WAVES + wave;
        const int byte = kib * 1024 + lane * 16;             // where this lane's chunk lands in the tile
        const int row = byte / geo::ROW_BYTES, slot = (byte % geo::ROW_BYTES) / 16;
        const int col = row / VS_PARTS;
        const uint32_t voff = (uint32_t)(row * geo::ROW_BYTES + ((slot ^ geo::swz(col)) * 16));
        const uint32_t soff = (uint32_t)tile * geo::TILE_BYTES;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, LDS_PTR(buf + kib * 1024), 16, voff, soff, 0, 0);
    };
#pragma unroll
    for (int j = 0; j < geo::LOADS; ++j) issue_load(0, j, lds);

    // the three parts of the wave's token rows (16 rows x 32 k per fragment), resident in registers
    bf16x8 a[RB][KS][VS_PARTS];
    const float *vbase = v + bi * vs0 + g * vs1;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = min(row0 + rb * 16 + l16, n - 1);
        const float *p = vbase + (int64_t)row * vs2 + kc * 8;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const float4 x = *reinterpret_cast<const float4 *>(p + s * 32), y = *reinterpret_cast<const float4 *>(p + s * 32 + 4);
            split8(x, y, a[rb][s]);
        }
    }
    float sum[RB][4];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < 4; ++j) sum[rb][j] = 0.f;
    f32x4 acc[2][RB];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[p][rb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // byte offsets of the fragments of part 0 inside a 16-column block; part p lies ROW_BYTES * p behind
    int boff[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) boff[s] = l16 * geo::COL_BYTES + (((4 * s + kc) ^ geo::swz(l16)) * 16);
    bf16x8 b[KS][VS_PARTS];
    auto read_b = [&](const char *block, int s, int p) {
        b[s][p] = *reinterpret_cast<const bf16x8 *>(block + boff[s] + p * geo::ROW_BYTES);
    };
    __syncthreads();
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int p = 0; p < VS_PARTS; ++p) read_b(lds, s, p);

    const int tiles = dm / VS_TN;
    auto tile_step = [&](auto buf_c, int t) {
        constexpr int BUF = decltype(buf_c)::value;
        const char *cur = lds + BUF * geo::TILE_BYTES;
        char *nxt = lds + (BUF ^ 1) * geo::TILE_BYTES;
        const int tn = min(t + 1, tiles - 1); // the last iteration re-fetches its own tile into the idle buffer
#pragma unroll
        for (int j = 0; j < geo::LOADS; ++j) issue_load(tn, j, nxt);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int pp = cb & 1;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                // (part of W_O, part of V), smallest products first
                constexpr int WP[6] = {2, 1, 0, 1, 0, 0}, VP[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
                for (int q = 0; q < 6; ++q) {
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        if (s == 0 && q == 0)
                            acc[pp][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[s][WP[q]], a[rb][s][VP[q]], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                        else
                            acc[pp][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[s][WP[q]], a[rb][s][VP[q]], acc[pp][rb], 0, 0, 0);
                    }
                    // after a part's last use in this block, its slot takes the next block's fragment
                    if (cb + 1 < CB && (q == 0 || q == 3 || q == 5)) read_b(cur + (cb + 1) * 16 * geo::COL_BYTES, s, WP[q]);
                    // the previous column block's products, spread over the k-steps
                    if (q < RB) {
#pragma unroll
                        for (int e = 0; e < 4 / KS; ++e) drain<L2>(sum[q][s * (4 / KS) + e], acc[pp ^ 1][q][s * (4 / KS) + e]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int p = 0; p < VS_PARTS; ++p) read_b(nxt, s, p);
    };
    static_assert(RB <= 6, "one row block is drained per product group");
    for (int t = 0; t < tiles; t += 2) {
        tile_step(std::integral_constant<int, 0>{}, t);
        if (t + 1 < tiles) tile_step(std::integral_constant<int, 1>{}, t + 1);
    }
    float *out = vnorm + (size_t)hb * (size_t)n;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int j = 0; j < 4; ++j) drain<L2>(sum[rb][j], acc[(CB - 1) & 1][rb][j]);
        float x = (sum[rb][0] + sum[rb][1]) + (sum[rb][2] + sum[rb][3]);
        x += __shfl_xor(x, 16);
        x += __shfl_xor(x, 32);
        const int row = row0 + rb * 16 + l16;
        const bool lost = x != x; // an operand without three parts
        if (kc == 0 && row < n && !lost) out[row] = L2 ? sqrtf(x) : x;
        const uint32_t again = (uint32_t)__ballot(kc == 0 && row < n && lost); // (rows are the lanes 0 .. 15)
#pragma unroll 1
        for (int r8 = 0; r8 < 16; r8 += VS_EXACT) {
            if (!((again >> r8) & ((1u << VS_EXACT) - 1u))) continue; // uniform over the wave
            float exact[VS_EXACT];
            const int first = row0 + rb * 16 + r8;
            if (out_in) exact_rows<DH, L2, true>(vbase, vs2, first, n, w_o + h * DH, (int64_t)H * DH, dm, exact);
            else exact_rows<DH, L2, false>(vbase, vs2, first, n, w_o + (int64_t)h * DH * dm, dm, dm, exact);
#pragma unroll
            for (int j = 0; j < VS_EXACT; ++j)
                if (lane == 0 && ((again >> (r8 + j)) & 1u)) out[first + j] = L2 ? sqrtf(exact[j]) : exact[j];
        }
    }
}

template <int DH, int RB>
static void launch_project(const Dims &d, int out_in, const void *v, const void *w_o, const void *w3, float *vnorm,
                           hipStream_t s)
{
    const int rows_per_wg = VS_WAVES * RB * 16, row_tiles = (d.n + rows_per_wg - 1) / rows_per_wg;
    const int heads = d.batch * d.H;
    const dim3 grid((unsigned)(8ll * (((long long)heads * row_tiles + 7) / 8))), block(VS_THREADS);
    if (d.norm == CKV_NORM_L2)
        hipLaunchKernelGGL((vproj_split_kernel<DH, RB, true>), grid, block, 0, s, (const float *)v, (const float *)w_o, out_in,
                           (const bf16_t *)w3, vnorm, d.H, d.G, d.n, d.dm, d.vs[0], d.vs[1], d.vs[2], row_tiles, heads);
    else
        hipLaunchKernelGGL((vproj_split_kernel<DH, RB, false>), grid, block, 0, s, (const float *)v, (const float *)w_o, out_in,
                           (const bf16_t *)w3, vnorm, d.H, d.G, d.n, d.dm, d.vs[0], d.vs[1], d.vs[2], row_tiles, heads);
}

size_t vproj_split_bytes(const Dims &d) { return (size_t)d.H * d.dh * d.dm * VS_PARTS * 2; }

bool vproj_split_supported(const Dims &d)
{
    return (d.dh == 64 || d.dh == 128) && d.dm % VS_TN == 0 && (size_t)d.dm * VS_PARTS * d.dh * 2 < ((size_t)1 << 31) &&
           ((long long)d.batch * d.H + 8) * (d.n / 64 + 2) < (1ll << 31) &&
           (long long)d.dm * (d.H * (long long)d.dh / 8) < (256ll << 31) && d.H * (long long)d.dh / 64 < 65536;
}

// Row blocks per wave, by the cost of the launch's rounds: an XCD holds 64 workgroups (two per CU); a round's time was
// measured as proportional to RB + c2 with two workgroups on every CU and to 0.48 RB + c1 with one (16 heads, d_model 2048:
// c2 = 0.40, c1 = 0.38 at d_h 128, 0.50 and 0.55 at d_h 64), as for the bf16 kernel.  The stage's time there with 1 / 2 / 3
// blocks, us: n 1024 60 / 81 / 106, 4096 149 / 143 / 179, 6144 214 / 205 / 197, 16384 537 / 509 / 525.
static int pick_row_blocks(const Dims &d, const int *choices, int count)
{
    return cheapest_rounds(d, VS_WAVES * 16, d.dh == 128 ? 0.40 : 0.50, d.dh == 128 ? 0.38 : 0.55, choices, count);
}

hipError_t launch_vproj_split(const Dims &d, int out_in, const void *v, const void *w_o, void *w3, float *vnorm, hipStream_t s)
{
    if (out_in) {
        const size_t threads = (size_t)d.dm * (d.H * d.dh / 8);
        hipLaunchKernelGGL(split_wo_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, (const float *)w_o,
                           (bf16_t *)w3, d.H, d.dh, d.dm);
    } else {
        hipLaunchKernelGGL(split_wo_turn_kernel, dim3(d.dm / 32, d.H * d.dh / 64), dim3(256), 0, s, (const float *)w_o,
                           (bf16_t *)w3, d.dh, d.dm);
    }
    if (d.dh == 64) { // (six blocks spill, and five are nowhere the best)
        const int choices[] = {4, 3, 2, 1};
        switch (pick_row_blocks(d, choices, 4)) {
        case 4: launch_project<64, 4>(d, out_in, v, w_o, w3, vnorm, s); break;
        case 3: launch_project<64, 3>(d, out_in, v, w_o, w3, vnorm, s); break;
        case 2: launch_project<64, 2>(d, out_in, v, w_o, w3, vnorm, s); break;
        default: launch_project<64, 1>(d, out_in, v, w_o, w3, vnorm, s); break;
        }
    } else { // (the registers hold three)
        const int choices[] = {3, 2, 1};
        switch (pick_row_blocks(d, choices, 3)) {
        case 3: launch_project<128, 3>(d, out_in, v, w_o, w3, vnorm, s); break;
        case 2: launch_project<128, 2>(d, out_in, v, w_o, w3, vnorm, s); break;
        default: launch_project<128, 1>(d, out_in, v, w_o, w3, vnorm, s); break;
        }
    }
    return hipGetLastError();
}

} // namespace ckv
