// The bodies of the fp32 magnitudes' kernels, shared by their own launches and those that run the key sweeps beside them.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace ckv {

typedef _Float16 f16_t;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int VS_THREADS = 256;
constexpr int VS_WAVES = 4;
constexpr int VS_TN = 32;   // output columns per LDS tile (every supported d_model is a multiple)
constexpr int VS_PARTS = 2;
// A row's sum of scaled |products| over d_model is typically 2^29 per column in units of the columns' factors.  What the
// parts leave out of small entries is at most 2^-9 per product (2^-24 of 2^15, times 2^15), random in sign: below 2^-24 of a
// sum of 2^19 per column.  Rows under that are computed again; no row of which less than all but 2^-10 cancels is.
constexpr float VS_SMALL = 524288.0f;

#define LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

// The power of two that takes a largest magnitude (its bits) to [2^14, 2^15), and its inverse.  Zero needs none; for any
// other magnitude outside 2^-60 .. 2^60 (infinities and NaN too) both are NaN, and so is every result they meet.
__device__ __forceinline__ void part_scale(uint32_t largest, float &up, float &down)
{
    const uint32_t e = largest >> 23; // (the sign bit is clear)
    const bool fits = e - (127u - 60u) < 120u;
    up = __uint_as_float(fits ? (127u + 127u + 14u - e) << 23 : largest ? 0x7FC00000u : 0x3F800000u);
    down = __uint_as_float(fits ? (e - 14u) << 23 : largest ? 0x7FC00000u : 0u);
}

// Eight consecutive values, scaled, as two fragments.
__device__ __forceinline__ void split8(const float (&x)[8], float scale, f16x8 &hi, f16x8 &lo)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float y = x[e] * scale;
        hi[e] = (f16_t)y;
        lo[e] = (f16_t)(y - (float)hi[e]);
    }
}

__device__ __forceinline__ uint32_t largest8(const float (&x)[8])
{
    uint32_t m = 0u; // magnitudes compare as their bits do, and a NaN is the largest of all
#pragma unroll
    for (int e = 0; e < 8; ++e) m = max(m, __float_as_uint(x[e]) & 0x7FFFFFFFu);
    return m;
}

__device__ __forceinline__ void load_eight(const float *p, float (&x)[8])
{
    const float4 a = reinterpret_cast<const float4 *>(p)[0], b = reinterpret_cast<const float4 *>(p)[1];
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}

// ---- split of W_O -----------------------------------------------------------------------------------
// One workgroup per (tile of VS_TN columns, head); a thread takes 8 neighbouring values of one column (two of them at
// d_h 128).  OUT_IN: source [d_model][H * d_h].  Else [H * d_h][d_model], turned in LDS on the way.
template <int DH, bool OUT_IN>
__device__ __forceinline__ void split_wo_body(const float *__restrict__ w, f16_t *__restrict__ out, float *__restrict__ factor,
                                              int H, int dm, int tile_x, int h)
{
    constexpr int PER = VS_TN * DH / 8 / VS_THREADS, PIECES = DH / 8; // pieces of 8 values: per thread, per column
    __shared__ float tile[OUT_IN ? 1 : DH][VS_TN + 1];
    __shared__ uint32_t largest[VS_WAVES];
    const int c0 = tile_x * VS_TN; // d_model is a multiple of VS_TN
    float x[PER][8];
    if constexpr (!OUT_IN) {
        const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
        for (int j = 0; j < DH / 8; ++j) tile[ty + 8 * j][tx] = w[((size_t)h * DH + ty + 8 * j) * dm + c0 + tx];
        __syncthreads();
    }
    uint32_t m = 0u;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int piece = u * VS_THREADS + (int)threadIdx.x, c = piece / PIECES, e = piece % PIECES * 8;
        if constexpr (OUT_IN) {
            load_eight(w + (size_t)(c0 + c) * H * DH + h * DH + e, x[u]);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) x[u][j] = tile[e + j][c];
        }
        m = max(m, largest8(x[u]));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o));
    if ((threadIdx.x & 63) == 0) largest[threadIdx.x >> 6] = m;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < VS_WAVES; ++i) m = max(m, largest[i]);
    float up, down;
    part_scale(m, up, down);
    if (threadIdx.x == 0) factor[(size_t)h * (dm / VS_TN) + tile_x] = down;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int piece = u * VS_THREADS + (int)threadIdx.x, c = piece / PIECES, e = piece % PIECES * 8;
        f16x8 hi, lo;
        split8(x[u], up, hi, lo);
        f16_t *dst = out + ((size_t)h * dm + c0 + c) * VS_PARTS * DH + e;
        *reinterpret_cast<f16x8 *>(dst) = hi;
        *reinterpret_cast<f16x8 *>(dst + DH) = lo;
    }
}

// ---- projection -------------------------------------------------------------------------------------
template <int DH>
struct SGeo {
    static constexpr int KS = DH / 32;                     // k-steps of one 16x16x32 MFMA chain
    static constexpr int CPR = DH * 2 / 16;                // 16-byte chunks of one part of a column
    static constexpr int COL_BYTES = VS_PARTS * DH * 2;    // the parts of a column are neighbours
    static constexpr int TILE_BYTES = VS_TN * COL_BYTES;   // 16 or 8 KiB
    static constexpr int LOADS = TILE_BYTES / 1024 / VS_WAVES; // direct loads per wave per tile
    // chunk q of column c (its parts' chunks counted through) sits at slot q ^ (c % 16): the 16 columns of a fragment read
    // then fall on different banks
};

// (NaN in either operand stays)
template <bool L2> __device__ __forceinline__ void drain(float &to, float x, float factor)
{
    if (L2) {
        const float y = x * factor;
        to = fmaf(y, y, to);
    } else {
        to = fmaf(fabsf(x), factor, to);
    }
}

// The magnitudes of VS_EXACT neighbouring rows from the fp32 operands themselves, by one wave: a lane takes every 64th
// column, one fma chain over d_h per row.  For rows that the parts do not serve: rare, so all that is asked of it is the rate
// of the vector kernel.  The score call at 16 heads over 4 kv heads, d_model 2048, 8192 tokens: 2.55 ms with
// the vector kernel; 0.18 here, 0.32 with one such row, 0.39 with one in 64, 1.93 with one in every row.
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
        for (int j = 0; j < VS_EXACT; ++j) drain<L2>(out[j], p[j], 1.f);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int j = 0; j < VS_EXACT; ++j) out[j] += __shfl_xor(out[j], o);
}

struct SplitArgs {
    const float *v, *w_o;
    const f16_t *parts;
    const float *factors;
    float *vnorm;
    int out_in, H, G, n, dm;
    int64_t vs0, vs1, vs2;
    int row_tiles, heads; // heads: batch * H
};

// Workgroup wg's share, with 2 * SGeo<DH>::TILE_BYTES of LDS.
template <int DH, int RB, bool L2>
__device__ __forceinline__ void vproj_split_body(const SplitArgs &P, char *lds, int wg)
{
    using geo = SGeo<DH>;
    constexpr int KS = geo::KS, CB = VS_TN / 16;
    const float *__restrict__ v = P.v, *__restrict__ w_o = P.w_o, *__restrict__ factors = P.factors;
    const f16_t *__restrict__ parts = P.parts;
    float *__restrict__ vnorm = P.vnorm;
    const int out_in = P.out_in, H = P.H, G = P.G, n = P.n, dm = P.dm, row_tiles = P.row_tiles, heads = P.heads;
    const int64_t vs0 = P.vs0, vs1 = P.vs1, vs2 = P.vs2;
    // workgroup L runs on XCD L % 8; an XCD takes an eighth of the (head, row tile) pairs in head order, so that the
    // workgroups resident on it stream the same head's parts out of its L2, whatever the number of heads
    const int total = heads * row_tiles, per_xcd = (total + 7) >> 3;
    const int k_in_xcd = wg >> 3, item = (wg & 7) * per_xcd + k_in_xcd;
    if (k_in_xcd >= per_xcd || item >= total) return;                 // uniform over the workgroup
    const int hb = item / row_tiles, tile_x = item % row_tiles;       // batch * H + head
    const int h = hb % H, bi = hb / H, g = h / G;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kc = lane >> 4;
    const int row0 = (tile_x * VS_WAVES + wave) * (RB * 16);
    const int tiles = dm / VS_TN;

    // one head's parts: d_model * COL_BYTES (the host checks that this stays below 2 GiB), and its tiles' factors
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(parts + (size_t)h * dm * VS_PARTS * DH), 0, dm * geo::COL_BYTES, 0x00020000);
    const __amdgpu_buffer_rsrc_t f_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(factors + (size_t)h * tiles), 0, tiles * 4, 0x00020000);
    // load j of this wave fills KiB m = j * 4 + wave of the tile
    auto issue_load = [&](int tile, int j, char *buf) {
        const int kib = j * VS_WAVES + wave;
        const int byte = kib * 1024 + lane * 16;             // where this lane's chunk lands in the tile
        const int col = byte / geo::COL_BYTES, slot = byte % geo::COL_BYTES / 16;
        const uint32_t voff = (uint32_t)(col * geo::COL_BYTES + ((slot ^ (col & 15)) * 16));
        const uint32_t soff = (uint32_t)tile * geo::TILE_BYTES;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, LDS_PTR(buf + kib * 1024), 16, voff, soff, 0, 0);
    };
    // a tile's factor by a vector load (a scalar one would make every wait for an LDS read wait for it too)
    auto load_factor = [&](int tile) {
        uint32_t zero = 0u;
        asm volatile("" : "+v"(zero));
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(f_rsrc, zero, tile * 4, 0));
    };
#pragma unroll
    for (int j = 0; j < geo::LOADS; ++j) issue_load(0, j, lds);
    float fac[2]; // of the tile at work, and of the other one: the next, and before its arrival the one before
    fac[0] = load_factor(0);
    fac[1] = 0.f;

    // both parts of the wave's token rows (16 rows x 32 k per fragment), resident in registers
    f16x8 a[RB][KS][VS_PARTS];
    float undo[RB]; // what the row's scale is undone by
    const float *vbase = v + bi * vs0 + g * vs1;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = min(row0 + rb * 16 + l16, n - 1);
        const float *p = vbase + (int64_t)row * vs2 + kc * 8;
        float x[KS][8];
        uint32_t m = 0u;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            load_eight(p + s * 32, x[s]);
            m = max(m, largest8(x[s]));
        }
        m = max(m, (uint32_t)__shfl_xor((int)m, 16));
        m = max(m, (uint32_t)__shfl_xor((int)m, 32));
        float up;
        part_scale(m, up, undo[rb]);
#pragma unroll
        for (int s = 0; s < KS; ++s) split8(x[s], up, a[rb][s][0], a[rb][s][1]);
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
    float fac_sum = 0.f; // over the tiles: what a sum of one per column would come to

    // byte offsets of the fragments inside a 16-column block
    int boff[KS][VS_PARTS];
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int p = 0; p < VS_PARTS; ++p) boff[s][p] = l16 * geo::COL_BYTES + (((geo::CPR * p + 4 * s + kc) ^ l16) * 16);
    f16x8 b[KS][VS_PARTS];
    auto read_b = [&](const char *block, int s, int p) { b[s][p] = *reinterpret_cast<const f16x8 *>(block + boff[s][p]); };
    __syncthreads();
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int p = 0; p < VS_PARTS; ++p) read_b(lds, s, p);

    auto tile_step = [&](auto buf_c, int t) {
        constexpr int BUF = decltype(buf_c)::value;
        const char *cur = lds + BUF * geo::TILE_BYTES;
        char *nxt = lds + (BUF ^ 1) * geo::TILE_BYTES;
        const int tn = min(t + 1, tiles - 1); // the last iteration re-fetches its own tile into the idle buffer
#pragma unroll
        for (int j = 0; j < geo::LOADS; ++j) issue_load(tn, j, nxt);
        const float next_fac = load_factor(tn);
        fac_sum = L2 ? fmaf(fac[BUF], fac[BUF], fac_sum) : fac_sum + fac[BUF];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int pp = cb & 1;
            const float drained = cb == 0 ? fac[BUF ^ 1] : fac[BUF]; // the previous column block is the previous tile's last
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                // (part of W_O, part of V), smallest products first
                constexpr int WP[3] = {1, 0, 0}, VP[3] = {0, 1, 0};
#pragma unroll
                for (int q = 0; q < 3; ++q) {
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        if (s == 0 && q == 0)
                            acc[pp][rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b[s][WP[q]], a[rb][s][VP[q]], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                        else
                            acc[pp][rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b[s][WP[q]], a[rb][s][VP[q]], acc[pp][rb], 0, 0, 0);
                    }
                    // after a part's last use in this block, its slot takes the next block's fragment
                    if (cb + 1 < CB && q != 1) read_b(cur + (cb + 1) * 16 * geo::COL_BYTES, s, WP[q]);
                    // the previous column block's products, spread over the steps
                    constexpr int STEPS = 3 * KS;
#pragma unroll
                    for (int x = (3 * s + q) * RB * 4 / STEPS; x < (3 * s + q + 1) * RB * 4 / STEPS; ++x)
                        drain<L2>(sum[x % RB][x / RB], acc[pp ^ 1][x % RB][x / RB], drained);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        fac[BUF ^ 1] = next_fac;
        __syncthreads();
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int p = 0; p < VS_PARTS; ++p) read_b(nxt, s, p);
    };
    for (int t = 0; t < tiles; t += 2) {
        tile_step(std::integral_constant<int, 0>{}, t);
        if (t + 1 < tiles) tile_step(std::integral_constant<int, 1>{}, t + 1);
    }
    const float last_fac = (tiles & 1) ? fac[0] : fac[1];
    const float small = L2 ? VS_SMALL * VS_SMALL * VS_TN * fac_sum : VS_SMALL * VS_TN * fac_sum;
    float *out = vnorm + (size_t)hb * (size_t)n;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int j = 0; j < 4; ++j) drain<L2>(sum[rb][j], acc[(CB - 1) & 1][rb][j], last_fac);
        // the sixteen accumulators of a row merge in 64 bits: in fp32 these four additions would be most of the result's error
        double all = ((double)sum[rb][0] + (double)sum[rb][1]) + ((double)sum[rb][2] + (double)sum[rb][3]);
        all += __shfl_xor(all, 16);
        all += __shfl_xor(all, 32);
        const float x = (float)all;
        const int row = row0 + rb * 16 + l16;
        // (a row of zeros is exact as it is; a sum that overflows under its scales may not overflow without them)
        const bool lost = !(x >= small && x < INFINITY) && undo[rb] != 0.f;
        if (kc == 0 && row < n && !lost) out[row] = (L2 ? sqrtf(x) : x) * undo[rb];
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

// row blocks per wave that the launcher takes, and the arguments and workgroups that go with them; scratch holds the parts
// and behind them the tiles' factors
int vproj_split_row_blocks(const Dims &d);
SplitArgs vproj_split_args(const Dims &d, int row_blocks, int out_in, const void *v, const void *w_o, void *scratch, float *vnorm,
                           unsigned *wgs);

} // namespace ckv
