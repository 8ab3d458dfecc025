// The projection kernel's body, shared by its own launch and the one that runs the second key sweep beside it.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace ckv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int VM_THREADS = 256;
constexpr int VM_WAVES = 4;
constexpr int VM_TILE_BYTES = 32768;       // one LDS tile of W_O columns
constexpr int VM_LOADS = VM_TILE_BYTES / 1024 / VM_WAVES; // direct loads per wave per tile

template <int DH>
struct VGeo {
    static constexpr int KS = DH / 32;                 // k-steps of one 16x16x32 MFMA chain
    static constexpr int COL_BYTES = DH * 2;           // one W_O column of the head: 16 or 8 chunks of 16 B
    static constexpr int CPR = COL_BYTES / 16;         // chunks per column
    static constexpr int TN = VM_TILE_BYTES / COL_BYTES; // W_O columns per LDS tile (128 or 256)
    static constexpr int CB = TN / 16;                 // 16-column blocks per tile
    static constexpr int CPK = 1024 / COL_BYTES;       // columns per KiB (one direct load of a wave)
    static constexpr int LPC = KS / 2;                 // direct loads issued per column block (first half of a tile)
};

#define LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

struct VprojArgs {
    const bf16_t *v, *w_t;
    float *vnorm;
    int H, G, n, dm;
    int64_t vs0, vs1, vs2;
    int row_tiles, heads; // heads: batch * H
    int pair;             // heads 2p and 2p + 1 take turns on every row tile
};

constexpr int VM_LDS = 2 * VM_TILE_BYTES;

// Workgroup wg's share, with VM_LDS bytes of LDS.
template <int DH, int RB>
__device__ __forceinline__ void vproj_mfma_body(const VprojArgs &P, char *lds, int wg)
{
    using geo = VGeo<DH>;
    constexpr int VM_KS = geo::KS, VM_CB = geo::CB, VM_TN = geo::TN, VM_COL_BYTES = geo::COL_BYTES, VM_DH = DH;
    static_assert(VM_LOADS * 2 == VM_CB * geo::LPC, "the next tile's loads go out during the first half of a tile");
    const bf16_t *__restrict__ v = P.v, *__restrict__ w_t = P.w_t;
    float *__restrict__ vnorm = P.vnorm;
    const int H = P.H, G = P.G, n = P.n, dm = P.dm, row_tiles = P.row_tiles, heads = P.heads, pair = P.pair;
    const int64_t vs0 = P.vs0, vs1 = P.vs1, vs2 = P.vs2;
    // XCD-aware work mapping.  Workgroups of a 1-D grid are handed to the 8 XCDs round-robin (workgroup L
    // runs on XCD L % 8) and every XCD has its own 4 MiB L2.  An XCD gets an eighth of the (query head, row tile) items in
    // head order, i.e. consecutive heads of one kv group, and walks the heads two at a time: the two take turns on every
    // row tile, so the second one finds the tile's V rows in that L2, and the workgroups resident on the XCD stream
    // the same two 1 MiB W_O slices, which stay in L2 as well.  (Four heads in turn were measured slower: their
    // four slices evict each other.  Measured against one head at a time: same speed, half the L2 misses -- as
    // long as two slices leave room in L2: at d_model 5120 (2 x 1.25 MiB) pairing was 13 % slower, so the host
    // pairs heads only up to d_model 4096.  Dealing out whole heads left an XCD idle with 28 of them and half idle with 12:
    // 32768 tokens 592 / 140 us, now 532 / 107.)
    const int total = heads * row_tiles, per_xcd = (total + 7) >> 3;
    const int k_in_xcd = wg >> 3, item = (wg & 7) * per_xcd + k_in_xcd;
    if (k_in_xcd >= per_xcd || item >= total) return; // uniform over the workgroup
    // pair = 1: heads 2p and 2p + 1 alternate over their row tiles (a last head without a partner runs alone)
    const int first = pair ? item / (2 * row_tiles) * 2 : item / row_tiles, in_head = item - first * row_tiles;
    const bool turns = pair && first + 1 < heads;
    const int hb = first + (turns ? in_head & 1 : 0);    // batch * H + head
    const int tile_x = turns ? in_head >> 1 : in_head;
    const int h = hb % H, bi = hb / H, g = h / G;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); // wave-uniform, kept in a scalar register
    const int l16 = lane & 15, kc = lane >> 4;
    const int row0 = (tile_x * VM_WAVES + wave) * (RB * 16);

    // V fragments (16 token rows x 32 k each), resident in registers
    bf16x8 a[RB][VM_KS];
    const bf16_t *vbase = v + bi * vs0 + g * vs1;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = min(row0 + rb * 16 + l16, n - 1);
        const bf16_t *p = vbase + (int64_t)row * vs2 + kc * 8;
#pragma unroll
        for (int s = 0; s < VM_KS; ++s) a[rb][s] = *reinterpret_cast<const bf16x8 *>(p + s * 32);
    }

    float sum[RB][4];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < 4; ++j) sum[rb][j] = 0.f;

    // Direct loads: instruction j of wave w fills LDS KiB m = j * 4 + w of the tile = columns CPK*m .. (CPK = 4 at
    // d_h 128); lane i writes slot i % CPR of column CPK*m + i / CPR and therefore fetches chunk
    // (i % CPR) ^ (column & (CPR-1)).
    // They are buffer loads (not flat/global ones): the compiler then keeps exact LDS wait counts.
    const size_t ldw = (size_t)H * VM_DH; // elements between consecutive output columns
    const int ld_col = wave * geo::CPK + lane / geo::CPR;                // column of this lane for j = 0
    const uint32_t ld_voff = (uint32_t)(((size_t)h * VM_DH + (size_t)ld_col * ldw +
                                         (size_t)(((lane % geo::CPR) ^ (ld_col & (geo::CPR - 1))) * 8)) * 2);
    // (columns advance by 4 * CPK per instruction, a multiple of CPR, which leaves the chunk unchanged)
    const int tiles = dm / VM_TN; // host guarantees dm % VM_TN == 0 and the whole matrix < 2 GiB
    const __amdgpu_buffer_rsrc_t w_rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void *)w_t, 0, (int)((size_t)dm * ldw * 2), 0x00020000);

    auto issue_load = [&](int tile, int j, char *buf) {
        const uint32_t soff = (uint32_t)(((size_t)tile * VM_TN + (size_t)j * 4 * geo::CPK) * ldw * 2);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, LDS_PTR(buf + (j * 4 + wave) * 1024), 16, ld_voff, soff, 0, 0);
    };

#pragma unroll
    for (int j = 0; j < VM_LOADS; ++j) issue_load(0, j, lds);

    // per-lane byte offsets of the 4 W_O fragments inside a 16-column block
    int boff[VM_KS];
#pragma unroll
    for (int s = 0; s < VM_KS; ++s) boff[s] = l16 * VM_COL_BYTES + (((4 * s + kc) ^ (l16 & (geo::CPR - 1))) * 16);

    f32x4 acc[2][RB];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[p][rb] = f32x4{0.f, 0.f, 0.f, 0.f};

    __syncthreads();
    bf16x8 b[VM_KS];
#pragma unroll
    for (int s = 0; s < VM_KS; ++s) b[s] = *reinterpret_cast<const bf16x8 *>(lds + boff[s]);

    // One tile.  BUF (which LDS buffer holds it) is a compile-time constant so that every fragment
    // read is "per-lane offset register + immediate": the tile loop below is unrolled by two.
    auto tile_step = [&](auto buf_c, int t) {
        constexpr int BUF = decltype(buf_c)::value;
        const char *cur = lds + BUF * VM_TILE_BYTES;
        char *nxt = lds + (BUF ^ 1) * VM_TILE_BYTES;
        const int tn = min(t + 1, tiles - 1); // the last iteration re-fetches its own tile into the idle buffer
#pragma unroll
        for (int cb = 0; cb < VM_CB; ++cb) {
            const int pp = cb & 1;
#pragma unroll
            for (int s = 0; s < VM_KS; ++s) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    // the next tile's loads go out early in this tile (its buffer is idle since the last barrier),
                    // so that they have landed long before the barrier at the end
                    if (cb < VM_CB / 2 && (s & 1) && rb == 0) issue_load(tn, geo::LPC * cb + (s >> 1), nxt);
                    // RB independent accumulator chains, taken in turns (a chain's next link is RB MFMAs later)
                    if (s == 0)
                        acc[pp][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[s], a[rb][s], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    else
                        acc[pp][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[s], a[rb][s], acc[pp][rb], 0, 0, 0);
                    // after its last use in this block, refill the fragment slot for the next block
                    if (rb == RB - 1 && cb + 1 < VM_CB)
                        b[s] = *reinterpret_cast<const bf16x8 *>(cur + (cb + 1) * 16 * VM_COL_BYTES + boff[s]);
                    // drain the previous column block's accumulators (complete since >= RB MFMAs): 4 / KS values per MFMA
#pragma unroll
                    for (int v = 0; v < 4 / VM_KS; ++v) sum[rb][s * (4 / VM_KS) + v] += fabsf(acc[pp ^ 1][rb][s * (4 / VM_KS) + v]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < VM_KS; ++s) b[s] = *reinterpret_cast<const bf16x8 *>(nxt + boff[s]);
    };
    for (int t = 0; t < tiles; t += 2) {
        tile_step(std::integral_constant<int, 0>{}, t);
        if (t + 1 < tiles) tile_step(std::integral_constant<int, 1>{}, t + 1);
    }
    // the last column block is still in acc[(VM_CB - 1) & 1]
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < 4; ++j) sum[rb][j] += fabsf(acc[(VM_CB - 1) & 1][rb][j]);

    // accumulator value j of lane (l16, kc) is output column 4 * kc + j of token l16: merge the four values and
    // the four lanes of a token
    float *out = vnorm + ((size_t)bi * H + h) * (size_t)n;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        float x = (sum[rb][0] + sum[rb][1]) + (sum[rb][2] + sum[rb][3]);
        x += __shfl_xor(x, 16);
        x += __shfl_xor(x, 32);
        const int row = row0 + rb * 16 + l16;
        if (kc == 0 && row < n) out[row] = x;
    }
}

// row blocks per wave that the launcher takes, and the arguments and workgroups that go with them
int vproj_mfma_row_blocks(const Dims &d);
VprojArgs vproj_mfma_args(const Dims &d, int row_blocks, const void *v, const void *w_t, float *vnorm, unsigned *wgs);

} // namespace ckv
