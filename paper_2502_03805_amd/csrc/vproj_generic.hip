// Per-entry L1 (or L2) magnitude of the projected value on the vector ALUs
// (Theorem 3.3; Algorithm 1, lines 2-3):  N^h_i = sum_c | sum_t V^g[i,t] * W_O^h[t,c] |.
//
// Serves what the matrix-core kernels do not cover (bf16 with the 2-norm at d_h 64 or a d_model that 512 does not divide, with
// the 1-norm a d_model that a tile of columns does not divide, CKV_NO_MFMA, fp32 layers whose workspace has no room for the
// two-part copy of W_O).  One thread owns
// one token row (kept in registers); the head's W_O slice is streamed through LDS in tiles
// of TC output columns and read as broadcasts.  The n x d_model products are reduced on the
// fly and never stored.
#include "common.hpp"

namespace ckv {

constexpr int VG_THREADS = 256;
constexpr int VG_TC = 32; // output columns per LDS tile

template <typename T, int DH, bool L2>
__global__ __launch_bounds__(VG_THREADS) void vproj_generic_kernel(const T *__restrict__ v, const T *__restrict__ w_t,
                                                                   float *__restrict__ vnorm, int H, int G, int n,
                                                                   int dm, int64_t vs0, int64_t vs1, int64_t vs2)
{
    __shared__ float w_lds[VG_TC * DH];
    const int h = blockIdx.y, bi = blockIdx.z, g = h / G;
    const int i = blockIdx.x * VG_THREADS + threadIdx.x;
    const bool valid = i < n;
    const T *row = v + bi * vs0 + g * vs1 + (int64_t)(valid ? i : n - 1) * vs2;
    float vr[DH];
#pragma unroll
    for (int t = 0; t < DH; ++t) vr[t] = to_f32(row[t]);
    const size_t ldw = (size_t)H * DH; // row pitch of w_t [dm, H*DH]
    float acc = 0.f;
    for (int c0 = 0; c0 < dm; c0 += VG_TC) {
        __syncthreads();
        for (int e = threadIdx.x; e < VG_TC * DH; e += VG_THREADS) {
            const int c = e / DH, t = e % DH;
            w_lds[e] = to_f32(w_t[(size_t)(c0 + c) * ldw + (size_t)h * DH + t]);
        }
        __syncthreads();
#pragma unroll 4
        for (int c = 0; c < VG_TC; ++c) {
            float p = 0.f;
#pragma unroll
            for (int t = 0; t < DH; t += 4) {
                const float4 ww = *reinterpret_cast<const float4 *>(&w_lds[c * DH + t]);
                p = fmaf(vr[t], ww.x, p); p = fmaf(vr[t + 1], ww.y, p);
                p = fmaf(vr[t + 2], ww.z, p); p = fmaf(vr[t + 3], ww.w, p);
            }
            acc += L2 ? p * p : fabsf(p);
        }
    }
    if (valid) vnorm[((size_t)bi * H + h) * (size_t)n + i] = L2 ? sqrtf(acc) : acc;
}

template <typename T, int DH>
static hipError_t vproj_generic_t(const Dims &d, const void *v, const void *w_t, float *vnorm, hipStream_t s)
{
    dim3 grid((d.n + VG_THREADS - 1) / VG_THREADS, d.H, d.batch);
    if (d.norm == CKV_NORM_L2)
        hipLaunchKernelGGL((vproj_generic_kernel<T, DH, true>), grid, dim3(VG_THREADS), 0, s, (const T *)v, (const T *)w_t,
                           vnorm, d.H, d.G, d.n, d.dm, d.vs[0], d.vs[1], d.vs[2]);
    else
        hipLaunchKernelGGL((vproj_generic_kernel<T, DH, false>), grid, dim3(VG_THREADS), 0, s, (const T *)v, (const T *)w_t,
                           vnorm, d.H, d.G, d.n, d.dm, d.vs[0], d.vs[1], d.vs[2]);
    return hipGetLastError();
}

hipError_t launch_vproj_generic(const Dims &d, int dtype, const void *v, const void *w_t, float *vnorm, hipStream_t s)
{
    if (dtype == CKV_F32)
        return d.dh == 64 ? vproj_generic_t<float, 64>(d, v, w_t, vnorm, s) : vproj_generic_t<float, 128>(d, v, w_t, vnorm, s);
    return d.dh == 64 ? vproj_generic_t<bf16_t, 64>(d, v, w_t, vnorm, s) : vproj_generic_t<bf16_t, 128>(d, v, w_t, vnorm, s);
}

// ---- layout change: [rows, cols] -> [cols, rows] ---------------------------------------------------
// Bound by memory.  No LDS: a lane turns a square block of 16-byte rows (8 x 8 bf16 or 4 x 4 fp32) in registers, and the
// wave's 8 x 8 lanes make every load and every store instruction move whole 128-byte lines; eight (four) loads are in
// flight per lane; the stores pass the caches by, so that they do not push out what is still to be read.  4096 x 4096 bf16:
// 21.5 us with a 32 x 32 LDS tile of single elements, 13.1 like this with ordinary stores, 11.7 with these (64 MiB, 5.7 TB/s; a
// copy of 1 GiB runs at 5.1); 5120 x 8192 29.0 / 24.4.
// In place of bounds checks inside a block: rows and cols are multiples of the block (cols of 32, rows of 64).
__device__ __forceinline__ void turn_block(uint4 (&x)[8]) // 8 x 8 of 16 bits
{
    uint32_t w[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i) { w[i][0] = x[i].x; w[i][1] = x[i].y; w[i][2] = x[i].z; w[i][3] = x[i].w; }
    // word k of output row j holds rows 2k and 2k + 1 of column j
    uint32_t o[8][4];
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k)
            o[j][k] = __builtin_amdgcn_perm(w[2 * k + 1][j >> 1], w[2 * k][j >> 1], (j & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = make_uint4(o[j][0], o[j][1], o[j][2], o[j][3]);
}
__device__ __forceinline__ void turn_block(uint4 (&x)[4]) // 4 x 4 of 32 bits
{
    const uint4 a = x[0], b = x[1], c = x[2], d = x[3];
    x[0] = make_uint4(a.x, b.x, c.x, d.x); x[1] = make_uint4(a.y, b.y, c.y, d.y);
    x[2] = make_uint4(a.z, b.z, c.z, d.z); x[3] = make_uint4(a.w, b.w, c.w, d.w);
}

template <typename T>
__global__ __launch_bounds__(256) void transpose_kernel(const T *__restrict__ in, T *__restrict__ out, int rows, int cols)
{
    constexpr int E = 16 / sizeof(T); // block edge: elements per 16 bytes
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // the eight lanes of a load that differ in lane & 7 read neighbouring column blocks of a row; in a store, the eight
    // that differ in lane >> 3 write neighbouring row blocks of a column
    const int lr = blockIdx.y * (8 * E) + (lane >> 3) * E, lc = (blockIdx.x * 4 + wave) * (8 * E) + (lane & 7) * E;
    if (lr >= rows || lc >= cols) return;
    uint4 x[E];
#pragma unroll
    for (int i = 0; i < E; ++i) x[i] = *reinterpret_cast<const uint4 *>(in + (size_t)(lr + i) * cols + lc);
    turn_block(x);
#pragma unroll
    for (int j = 0; j < E; ++j) store16_once(out + (size_t)(lc + j) * rows + lr, u32x4{x[j].x, x[j].y, x[j].z, x[j].w});
}

hipError_t launch_transpose(int dtype, const void *in, void *out, int rows, int cols, hipStream_t s)
{
    const int edge = dtype == CKV_F32 ? 32 : 64; // rows and columns of one wave's tile; four waves side by side
    dim3 grid((cols + 4 * edge - 1) / (4 * edge), (rows + edge - 1) / edge);
    if (dtype == CKV_F32)
        hipLaunchKernelGGL(transpose_kernel<float>, grid, dim3(256), 0, s, (const float *)in, (float *)out, rows, cols);
    else
        hipLaunchKernelGGL(transpose_kernel<bf16_t>, grid, dim3(256), 0, s, (const bf16_t *)in, (bf16_t *)out, rows, cols);
    return hipGetLastError();
}

} // namespace ckv
