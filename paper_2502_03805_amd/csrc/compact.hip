// Gather of the selected K/V rows into the compacted cache (Algorithm 1, line 10).
// Pure data movement: each row is dh * sizeof(elem) bytes, copied as 16-byte pieces by
// consecutive lanes so that both the read of a row and the write are contiguous.  With new rows behind the kept ones (the
// next chunk of a chunked prefill) the cache that the next pass scores is written in the same launch: 8 heads, 1024 kept and
// 2048 new rows of 256 bytes, us: gather 4.2 and two concatenations of 8.2 -> 5.4.
#include "common.hpp"

namespace ckv {

constexpr int CP_THREADS = 256;

struct NewRows { // rows appended to the gathered ones (none: n = 0)
    const char *k, *v;
    int n;
    int64_t ks0, ks1, ks2, vs0, vs1, vs2;
};

// STREAM: rows pass the caches by on both sides.  Where K and V together are longer than the Infinity Cache (256 MiB) they
// come from HBM, and in the ordinary order reads and write-backs push each other out.  8 heads of 131072 rows, us, ordinary /
// nontemporal stores / both: 52429 kept 82 / 78 / 70 (6.1 TB/s; a copy of 1 GiB runs at 5.1), 19661 kept 33.5 / 30 / 28; fp32
// rows, 8 heads of 60000, 18000 kept 58 / 55 / 50.  Shorter ones may still be there from the sweeps: 16 heads of 20011, 4002
// kept, in a chain of calls on rotating inputs 11.4 / 12.4 (both).
constexpr long long CP_STREAM_BYTES = 256ll << 20;

template <bool APPEND, bool STREAM>
__global__ __launch_bounds__(CP_THREADS) void compact_kernel(const char *__restrict__ k, const char *__restrict__ v,
                                                             const int32_t *__restrict__ idx,
                                                             const int32_t *__restrict__ count, char *__restrict__ k_out,
                                                             char *__restrict__ v_out, int Hkv, int n, int max_budget,
                                                             int row_bytes, int64_t ks0, int64_t ks1, int64_t ks2,
                                                             int64_t vs0, int64_t vs1, int64_t vs2, int esize,
                                                             NewRows N)
{
    const int head = blockIdx.y;            // bi * Hkv + g
    const int bi = head / Hkv, g = head % Hkv;
    const int pieces = row_bytes >> 4;      // 16-byte pieces per row
    const int cnt = min(count[head], max_budget);
    const long long t = (long long)blockIdx.x * CP_THREADS + threadIdx.x;
    const int j = (int)(t / pieces), piece = (int)(t % pieces);
    const char *krow, *vrow;
    if (APPEND && j >= max_budget) {
        const int i = j - max_budget;
        if (i >= N.n) return;
        krow = N.k + (bi * N.ks0 + g * N.ks1 + (int64_t)i * N.ks2) * esize;
        vrow = N.v + (bi * N.vs0 + g * N.vs1 + (int64_t)i * N.vs2) * esize;
    } else {
        if (j >= cnt) return;
        const int i = idx[(size_t)head * max_budget + j];
        if (i < 0 || i >= n) return;
        krow = k + (bi * ks0 + g * ks1 + (int64_t)i * ks2) * esize;
        vrow = v + (bi * vs0 + g * vs1 + (int64_t)i * vs2) * esize;
    }
    // the K piece and the V piece of the same row: one index read, two loads in flight per lane
    const u32x4 *kp = reinterpret_cast<const u32x4 *>(krow) + piece, *vp = reinterpret_cast<const u32x4 *>(vrow) + piece;
    const u32x4 kk = STREAM ? load16_once(kp) : *kp;
    const u32x4 vv = STREAM ? load16_once(vp) : *vp;
    const size_t o = ((size_t)head * (max_budget + (APPEND ? N.n : 0)) + j) * (size_t)row_bytes;
    u32x4 *ko = reinterpret_cast<u32x4 *>(k_out + o) + piece, *vo = reinterpret_cast<u32x4 *>(v_out + o) + piece;
    if (STREAM) {
        store16_once(ko, kk);
        store16_once(vo, vv);
    } else {
        *ko = kk;
        *vo = vv;
    }
}

template <bool APPEND>
static hipError_t launch(const Dims &d, int dtype, const void *k, const void *v, const int32_t *idx, const int32_t *count,
                         int max_budget, void *k_out, void *v_out, const NewRows &N, hipStream_t s)
{
    const int esize = dtype == CKV_F32 ? 4 : 2;
    const int row_bytes = d.dh * esize;
    const long long threads = ((long long)max_budget + N.n) * (row_bytes / 16);
    dim3 grid((unsigned)((threads + CP_THREADS - 1) / CP_THREADS), d.batch * d.Hkv);
    const bool stream = 2ll * d.batch * d.Hkv * d.n * row_bytes > CP_STREAM_BYTES;
    const auto kernel = stream ? compact_kernel<APPEND, true> : compact_kernel<APPEND, false>;
    hipLaunchKernelGGL(kernel, grid, dim3(CP_THREADS), 0, s, (const char *)k, (const char *)v, idx, count,
                       (char *)k_out, (char *)v_out, d.Hkv, d.n, max_budget, row_bytes, d.ks[0], d.ks[1], d.ks[2],
                       d.vs[0], d.vs[1], d.vs[2], esize, N);
    return hipGetLastError();
}

hipError_t launch_compact(const Dims &d, int dtype, const void *k, const void *v, const int32_t *idx,
                          const int32_t *count, int max_budget, void *k_out, void *v_out, hipStream_t s)
{
    return launch<false>(d, dtype, k, v, idx, count, max_budget, k_out, v_out, NewRows{}, s);
}

hipError_t launch_compact_append(const Dims &d, int dtype, const void *k, const void *v, const int32_t *idx,
                                 const int32_t *count, int max_budget, const void *k_new, const void *v_new, int n_new,
                                 const int64_t *ks_new, const int64_t *vs_new, void *k_out, void *v_out, hipStream_t s)
{
    const NewRows N = {(const char *)k_new, (const char *)v_new, n_new, ks_new[0], ks_new[1], ks_new[2], vs_new[0], vs_new[1], vs_new[2]};
    return launch<true>(d, dtype, k, v, idx, count, max_budget, k_out, v_out, N, s);
}

} // namespace ckv
