// Internal declarations shared by the host dispatch and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "criticalkv.h"

namespace ckv {

// bf16 storage type: raw 16 bits; conversion to float is a shift (exact).
typedef uint16_t bf16_t;

__device__ __forceinline__ float bf16_to_f32(bf16_t x) { return __uint_as_float(((uint32_t)x) << 16); }
__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return bf16_to_f32(x); }

// 16 bytes past the caches' replacement order (what is read once, or written for a reader that comes much later).
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
__device__ __forceinline__ u32x4 load16_once(const void *p) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p)); }
__device__ __forceinline__ void store16_once(void *p, u32x4 x) { __builtin_nontemporal_store(x, reinterpret_cast<u32x4 *>(p)); }

// Problem sizes resolved from the descriptor (strides filled in).
struct Dims {
    int batch, H, Hkv, G, dh, dm, n, W, pool_k;
    int window_sum;
    int norm; // CKV_NORM_L1 or CKV_NORM_L2
    int attn_only; // no magnitudes in this call
    int causal;  // window row w sees keys <= n - W + w only
    int protect; // trailing entries the selection keeps as they are (0 or W)
    float scale, eps;
    int64_t ks[3], vs[3];
};

// Workspace carving for criticalkv_score / criticalkv_select (byte offsets, 256-aligned).
struct Workspace {
    size_t a_raw;      // [batch, H, n] f32: window score per query head before pooling
    size_t vnorm;      // [batch, H, n] f32: projected-value norm (when the caller passes none)
    size_t stats_part; // [batch, H, W, chunks, 2] f32: per-chunk (max, sum of exp)
    size_t stats;      // [batch, H, W, 2] f32: per-row (max + log sum, unused)
    size_t w_t;        // [d_model, H*dh] copy of W_O in output-major layout (when given canonical)
    size_t sel_keys;   // [batch*Hkv, n] u32: stage-2 keys with stage-1 entries marked
    size_t l2_scratch; // Gram partial sums and the split bf16 Gram matrices (L2 norm only)
    size_t diag_part;  // per-chunk partial sums of the perturbation diagnostics
    size_t alloc_tmp;  // budget allocation: counts per head (batch * Hkv words of what max_budget reserves)
    size_t sel_scratch; // digit histograms, per-head state, per-slice counts of the selection kernels
    size_t total;
    size_t w_split;    // fp32 layers: the two-part copy of W_O; lies behind what every call needs (see carve_workspace)
    size_t total_split;
    int max_chunks;    // capacity of stats_part per window row
};

constexpr int ATTN_MIN_CHUNK = 128; // fewest keys an attention kernel gives one workgroup (sizes stats_part), and of those
constexpr int ATTN_SHORT_CHUNK = 64; // bf16 launches that have no more workgroups than the chip has CUs
constexpr int ATTN_SHORT_WGS = 256;
int generic_attn_chunks(const Dims &d);
int mfma_attn_chunks(const Dims &d);
bool attn_mfma_supported(const Dims &d);  // shapes the matrix-core attention kernels cover (shared key tiles)
bool attn_wave_supported(const Dims &d);  // shapes the wave-private matrix-core attention kernels cover
int wave_attn_chunks(const Dims &d);
bool vproj_mfma_supported(const Dims &d); // shapes the matrix-core projection kernel covers

Workspace carve_workspace(const Dims &d, int dtype, int max_budget);

// ---- kernel launchers (each returns hipGetLastError after its launches) -------------------------
// window attention, pass 1: per (row, key chunk) running max and sum of exp
hipError_t launch_attn_stats_generic(const Dims &d, int dtype, const void *q, const void *k, float *part,
                                     int chunks, hipStream_t s);
// reduce chunk partials to one (max, 1/sum) pair per window row
hipError_t launch_attn_stats_reduce(const Dims &d, const float *part, int chunks, float *stats, hipStream_t s);
// window attention, pass 2: a_raw[b,h,i] = reduce_w exp(s - max_w) / sum_w
hipError_t launch_attn_colsum_generic(const Dims &d, int dtype, const void *q, const void *k, const float *stats,
                                      float *a_raw, hipStream_t s);
// (attn_mfma_merges: pass 2 takes the chunks' pairs in `part` instead of the reduced rows)
bool attn_mfma_merges(const Dims &d);
bool attn_wave_merges(const Dims &d);
hipError_t launch_attn_stats_mfma(const Dims &d, const void *q, const void *k, float *part, hipStream_t s);
// matrix-core path: partials are in the log2 domain; per row E = log2(sum 2^t) (+ log2 W for the mean)
hipError_t launch_attn_stats_reduce_log2(const Dims &d, const float *part, int chunks, float *stats, hipStream_t s);
hipError_t launch_attn_colsum_mfma(const Dims &d, const void *q, const void *k, const float *stats, float *a_raw,
                                   hipStream_t s);
// the same two sweeps with wave-private key streams (larger groups and windows, d_h = 64); same partial layout
hipError_t launch_attn_stats_wave(const Dims &d, const void *q, const void *k, float *part, int chunks, hipStream_t s);
hipError_t launch_attn_colsum_wave(const Dims &d, const void *q, const void *k, const float *stats, float *a_raw,
                                   hipStream_t s);
// both sweeps for fp32 layers on the fp32 matrix instruction (pass 1, with the rows' (M, weight) left in part or stats, else
// pass 2); part holds part_floats floats
bool attn_f32_taken(const Dims &d, size_t part_floats);
hipError_t launch_attn_f32(const Dims &d, const void *q, const void *k, float *part, size_t part_floats, float *stats,
                           float *a_raw, bool pass1, hipStream_t s);
// projected-value L1 norm; w_t is [d_model, H*dh]
hipError_t launch_vproj_generic(const Dims &d, int dtype, const void *v, const void *w_t, float *vnorm,
                                hipStream_t s);
hipError_t launch_vproj_mfma(const Dims &d, const void *v, const void *w_t, float *vnorm, hipStream_t s);
// the projection and pass 2 of the shared-tile attention in one launch (short contexts)
bool vproj_colsum_room(const Dims &d);  // the projection leaves room for it
bool vproj_colsum_taken(const Dims &d); // ... and pass 2 merges the rows itself
hipError_t launch_vproj_colsum(const Dims &d, const void *q, const void *k, const void *v, const void *w_t, const float *part,
                               float *a_raw, float *vnorm, hipStream_t s);
// Row blocks per wave of a projection launch: of `choices`, the one whose rounds of workgroups cost least (the first of
// equals).  An XCD runs 64 workgroups at a time; a round costs RB + c2 with more than 32 of them, 0.48 RB + c1 with fewer.
int cheapest_rounds(const Dims &d, int rows_per_block, double c2, double c1, const int *choices, int count);
// the same (either norm) for fp32 layers, on the f16 matrix cores with every operand split into two parts; w_o in
// either layout, scratch holds vproj_split_bytes(d)
bool vproj_split_supported(const Dims &d);
size_t vproj_split_bytes(const Dims &d);
hipError_t launch_vproj_split(const Dims &d, int out_in, const void *v, const void *w_o, void *scratch, float *vnorm,
                              hipStream_t s);
// fp32 magnitudes and both sweeps, side by side where they do not depend on each other (short contexts)
bool split_colsum_taken(const Dims &d);
hipError_t launch_score_f32_short(const Dims &d, int out_in, const void *q, const void *k, const void *v, const void *w_o,
                                  void *scratch, float *part, size_t part_floats, float *stats, float *a_raw, float *vnorm,
                                  hipStream_t s);
// L2 norm through the Gram matrix W_O^h W_O^h^T (bf16, d_h = 128)
bool vproj_l2_mfma_supported(const Dims &d);
size_t vproj_l2_workspace_bytes(const Dims &d);
size_t vproj_l2_gram_bytes(const Dims &d); // the split bf16 Gram matrices alone
// w_o: the canonical [H*dh, d_model] projection
hipError_t launch_gram(const Dims &d, const void *w_o, void *gram_out, void *partial_scratch, hipStream_t s);
hipError_t launch_vproj_l2_mfma(const Dims &d, const void *v, const void *gram, float *vnorm, hipStream_t s);
// [rows, cols] -> [cols, rows]; rows and cols are multiples of 8 (bf16) or 4 (fp32) elements
hipError_t launch_transpose(int dtype, const void *in, void *out, int rows, int cols, hipStream_t s);
// pool + eps + product + group mean; crit may be null (only the pooled attention is written)
hipError_t launch_combine(const Dims &d, const float *a_raw, const float *vnorm, float *attn, float *crit,
                          hipStream_t s);
size_t select_workspace_words(int heads, int n); // u32 words of histogram / state / per-slice scratch
hipError_t launch_select(const Dims &d, const float *attn, const float *crit, const int32_t *budget, float alpha,
                         int max_budget, int32_t *idx, int32_t *count, uint32_t *keys2, uint32_t *scratch,
                         hipStream_t s);
// per-head budgets from a per-batch-item total; tmp holds batch * Hkv words, keys2 and scratch what a selection of these
// rows needs
hipError_t launch_allocate(const Dims &d, const float *attn, int total, float floor_frac, int32_t *budget_out,
                           uint32_t *keys2, uint32_t *scratch, int32_t *tmp, hipStream_t s);
// perturbation quantities of a finished selection; part holds diagnostics_workspace_floats(d) floats
size_t diagnostics_workspace_floats(const Dims &d);
hipError_t launch_diagnostics(const Dims &d, int dtype, int out_in, const void *v, const void *w_o, const float *a_raw,
                              const float *vnorm, const uint32_t *keys2, const int32_t *idx, const int32_t *count,
                              int max_budget, float *part, float *out, hipStream_t s);
hipError_t launch_compact(const Dims &d, int dtype, const void *k, const void *v, const int32_t *idx,
                          const int32_t *count, int max_budget, void *k_out, void *v_out, hipStream_t s);
// the same with n_new rows (strides in elements) behind the max_budget gathered ones of every head
hipError_t launch_compact_append(const Dims &d, int dtype, const void *k, const void *v, const int32_t *idx,
                                 const int32_t *count, int max_budget, const void *k_new, const void *v_new, int n_new,
                                 const int64_t *ks_new, const int64_t *vs_new, void *k_out, void *v_out, hipStream_t s);

} // namespace ckv
