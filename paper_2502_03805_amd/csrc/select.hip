// Budget split and the two Top-k stages (Algorithm 1, lines 4-9).
//
//   b' = floor(alpha * B), b'' = B - b'
//   S1 = the b' largest attn;  S2 = the b'' largest crit among entries outside S1
//   idx = S1 u S2 in ascending token order
// With a kept observation window (protect = W > 0) the last min(W, B) entries are part of the result as they
// are, and the two stages run on entries 0 .. n-W-1 with the budget that is left (B above is then that rest).
// Top-k is an exact order statistic: a most-significant-digit radix select on an order-preserving
// 32-bit image of the float keys (digits of 11, 11 and 10 bits).  Equal keys are taken in ascending
// token order: after the last digit the threshold key tau and the number r of entries equal to tau that
// still fit are known, and the r-th tie is located with ordered prefix counts.
//
// A head's n keys are cut into slices of 2048 tokens, one 256-thread workgroup per (slice, head), so the
// whole chip works on a layer's few heads.  Workgroups only meet at kernel boundaries:
//   zero      clear the digit histograms
//   hist 1.0  digit-0 histogram of attn            (LDS histogram per slice, flushed with integer atomics)
//   hist 1.1  find digit 0, digit-1 histogram of the entries that match it
//   hist 1.2  find digit 1, digit-2 histogram (each slice also keeps its own copy)
//   mark      find digit 2 -> tau1, r1; stage-1 membership (ties ranked through the slices' own digit-2
//             histograms: the ties of a slice are its count at digit 2 of tau1), stage-2 keys written
//             (stage-1 entries carry a reserved key), digit-0 histogram of stage 2
//   hist 2.1, hist 2.2  (each slice also counts its entries above the digit just decided; 2.2 keeps the slice's
//             digit-2 counts as suffix sums)
//   write     find digit 2 -> tau2, r2; ordered write of S1 u S2: what earlier slices contribute is read from
//             their per-slice counts; -1 tail; count
// Every decision is integer arithmetic on exact counts, so the result does not depend on scheduling.
#include <algorithm>

#include "common.hpp"

namespace ckv {

constexpr int SEL_THREADS = 256;
constexpr int SEL_PER_THREAD = 8;
constexpr int SEL_SLICE = SEL_THREADS * SEL_PER_THREAD; // tokens per workgroup
constexpr int SEL_BINS = 2048;
constexpr uint32_t SEL_TAKEN = 0xFFFFFFFFu; // image of no finite float: marks stage-1 entries
constexpr int DSHIFT0 = 21, DSHIFT1 = 10;
constexpr uint32_t DMASK0 = 0x7FFu, DMASK1 = 0x7FFu, DMASK2 = 0x3FFu;

// per-head state words
enum { ST_D0 = 0, ST_A0, ST_D1, ST_A1, ST_TAU, ST_R, ST_WORDS = 8 };

struct SelArgs {
    const uint32_t *attn; // float bits
    const uint32_t *crit;
    const int32_t *budget; // null: max_budget for every head
    uint32_t *keys2;   // [heads][n]
    uint32_t *hist;    // [heads][2 stages][3 passes][SEL_BINS]
    uint32_t *state;   // [heads][2 stages][ST_WORDS]
    uint32_t *slices;  // [heads][3][n_slices]: stage-1 members; stage-2 entries above the threshold at digit 0; at digit 1
    uint32_t *slice_suf; // [heads][n_slices][1025]: each slice's digit-2 suffix counts of stage 2
    uint32_t *slice_hist; // [heads][n_slices][1024]: each slice's digit-2 histogram of stage 1
    int32_t *idx;
    int32_t *count;
    double alpha;
    int n, max_budget, n_slices;
    int share;  // allocation: rows of one batch item share a histogram and a threshold (1: every row has its own)
    int n_rank; // entries 0 .. n_rank-1 compete in the two stages (n minus the kept window)
};

// Monotone map float -> uint32 (larger float, larger key); -0 and +0 share a key.
__device__ __forceinline__ uint32_t order_key(uint32_t u)
{
    u = __float_as_uint(__uint_as_float(u) + 0.f); // (-0 becomes +0)
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

// B: entries the head keeps in all; kept: how many of them are the kept window's (the last `kept` entries);
// b1, b2: the two stages' shares of the rest
__device__ __forceinline__ void head_budget(const SelArgs &A, int head, int &B, int &b1, int &b2, int &kept)
{
    B = max(0, min(A.budget ? A.budget[head] : A.max_budget, min(A.n, A.max_budget)));
    kept = min(A.n - A.n_rank, B);
    const int rest = B - kept;
    b1 = (int)floor(A.alpha * (double)rest);
    b2 = rest - b1;
}

struct SelShared {
    uint32_t hist[SEL_BINS];
    uint32_t wave_tot[SEL_THREADS / 64];
    uint32_t digit, above;
};

// Inclusive prefix sum over the wave: shifts inside rows of 16 lanes, then the rows' last lanes broadcast to the rows
// behind (no LDS round trips, which a shuffle costs: they were a fifth of a row kernel's time).
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false); // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false); // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false); // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false); // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false); // row_bcast:15 into rows 1, 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false); // row_bcast:31 into rows 2, 3
    return x;
}

// Exclusive prefix sum over the workgroup in thread order; total in `total`.
__device__ __forceinline__ uint32_t block_exclusive_scan(SelShared &sh, uint32_t x, uint32_t &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t incl = wave_inclusive_scan(x);
    __syncthreads(); // wave_tot may still be read by a previous scan
    if (lane == 63) sh.wave_tot[wave] = incl;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < SEL_THREADS / 64; ++w) {
        const uint32_t t = sh.wave_tot[w];
        if (w < wave) base += t;
        tot += t;
    }
    total = tot;
    return base + incl - x;
}

__device__ __forceinline__ uint32_t block_sum(SelShared &sh, uint32_t x)
{
    uint32_t total;
    (void)block_exclusive_scan(sh, x, total);
    return total;
}

// How a row lies in its array: words from the last 16-byte boundary to its start, and words from its start to the
// array's end (rows are packed, so a row of odd length shifts the next one's alignment).
struct RowPlace {
    int shift;
    long long avail, total;
};
__device__ __forceinline__ RowPlace row_place(int row, int rows, int n)
{
    RowPlace p;
    p.shift = (int)(((long long)row * n) & 3);
    p.avail = (long long)(rows - row) * n;
    p.total = (long long)rows * n;
    return p;
}

// The thread's 8 consecutive words starting at token i0 (a multiple of 8); the caller masks those at or beyond n.  A
// shifted row is read as the three aligned 16-byte pieces around the eight words (they lie inside the array: in this row
// or its neighbours); single words only where a piece would cross the array's end.  (n 20011 against 20000, all eight
// kernels: 44.5 / 38 us when a shifted row was read word by word.)
__device__ __forceinline__ void load8(const uint32_t *base, int i0, int n, RowPlace at, uint32_t (&out)[8])
{
    if (i0 + 7 < n && i0 + 11 - at.shift < at.avail) {
        const uint4 *p = reinterpret_cast<const uint4 *>(base + i0 - at.shift);
        const uint4 a = p[0], b = p[1];
        uint4 c = make_uint4(0u, 0u, 0u, 0u);
        if (at.shift) c = p[2]; // uniform
        const uint32_t w[12] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x, c.y, c.z, c.w};
        const uint32_t odd = (at.shift & 1) ? 0xFFFFFFFFu : 0u, two = (at.shift & 2) ? 0xFFFFFFFFu : 0u;
        uint32_t x[10];
#pragma unroll
        for (int j = 0; j < 10; ++j) x[j] = (w[j] & ~odd) | (w[j + 1] & odd);
#pragma unroll
        for (int j = 0; j < 8; ++j) out[j] = (x[j] & ~two) | (x[j + 2] & two);
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) out[j] = (i0 + j < n) ? base[i0 + j] : 0u;
    }
}

// Largest digit d of a global histogram with  #(digit > d) < remaining <= #(digit >= d); also #(digit > d).
__device__ void find_digit(SelShared &sh, const uint32_t *ghist, int nbins, uint32_t remaining, uint32_t &digit,
                           uint32_t &above)
{
    constexpr int PER = SEL_BINS / SEL_THREADS; // 8 bins per thread, descending order
    uint32_t h[PER], local = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int bin = nbins - 1 - (threadIdx.x * PER + j);
        h[j] = bin >= 0 ? ghist[bin] : 0u;
        local += h[j];
    }
    if (threadIdx.x == 0) { sh.digit = 0u; sh.above = 0u; }
    uint32_t total;
    uint32_t run = block_exclusive_scan(sh, local, total);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (run < remaining && remaining <= run + h[j]) {
            sh.digit = (uint32_t)(nbins - 1 - (threadIdx.x * PER + j));
            sh.above = run;
        }
        run += h[j];
    }
    __syncthreads();
    digit = sh.digit;
    above = sh.above;
    __syncthreads();
}

__global__ __launch_bounds__(256) void select_zero_kernel(uint32_t *p, size_t words)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < words) p[i] = 0u;
}

// Histogram of one digit over a slice.  STAGE 0 reads attn floats, STAGE 1 the stage-2 key array.
// PASS 0 histograms digit 0 of every entry; PASS 1 / 2 first decode the previous digit(s) of the threshold.
// COUNT: slices keep their counts above the threshold (stage 2, and the allocation, whose A.share rows make up one).
template <int STAGE, int PASS, bool COUNT = STAGE == 1>
__global__ __launch_bounds__(SEL_THREADS) void select_hist_kernel(SelArgs A)
{
    __shared__ SelShared sh;
    const int slice = blockIdx.x, head = blockIdx.y;
    int B, b1, b2, kept;
    head_budget(A, head, B, b1, b2, kept);
    const bool alloc = STAGE == 0 && COUNT;
    const uint32_t want = alloc ? (uint32_t)A.max_budget : STAGE == 0 ? (uint32_t)b1 : (uint32_t)b2;
    if (want == 0) return;
    const int owner = alloc ? head / A.share : head; // whose threshold this row's keys are compared with
    const bool first = slice == 0 && threadIdx.x == 0 && (!alloc || head % A.share == 0);
    uint32_t *hist = A.hist + ((size_t)owner * 2 + STAGE) * 3 * SEL_BINS;
    uint32_t *st = A.state + ((size_t)owner * 2 + STAGE) * ST_WORDS;
    uint32_t prefix = 0u, pmask = 0u;
    if (PASS == 1) {
        uint32_t d0, a0;
        find_digit(sh, hist, 2048, want, d0, a0);
        if (first) { st[ST_D0] = d0; st[ST_A0] = a0; }
        prefix = d0 << DSHIFT0; pmask = DMASK0 << DSHIFT0;
    } else if (PASS == 2) {
        const uint32_t d0 = st[ST_D0], a0 = st[ST_A0];
        uint32_t d1, a1;
        find_digit(sh, hist + SEL_BINS, 2048, want - a0, d1, a1);
        if (first) { st[ST_D1] = d1; st[ST_A1] = a1; }
        prefix = (d0 << DSHIFT0) | (d1 << DSHIFT1);
        pmask = (DMASK0 << DSHIFT0) | (DMASK1 << DSHIFT1);
    }
    const int shift = PASS == 0 ? DSHIFT0 : PASS == 1 ? DSHIFT1 : 0;
    const uint32_t mask = PASS == 2 ? DMASK2 : DMASK0;

    for (int b = threadIdx.x; b < SEL_BINS; b += SEL_THREADS) sh.hist[b] = 0u;
    __syncthreads();
    const uint32_t *src = (STAGE == 0 ? A.attn : A.keys2) + (size_t)head * A.n;
    const int i0 = slice * SEL_SLICE + threadIdx.x * SEL_PER_THREAD;
    uint32_t w[8];
    load8(src, i0, A.n, row_place(head, gridDim.y, A.n), w);
    // runs of equal digits inside a thread's 8 tokens are merged into one atomic
    uint32_t run_digit = 0u, run_len = 0u, n_above = 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t key = STAGE == 0 ? order_key(w[j]) : w[j];
        const bool on = (i0 + j < A.n_rank) && key != SEL_TAKEN && (key & pmask) == prefix;
        if (COUNT && PASS >= 1) {
            // entries that beat the threshold at the digit this kernel has just decided (and agree with it
            // on the digit before): the ordered write adds these per-slice counts up instead of counting again
            constexpr uint32_t M0 = DMASK0 << DSHIFT0;
            const bool above = (i0 + j < A.n_rank) && key != SEL_TAKEN && (key & pmask) > prefix &&
                               (PASS == 1 || (key & M0) == (prefix & M0));
            n_above += above ? 1u : 0u;
        }
        const uint32_t d = (key >> shift) & mask;
        if (on && run_len && d == run_digit) {
            ++run_len;
        } else {
            if (run_len) atomicAdd(&sh.hist[run_digit], run_len);
            run_digit = d;
            run_len = on ? 1u : 0u;
        }
    }
    if (run_len) atomicAdd(&sh.hist[run_digit], run_len);
    __syncthreads();
    uint32_t *dst = hist + PASS * SEL_BINS;
    for (int b = threadIdx.x; b < SEL_BINS; b += SEL_THREADS) {
        const uint32_t c = sh.hist[b];
        if (c) atomicAdd(&dst[b], c);
    }
    if (STAGE == 0 && PASS == 2 && !COUNT) { // the slice's own counts: the mark kernel reads its ties from here
        uint32_t *mine = A.slice_hist + ((size_t)head * A.n_slices + slice) * 1024;
        for (int b = threadIdx.x; b < 1024; b += SEL_THREADS) mine[b] = sh.hist[b];
    }
    if (COUNT && PASS >= 1) {
        uint32_t *sl = A.slices + (size_t)head * 3 * A.n_slices;
        const uint32_t tot = block_sum(sh, n_above);
        if (threadIdx.x == 0) sl[PASS * A.n_slices + slice] = tot;
    }
    if (COUNT && PASS == 2) {
        // the slice's digit-2 counts as suffix sums: suf[b] = entries of the slice (with the threshold's first two
        // digits) whose digit 2 is >= b; suf[1024] = 0.  The write kernel reads suf[d2 + 1] and suf[d2].
        static_assert(SEL_THREADS * 4 == 1024, "four bins per thread");
        uint32_t h[4], local = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) { h[j] = sh.hist[threadIdx.x * 4 + j]; local += h[j]; }
        uint32_t total;
        uint32_t below = block_exclusive_scan(sh, local, total); // entries in bins before this thread's
        uint32_t *suf = A.slice_suf + ((size_t)head * A.n_slices + slice) * 1025;
#pragma unroll
        for (int j = 0; j < 4; ++j) { suf[threadIdx.x * 4 + j] = total - below; below += h[j]; }
        if (threadIdx.x == 0) suf[1024] = 0u;
    }
}

// Stage-1 membership, stage-2 keys, digit-0 histogram of stage 2.
__global__ __launch_bounds__(SEL_THREADS) void select_mark_kernel(SelArgs A)
{
    __shared__ SelShared sh;
    const int slice = blockIdx.x, head = blockIdx.y;
    int B, b1, b2, kept;
    head_budget(A, head, B, b1, b2, kept);
    uint32_t *st1 = A.state + ((size_t)head * 2 + 0) * ST_WORDS;
    uint32_t tau1 = 0u, r1 = 0u, before = 0u;
    if (b1 > 0) { // uniform over the workgroup
        // last digit of the stage-1 threshold, decided redundantly by every workgroup
        const uint32_t d0 = st1[ST_D0], a0 = st1[ST_A0], d1 = st1[ST_D1], a1 = st1[ST_A1];
        uint32_t d2, a2;
        find_digit(sh, A.hist + ((size_t)head * 2 + 0) * 3 * SEL_BINS + 2 * SEL_BINS, 1024, (uint32_t)b1 - a0 - a1, d2, a2);
        tau1 = (d0 << DSHIFT0) | (d1 << DSHIFT1) | d2;
        r1 = (uint32_t)b1 - a0 - a1 - a2;
        if (slice == 0 && threadIdx.x == 0) { st1[ST_TAU] = tau1; st1[ST_R] = r1; }
        // ties of stage 1 in earlier slices: their counts at digit d2 (only entries with the threshold's first two
        // digits were counted there)
        const uint32_t *sh2 = A.slice_hist + (size_t)head * A.n_slices * 1024 + d2;
        for (int s = threadIdx.x; s < slice; s += SEL_THREADS) before += sh2[(size_t)s * 1024];
        before = block_sum(sh, before);
    }

    const bool vec_ok = (A.n & 3) == 0;
    const int i0 = slice * SEL_SLICE + threadIdx.x * SEL_PER_THREAD;
    uint32_t a[8], c[8];
    const RowPlace at = row_place(head, gridDim.y, A.n);
    load8(A.attn + (size_t)head * A.n, i0, A.n, at, a);
    load8(A.crit + (size_t)head * A.n, i0, A.n, at, c);
    bool gt[8], tie[8];
    uint32_t n_tie = 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t key = order_key(a[j]);
        const bool valid = i0 + j < A.n_rank;
        gt[j] = b1 > 0 && valid && key > tau1;
        tie[j] = b1 > 0 && valid && key == tau1;
        n_tie += tie[j] ? 1u : 0u;
    }
    uint32_t tot;
    uint32_t rank = before + block_exclusive_scan(sh, n_tie, tot);
    for (int b = threadIdx.x; b < SEL_BINS; b += SEL_THREADS) sh.hist[b] = 0u;
    __syncthreads();
    uint32_t key2[8];
    uint32_t run_digit = 0u, run_len = 0u, n_taken = 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        bool taken = gt[j] || (i0 + j >= A.n - kept && i0 + j < A.n); // the kept window carries the stage-1 mark
        if (tie[j]) { taken = rank < r1; ++rank; }
        n_taken += taken ? 1u : 0u;
        key2[j] = taken ? SEL_TAKEN : order_key(c[j]);
        const bool on = b2 > 0 && (i0 + j < A.n_rank) && !taken;
        const uint32_t d = (key2[j] >> DSHIFT0) & DMASK0;
        if (on && run_len && d == run_digit) {
            ++run_len;
        } else {
            if (run_len) atomicAdd(&sh.hist[run_digit], run_len);
            run_digit = d;
            run_len = on ? 1u : 0u;
        }
    }
    if (run_len) atomicAdd(&sh.hist[run_digit], run_len);
    uint32_t *k2 = A.keys2 + (size_t)head * A.n;
    if (vec_ok && i0 + 7 < A.n) {
        *reinterpret_cast<uint4 *>(k2 + i0) = make_uint4(key2[0], key2[1], key2[2], key2[3]);
        *reinterpret_cast<uint4 *>(k2 + i0 + 4) = make_uint4(key2[4], key2[5], key2[6], key2[7]);
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (i0 + j < A.n) k2[i0 + j] = key2[j];
    }
    __syncthreads();
    if (b2 > 0) {
        uint32_t *dst = A.hist + ((size_t)head * 2 + 1) * 3 * SEL_BINS;
        for (int b = threadIdx.x; b < SEL_BINS; b += SEL_THREADS) {
            const uint32_t cnt = sh.hist[b];
            if (cnt) atomicAdd(&dst[b], cnt);
        }
    }
    const uint32_t taken_here = block_sum(sh, n_taken);
    if (threadIdx.x == 0) A.slices[(size_t)head * 3 * A.n_slices + slice] = taken_here;
}

// Ordered write of S1 u S2.
__global__ __launch_bounds__(SEL_THREADS) void select_write_kernel(SelArgs A)
{
    __shared__ SelShared sh;
    const int slice = blockIdx.x, head = blockIdx.y;
    int B, b1, b2, kept;
    head_budget(A, head, B, b1, b2, kept);
    uint32_t *st2 = A.state + ((size_t)head * 2 + 1) * ST_WORDS;
    uint32_t tau2 = 0u, r2 = 0u, d2 = 0u;
    if (b2 > 0) { // uniform over the workgroup: last digit of the stage-2 threshold
        const uint32_t d0 = st2[ST_D0], a0 = st2[ST_A0], d1 = st2[ST_D1], a1 = st2[ST_A1];
        uint32_t a2;
        find_digit(sh, A.hist + ((size_t)head * 2 + 1) * 3 * SEL_BINS + 2 * SEL_BINS, 1024, (uint32_t)b2 - a0 - a1, d2, a2);
        tau2 = (d0 << DSHIFT0) | (d1 << DSHIFT1) | d2;
        r2 = (uint32_t)b2 - a0 - a1 - a2;
        if (slice == 0 && threadIdx.x == 0) { st2[ST_TAU] = tau2; st2[ST_R] = r2; }
    }
    const uint32_t *taken_cnt = A.slices + (size_t)head * 3 * A.n_slices;
    const uint32_t *above0 = taken_cnt + A.n_slices, *above1 = above0 + A.n_slices;
    const uint32_t *suf = A.slice_suf + (size_t)head * A.n_slices * 1025;
    // entries written and stage-2 ties seen by earlier slices: slice s' contributes its stage-1 members, its
    // stage-2 keys above tau2 (counted digit by digit by the histogram kernels) and
    // clamp(r2 - ties before s', 0, ties of s')
    uint32_t out_base = 0u, tie_base = 0u, carry = 0u;
    for (int c0 = 0; c0 < slice; c0 += SEL_THREADS) {
        const int s = c0 + threadIdx.x;
        uint32_t t = 0u, sel_s = 0u;
        if (s < slice) {
            sel_s = taken_cnt[s];
            if (b2 > 0) {
                const uint32_t ge = suf[(size_t)s * 1025 + d2], gt2 = suf[(size_t)s * 1025 + d2 + 1];
                t = ge - gt2;
                sel_s += above0[s] + above1[s] + gt2;
            }
        }
        uint32_t tot;
        const uint32_t tb = carry + block_exclusive_scan(sh, t, tot);
        uint32_t mine = 0u;
        if (s < slice) mine = sel_s + min(r2 > tb ? r2 - tb : 0u, t);
        out_base += block_sum(sh, mine);
        carry += tot;
    }
    tie_base = carry;

    const int i0 = slice * SEL_SLICE + threadIdx.x * SEL_PER_THREAD;
    uint32_t key[8];
    load8(A.keys2 + (size_t)head * A.n, i0, A.n, row_place(head, gridDim.y, A.n), key);
    bool sel[8], tie[8];
    uint32_t n_tie = 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const bool valid = i0 + j < A.n_rank; // window entries outside the budget carry ordinary keys: not ranked
        const bool taken = i0 + j < A.n && key[j] == SEL_TAKEN;
        sel[j] = taken || (b2 > 0 && valid && key[j] > tau2);
        tie[j] = b2 > 0 && valid && key[j] == tau2;
        n_tie += tie[j] ? 1u : 0u;
    }
    uint32_t tot;
    uint32_t rank = tie_base + block_exclusive_scan(sh, n_tie, tot);
    uint32_t n_sel = 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (tie[j]) { sel[j] = rank < r2; ++rank; }
        n_sel += sel[j] ? 1u : 0u;
    }
    uint32_t pos = out_base + block_exclusive_scan(sh, n_sel, tot);
    int32_t *out = A.idx + (size_t)head * A.max_budget;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (sel[j]) {
            if (pos < (uint32_t)A.max_budget) out[pos] = i0 + j;
            ++pos;
        }
    // unused tail and the count, spread over the slices
    for (int j = B + slice * SEL_THREADS + (int)threadIdx.x; j < A.max_budget; j += A.n_slices * SEL_THREADS) out[j] = -1;
    if (slice == 0 && threadIdx.x == 0) A.count[head] = B;
}

// ---- rows that one workgroup holds in registers ----------------------------------------------------------------------
// The whole selection of a head in one launch: a thread keeps KPT keys of both score arrays in registers (tokens
// (j * 1024 + thread) * 4 + e: every load is 16 bytes per lane), the digit histograms and prefix sums live in LDS.
// The same digits, thresholds and tie order as the sliced kernels above, so the result is the same set.
//   * a digit's histogram has several copies, interleaved (bin * copies + lane % copies): scores crowd into few bins, and
//     the lanes of an LDS atomic that hit one address are served one after the other.  Summing and clearing them costs too:
//     two copies for rows of up to 8192 keys, four for longer ones (1024 / 8192 / 24576 keys, us: two 9.9 / 13.5 / 27.6, four
//     10.9 / 14.3 / 27.0, eight 17 / 20 / 32)
//   * the thread that sums a bin also clears it, so a digit costs three barriers
//   * ties are ranked only when the threshold's ties do not all fit
//
//   * a key that does not compete (outside the row, chosen already) is 0, so that no mask has to be asked for it
//   * the digits end when all keys that share them fit: scores without ties are mostly told apart by two
//
// What bounds it: at short rows the six digits' barriers (about 0.7 us each, and 3 us for a launch that only loads and
// stores); at long ones the passes over the keys on one CU (a few vector instructions and an LDS atomic per key and digit, 2.3
// us a digit at 20011 keys), so the time grows with the row while the sliced kernels cost eight launches whatever its
// length.  Eight heads in a graph, us, sliced / one workgroup, with a mask of the competing keys and all six digits / like
// this: n 1024 36 / 11.2 / 9.7, 3072 36 / 11.4 / 10.1, 8192 37 / 14.8 / 12.8, 16384 37 / 21.6 / 17.9, 20011 37 / 26.5 / 21.6 (23.5 with
// all digits), 24576 38 / 27.5 / 22.9: rows of up
// to 24576 keys are taken whole (32 keys a thread spill).  (Merging runs of equal digits into one atomic, as the sliced
// kernels do, costs more instructions than it saves atomics here: 8192 keys 18.5 instead of 17.3 us when that was tried.)
constexpr int SEL_ROW_MAX = 24576;
constexpr int ROW_THREADS = 1024;
constexpr int ROW_WAVES = ROW_THREADS / 64;

struct RowShared {
    uint32_t hist[SEL_BINS * 4]; // row_copies(KPT) of the four interleaved
    uint32_t wave_tot[4][ROW_WAVES];
    uint32_t digit, above, inside;
};

constexpr int row_copies(int kpt) { return kpt <= 8 ? 2 : 4; }

// Sum of the totals of the waves before this one, and of all: lanes 0-15 of every row of lanes hold one total each.
__device__ __forceinline__ uint32_t waves_before(const uint32_t (&wave_tot)[ROW_WAVES], uint32_t &total)
{
    static_assert(ROW_WAVES == 16, "one total per lane of a DPP row");
    uint32_t x = wave_tot[threadIdx.x & 15];
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false); // row_shr:1, 2, 4, 8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    total = (uint32_t)__builtin_amdgcn_readlane((int)x, ROW_WAVES - 1);
    return wave ? (uint32_t)__builtin_amdgcn_readlane((int)x, wave - 1) : 0u;
}

// Exclusive prefix sums in thread order of NP words at once (two 16-bit counts each); totals as well.
template <int NP>
__device__ __forceinline__ void row_scan(RowShared &sh, const uint32_t (&x)[NP], uint32_t (&excl)[NP], uint32_t (&total)[NP])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) incl[p] = wave_inclusive_scan(x[p]);
    __syncthreads(); // the totals of the scan before may still be read
    if (lane == 63) {
#pragma unroll
        for (int p = 0; p < NP; ++p) sh.wave_tot[p][wave] = incl[p];
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint32_t base = waves_before(sh.wave_tot[p], total[p]);
        excl[p] = base + incl[p] - x[p];
    }
}

// The threshold of the `want` largest keys: its key, how many of its ties still fit, and whether that is all of them (then it
// is a bound between the chosen and the others, and its last digits may be left at 0).  Keys of 0 do not compete (no float but a NaN has that image); 0 as the threshold says that there are fewer than `want` others.
// The histogram is clear on entry and on exit.
template <int KPT>
__device__ __forceinline__ void row_threshold(RowShared &sh, const uint32_t (&key)[KPT], uint32_t want, uint32_t &tau,
                                              uint32_t &fit, bool &all_fit)
{
    constexpr int PER = SEL_BINS / ROW_THREADS, COPIES = row_copies(KPT);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t *mine = sh.hist + (lane & (COPIES - 1));
    uint32_t prefix = 0u, rest = want; // the threshold's digits so far
    uint32_t one = 1u;
    asm volatile("" : "+v"(one)); // (a register, not an instruction per key)
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
        const int width = pass == 2 ? DSHIFT1 : DSHIFT0 - DSHIFT1, shift = pass == 0 ? DSHIFT0 : pass == 1 ? DSHIFT1 : 0;
#pragma unroll
        for (int j = 0; j < KPT; ++j) {
            const bool on = pass == 0 ? key[j] != 0u : (key[j] >> (shift + width)) == prefix;
            // (the last digit is asked of few keys: most waves have none at a given j)
            if (pass == 2 && __builtin_amdgcn_ballot_w64(on) == 0ull) continue;
            if (on) atomicAdd(&mine[(pass == 0 ? key[j] >> shift : (key[j] >> shift) & ((1u << width) - 1u)) * COPIES], one);
        }
        __syncthreads();
        // bins in descending order, PER per thread
        uint32_t h[PER], local = 0u;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            uint32_t *bin = &sh.hist[(SEL_BINS - 1 - ((int)threadIdx.x * PER + j)) * COPIES];
            if constexpr (COPIES == 2) {
                const uint2 c = *reinterpret_cast<const uint2 *>(bin);
                *reinterpret_cast<uint2 *>(bin) = make_uint2(0u, 0u);
                h[j] = c.x + c.y;
            } else {
                const uint4 c = *reinterpret_cast<const uint4 *>(bin);
                *reinterpret_cast<uint4 *>(bin) = make_uint4(0u, 0u, 0u, 0u);
                h[j] = c.x + c.y + c.z + c.w;
            }
            local += h[j];
        }
        const uint32_t incl = wave_inclusive_scan(local);
        if (lane == 63) sh.wave_tot[0][wave] = incl;
        if (threadIdx.x == 0) { sh.digit = 0u; sh.above = 0u; sh.inside = 0u; }
        __syncthreads();
        uint32_t all, run = waves_before(sh.wave_tot[0], all) + incl - local;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (run < rest && rest <= run + h[j]) {
                sh.digit = (uint32_t)(SEL_BINS - 1 - ((int)threadIdx.x * PER + j));
                sh.above = run;
                sh.inside = h[j];
            }
            run += h[j];
        }
        __syncthreads();
        prefix = pass == 0 ? sh.digit : (prefix << width) | sh.digit;
        rest -= sh.above;
        all_fit = sh.inside == rest;
        tau = prefix << shift;
        if (all_fit) break; // uniform: every key with these digits is chosen, whatever its others
    }
    fit = rest;
}

// Keys a workgroup's quads have to cover: a row of odd length may begin up to three words into its first quad.
static int row_span(int n) { return n + (n & 3 ? 3 : 0); }

__device__ __forceinline__ int row_token(int j) { return ((j >> 2) * ROW_THREADS + (int)threadIdx.x) * 4 + (j & 3); }

// This thread's keys of a row: key j is token row_token(j) - at.shift, so that every quad is 16-byte aligned (the first may
// begin in the row before, the last end in the row behind: the caller masks tokens outside 0 .. n-1).  Every load is
// unconditional; quads behind the row's last, or behind the array's last whole one, re-read that.  Up to three words at
// the array's end are outside its whole quads and are read one by one.
template <int KPT>
__device__ __forceinline__ void row_load(const uint32_t *row, int n, RowPlace at, uint32_t (&key)[KPT])
{
    if (at.total < 4) { // (uniform) no whole quad
#pragma unroll
        for (int j = 0; j < KPT; ++j) {
            const int i = row_token(j) - at.shift;
            key[j] = i >= 0 && i < n ? row[i] : 0u;
        }
        return;
    }
    const int row_last = ((n - 1 + at.shift) & ~3) - at.shift;                       // start of the quad that ends the row
    const long long whole_end = ((at.avail + at.shift) & ~3ll) - at.shift;           // end of the array's last whole quad
    const int last = (int)min((long long)row_last, whole_end - 4);
#pragma unroll
    for (int q = 0; q < KPT / 4; ++q) {
        const uint4 a = *reinterpret_cast<const uint4 *>(row + min(row_token(4 * q) - at.shift, last));
        key[4 * q] = a.x; key[4 * q + 1] = a.y; key[4 * q + 2] = a.z; key[4 * q + 3] = a.w;
    }
    if (whole_end < n) { // uniform: the array's last row
#pragma unroll
        for (int q = 0; q < KPT / 4; ++q)
            if (row_token(4 * q) - at.shift == (int)whole_end) {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if ((int)whole_end + e < n) key[4 * q + e] = row[(int)whole_end + e];
            }
    }
}

// Where not all of the threshold's ties fit: those behind the first `fit` in token order drop below it, so that the keys at
// or above it are the chosen ones.
template <int KPT>
__device__ __forceinline__ void row_fit_ties(RowShared &sh, uint32_t (&key)[KPT], uint32_t tau, uint32_t fit, bool all_fit)
{
    constexpr int QUADS = KPT / 4, NP = (QUADS + 1) / 2;
    if (all_fit || tau == 0u) return; // uniform over the workgroup
    uint32_t cnt[NP], excl[NP], total[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) cnt[p] = 0u;
#pragma unroll
    for (int j = 0; j < KPT; ++j) cnt[j >> 3] += (key[j] == tau ? 1u : 0u) << (16 * ((j >> 2) & 1));
    row_scan<NP>(sh, cnt, excl, total);
    uint32_t before = 0u;
#pragma unroll
    for (int q = 0; q < QUADS; ++q) {
        uint32_t rank = before + ((excl[q >> 1] >> (16 * (q & 1))) & 0xFFFFu);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (key[4 * q + e] == tau) {
                if (rank >= fit) key[4 * q + e] = tau - 1u;
                ++rank;
            }
        before += (total[q >> 1] >> (16 * (q & 1))) & 0xFFFFu;
    }
}

// The row's keys from its words; 0 for the positions of the quads that lie outside tokens 0 .. n_rank - 1.
template <int KPT>
__device__ __forceinline__ void row_keys(uint32_t (&key)[KPT], int shift, int n_rank)
{
#pragma unroll
    for (int q = 0; q < KPT / 4; ++q) {
#pragma unroll
        for (int e = 0; e < 4; ++e) key[4 * q + e] = order_key(key[4 * q + e]);
        if ((q == 0 && shift) || (q + 1) * 4 * ROW_THREADS - shift > n_rank) { // uniform: not all of these are inside
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((uint32_t)(row_token(4 * q + e) - shift) >= (uint32_t)n_rank) key[4 * q + e] = 0u;
        }
    }
}

template <int KPT>
__global__ __launch_bounds__(ROW_THREADS) void select_row_kernel(SelArgs A)
{
    constexpr int QUADS = KPT / 4, NP = (QUADS + 1) / 2;
    __shared__ __attribute__((aligned(16))) RowShared sh;
    const int head = blockIdx.x;
    const uint32_t *attn = A.attn + (size_t)head * A.n, *crit = A.crit + (size_t)head * A.n;
    const RowPlace at = row_place(head, gridDim.x, A.n);
    auto token = [&](int j) { return row_token(j) - at.shift; };
    uint32_t key1[KPT], key2[KPT];
    // both rows are requested at the start; the longest rows would not fit the registers twice and take crit later
    constexpr bool LATE = KPT > 16;
    row_load<KPT>(attn, A.n, at, key1);
    if (!LATE) row_load<KPT>(crit, A.n, at, key2);
    int B, b1, b2, kept;
    head_budget(A, head, B, b1, b2, kept);
    for (int b = threadIdx.x * 4; b < SEL_BINS * 4; b += ROW_THREADS * 4) *reinterpret_cast<uint4 *>(&sh.hist[b]) = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    row_keys<KPT>(key1, at.shift, A.n_rank);
    // stage 1: chosen are the keys at or above tau1; nothing is with SEL_TAKEN, but for the kept window, which gets that key
    uint32_t tau1 = SEL_TAKEN, tau2 = SEL_TAKEN, fit;
    bool all_fit;
    if (b1 > 0) { // uniform over the workgroup, as everything derived from the budget
        row_threshold<KPT>(sh, key1, (uint32_t)b1, tau1, fit, all_fit);
        row_fit_ties<KPT>(sh, key1, tau1, fit, all_fit);
        tau1 = max(tau1, 1u); // (fewer competitors than b1: all of them)
    }
    if (kept > 0) {
#pragma unroll
        for (int j = 0; j < KPT; ++j)
            if (token(j) >= A.n - kept && token(j) < A.n) key1[j] = SEL_TAKEN;
    }
    if (LATE) row_load<KPT>(crit, A.n, at, key2);
    // the stage-2 keys with stage-1 entries marked are what the diagnostics read back
    uint32_t *k2 = A.keys2 + (size_t)head * A.n;
#pragma unroll
    for (int q = 0; q < QUADS; ++q) {
        uint32_t marked[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int j = 4 * q + e;
            const uint32_t k = order_key(key2[j]);
            const bool taken = key1[j] >= tau1;
            marked[e] = taken ? SEL_TAKEN : k;
            key2[j] = taken || key1[j] == 0u ? 0u : k; // (0 in key1: outside, or not of those that compete)
        }
        const int i0 = token(4 * q); // keys2 starts on a 16-byte boundary as the scores do: its rows are shifted alike
        if (i0 >= 0 && i0 + 3 < A.n) {
            *reinterpret_cast<uint4 *>(k2 + i0) = make_uint4(marked[0], marked[1], marked[2], marked[3]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i0 + e >= 0 && i0 + e < A.n) k2[i0 + e] = marked[e];
        }
    }
    if (b2 > 0) {
        row_threshold<KPT>(sh, key2, (uint32_t)b2, tau2, fit, all_fit);
        row_fit_ties<KPT>(sh, key2, tau2, fit, all_fit);
        tau2 = max(tau2, 1u);
    }
    // ordered write
    asm volatile("" : "+v"(tau1)); // (compared anew: kept from above, the comparisons would take more scalar registers than there are)
    uint32_t cnt[NP], excl[NP], total[NP], sel = 0u;
#pragma unroll
    for (int j = 0; j < KPT; ++j) sel |= (key1[j] >= tau1 || key2[j] >= tau2 ? 1u : 0u) << j;
#pragma unroll
    for (int p = 0; p < NP; ++p) cnt[p] = 0u;
#pragma unroll
    for (int q = 0; q < QUADS; ++q) cnt[q >> 1] += (uint32_t)__popc((sel >> (4 * q)) & 15u) << (16 * (q & 1));
    row_scan<NP>(sh, cnt, excl, total);
    int32_t *out = A.idx + (size_t)head * A.max_budget;
    uint32_t before = 0u;
#pragma unroll
    for (int q = 0; q < QUADS; ++q) {
        uint32_t pos = before + ((excl[q >> 1] >> (16 * (q & 1))) & 0xFFFFu);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if ((sel >> (4 * q + e)) & 1u) {
                if (pos < (uint32_t)A.max_budget) out[pos] = token(4 * q + e);
                ++pos;
            }
        before += (total[q >> 1] >> (16 * (q & 1))) & 0xFFFFu;
    }
    for (int j = B + (int)threadIdx.x; j < A.max_budget; j += ROW_THREADS) out[j] = -1;
    if (threadIdx.x == 0) A.count[head] = B;
}

size_t select_workspace_words(int heads, int n)
{
    const size_t n_slices = (size_t)(n + SEL_SLICE - 1) / SEL_SLICE;
    return (size_t)heads * (2 * 3 * SEL_BINS + 2 * ST_WORDS) + (size_t)heads * 3 * n_slices + (size_t)heads * n_slices * (1024 + 1025);
}

static SelArgs make_sel_args(int heads, int n, int protect, const float *attn, const float *crit, const int32_t *budget,
                             float alpha, int max_budget, int32_t *idx, int32_t *count, uint32_t *keys2, uint32_t *scratch)
{
    SelArgs A;
    A.attn = reinterpret_cast<const uint32_t *>(attn);
    A.crit = reinterpret_cast<const uint32_t *>(crit);
    A.budget = budget;
    A.keys2 = keys2;
    A.hist = scratch;
    A.state = scratch + (size_t)heads * 2 * 3 * SEL_BINS;
    A.slices = A.state + (size_t)heads * 2 * ST_WORDS;
    A.idx = idx; A.count = count;
    A.alpha = (double)alpha;
    A.n = n; A.max_budget = max_budget;
    A.n_rank = n - protect;
    A.share = 1;
    A.n_slices = (n + SEL_SLICE - 1) / SEL_SLICE;
    A.slice_hist = A.slices + (size_t)heads * 3 * A.n_slices;
    A.slice_suf = A.slice_hist + (size_t)heads * A.n_slices * 1024;
    return A;
}

// heads rows of n keys each (a row is one (batch item, kv head), or one whole batch item for the allocation)
hipError_t launch_select_rows(int heads, int n, int protect, const float *attn, const float *crit,
                              const int32_t *budget, float alpha, int max_budget, int32_t *idx, int32_t *count,
                              uint32_t *keys2, uint32_t *scratch, hipStream_t s)
{
    const int span = row_span(n);
    const SelArgs A = make_sel_args(heads, n, protect, attn, crit, budget, alpha, max_budget, idx, count, keys2, scratch);
    if (span <= SEL_ROW_MAX) {
        const dim3 grid(heads), block(ROW_THREADS);
        if (span <= 4 * ROW_THREADS) hipLaunchKernelGGL(select_row_kernel<4>, grid, block, 0, s, A);
        else if (span <= 8 * ROW_THREADS) hipLaunchKernelGGL(select_row_kernel<8>, grid, block, 0, s, A);
        else if (span <= 16 * ROW_THREADS) hipLaunchKernelGGL(select_row_kernel<16>, grid, block, 0, s, A);
        else hipLaunchKernelGGL(select_row_kernel<24>, grid, block, 0, s, A);
        return hipGetLastError();
    }
    const size_t zero_words = (size_t)heads * (2 * 3 * SEL_BINS + 2 * ST_WORDS);
    const dim3 grid(A.n_slices, heads), block(SEL_THREADS);
    hipLaunchKernelGGL(select_zero_kernel, dim3((unsigned)((zero_words + 255) / 256)), dim3(256), 0, s, scratch, zero_words);
    hipLaunchKernelGGL((select_hist_kernel<0, 0>), grid, block, 0, s, A);
    hipLaunchKernelGGL((select_hist_kernel<0, 1>), grid, block, 0, s, A);
    hipLaunchKernelGGL((select_hist_kernel<0, 2>), grid, block, 0, s, A);
    hipLaunchKernelGGL(select_mark_kernel, grid, block, 0, s, A);
    hipLaunchKernelGGL((select_hist_kernel<1, 1>), grid, block, 0, s, A);
    hipLaunchKernelGGL((select_hist_kernel<1, 2>), grid, block, 0, s, A);
    hipLaunchKernelGGL(select_write_kernel, grid, block, 0, s, A);
    return hipGetLastError();
}

hipError_t launch_select(const Dims &d, const float *attn, const float *crit, const int32_t *budget, float alpha,
                         int max_budget, int32_t *idx, int32_t *count, uint32_t *keys2, uint32_t *scratch,
                         hipStream_t s)
{
    return launch_select_rows(d.batch * d.Hkv, d.n, d.protect, attn, crit, budget, alpha, max_budget, idx, count, keys2,
                              scratch, s);
}

// ---- budget allocation across the kv heads of a batch item (Algorithm 2, line 1) -------------------------
// The P entries with the largest pooled score among all Hkv * n entries of a batch item are an order statistic of one row
// of Hkv * n keys: its threshold comes from the selection's stage-1 digits, and a head's share is the number of its
// entries above the threshold plus those of its ties that still fit (ties go to lower entries first, i.e. to lower heads).
// Only counts are needed, no membership and no index list: one launch where the row fits a workgroup, five where heads are
// about a slice long and more (clear, three digits, totals), six otherwise (clear, three digits, count, finish) -- the whole
// selection and a binary search in its list took ten (two rows of eight heads x 20011: 39.5 us in a chain of calls, now 20.6).
struct AllocArgs {
    int32_t *budget_out; // [batch][Hkv]
    uint32_t *above;     // [batch][Hkv]: entries above the threshold per head
    uint32_t *ties;      // [batch][Hkv * n] (the first Hkv words of a row are used)
    int Hkv, n, floor_each;
};

constexpr int ALLOC_MAX_HEADS = 64; // a head's workgroup also reads the slices of all heads before it

template <int KPT>
__global__ __launch_bounds__(ROW_THREADS) void allocate_row_kernel(SelArgs A, AllocArgs L)
{
    __shared__ __attribute__((aligned(16))) RowShared sh;
    const int row = blockIdx.x;
    uint32_t key[KPT];
    const RowPlace at = row_place(row, gridDim.x, A.n);
    row_load<KPT>(A.attn + (size_t)row * A.n, A.n, at, key);
    for (int b = threadIdx.x * 4; b < SEL_BINS * 4; b += ROW_THREADS * 4) *reinterpret_cast<uint4 *>(&sh.hist[b]) = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    row_keys<KPT>(key, at.shift, A.n);
    uint32_t tau, fit, sel = 0u;
    bool all_fit;
    row_threshold<KPT>(sh, key, (uint32_t)A.max_budget, tau, fit, all_fit);
    row_fit_ties<KPT>(sh, key, tau, fit, all_fit);
#pragma unroll
    for (int j = 0; j < KPT; ++j) sel |= (key[j] >= max(tau, 1u) ? 1u : 0u) << j;
    // the histogram is clear again: its words count the heads' entries (the host takes this kernel for Hkv <= 4 * SEL_BINS)
    __syncthreads();
#pragma unroll
    for (int q = 0; q < KPT / 4; ++q) {
        int g_run = -1;
        uint32_t run = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (!((sel >> (4 * q + e)) & 1u)) continue;
            const int g = (row_token(4 * q + e) - at.shift) / L.n;
            if (g != g_run && run) { atomicAdd(&sh.hist[g_run], run); run = 0u; }
            g_run = g;
            ++run;
        }
        if (run) atomicAdd(&sh.hist[g_run], run);
    }
    __syncthreads();
    for (int g = threadIdx.x; g < L.Hkv; g += ROW_THREADS)
        L.budget_out[(size_t)row * L.Hkv + g] = min(L.n, L.floor_each + (int)sh.hist[g]);
}

__global__ __launch_bounds__(256) void allocate_clear_kernel(uint32_t *hist, size_t words, AllocArgs L, int batch)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < words) hist[i] = 0u;
    if (i < (size_t)batch * L.Hkv) {
        L.above[i] = 0u;
        L.ties[i / L.Hkv * ((size_t)L.Hkv * L.n) + i % L.Hkv] = 0u;
    }
}

// One workgroup per slice of the row: its entries above the threshold and its ties, added to their heads' counts.
__global__ __launch_bounds__(SEL_THREADS) void allocate_count_kernel(SelArgs A, AllocArgs L)
{
    __shared__ SelShared sh;
    __shared__ uint32_t cnt[2][SEL_SLICE]; // above / ties of the heads this slice touches (at most one per token)
    const int slice = blockIdx.x, row = blockIdx.y;
    const int i0 = slice * SEL_SLICE + threadIdx.x * SEL_PER_THREAD;
    uint32_t w[8];
    load8(A.attn + (size_t)row * A.n, i0, A.n, row_place(row, gridDim.y, A.n), w);
    const uint32_t *st = A.state + (size_t)row * 2 * ST_WORDS;
    const uint32_t d0 = st[ST_D0], a0 = st[ST_A0], d1 = st[ST_D1], a1 = st[ST_A1];
    uint32_t d2, a2;
    find_digit(sh, A.hist + (size_t)row * 2 * 3 * SEL_BINS + 2 * SEL_BINS, 1024, (uint32_t)A.max_budget - a0 - a1, d2, a2);
    const uint32_t tau = (d0 << DSHIFT0) | (d1 << DSHIFT1) | d2, fit = (uint32_t)A.max_budget - a0 - a1 - a2;
    const int g0 = slice * SEL_SLICE / L.n, g1 = min(slice * SEL_SLICE + SEL_SLICE - 1, A.n - 1) / L.n;
    for (int g = threadIdx.x; g <= g1 - g0; g += SEL_THREADS) { cnt[0][g] = 0u; cnt[1][g] = 0u; }
    __syncthreads();
    uint32_t *above = L.above + (size_t)row * L.Hkv, *ties = L.ties + (size_t)row * A.n;
    if (g0 == g1) { // uniform: the slice lies inside one head
        uint32_t n_above = 0u, n_ties = 0u;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t key = order_key(w[j]);
            n_above += i0 + j < A.n && key > tau ? 1u : 0u;
            n_ties += i0 + j < A.n && key == tau ? 1u : 0u;
        }
        const uint32_t both = block_sum(sh, n_above | (n_ties << 16)); // 2048 of either at most
        if (threadIdx.x == 0) { cnt[0][0] = both & 0xFFFFu; cnt[1][0] = both >> 16; }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t key = order_key(w[j]);
            if (i0 + j < A.n && key >= tau) atomicAdd(&cnt[key == tau ? 1 : 0][(i0 + j) / L.n - g0], 1u);
        }
    }
    __syncthreads();
    for (int g = threadIdx.x; g <= g1 - g0; g += SEL_THREADS) {
        if (cnt[0][g]) atomicAdd(above + g0 + g, cnt[0][g]);
        if (cnt[1][g]) atomicAdd(ties + g0 + g, cnt[1][g]);
    }
    if (slice == 0 && threadIdx.x == 0) A.state[(size_t)row * 2 * ST_WORDS + ST_R] = fit;
}

// One workgroup per row: the heads' counts become budgets.  A launch of its own, and no ticket that lets the last workgroup
// of the count kernel do it: that needs a release by every wave that counted, and the write-backs of L2 these cost grow with
// the launch (the whole allocation, us, with one release per workgroup / like this: 64 rows of 8 heads x 8000 110 / 56, one
// of 8 x 131072 55 / 45, two of 8 x 20011 24.9 / 23.2; the line to the kernel above lies where launch_allocate draws it).
__global__ __launch_bounds__(SEL_THREADS) void allocate_finish_kernel(SelArgs A, AllocArgs L)
{
    __shared__ SelShared sh;
    const int row = blockIdx.x;
    const uint32_t *above = L.above + (size_t)row * L.Hkv, *ties = L.ties + (size_t)row * A.n;
    const uint32_t fit = A.state[(size_t)row * 2 * ST_WORDS + ST_R];
    uint32_t carry = 0u;
    for (int c0 = 0; c0 < L.Hkv; c0 += SEL_THREADS) { // heads in order: how many ties lie before each
        const int g = c0 + threadIdx.x;
        const uint32_t a = g < L.Hkv ? above[g] : 0u, t = g < L.Hkv ? ties[g] : 0u;
        uint32_t total;
        const uint32_t before = carry + block_exclusive_scan(sh, t, total);
        if (g < L.Hkv)
            L.budget_out[(size_t)row * L.Hkv + g] = min(L.n, L.floor_each + (int)(a + min(fit > before ? fit - before : 0u, t)));
        carry += total;
    }
}

// The same from counts that the histogram kernels kept per slice of every head (slices do not cross heads there): one
// workgroup per head adds up its slices' entries above the threshold and the ties before and inside it.
__global__ __launch_bounds__(SEL_THREADS) void allocate_total_kernel(SelArgs A, AllocArgs L)
{
    __shared__ SelShared sh;
    const int g = blockIdx.x, row = blockIdx.y, ns = A.n_slices;
    const uint32_t *st = A.state + (size_t)row * 2 * ST_WORDS;
    const uint32_t d0_above = st[ST_A0], d1_above = st[ST_A1];
    uint32_t d2, a2;
    find_digit(sh, A.hist + (size_t)row * 2 * 3 * SEL_BINS + 2 * SEL_BINS, 1024, (uint32_t)A.max_budget - d0_above - d1_above, d2, a2);
    const uint32_t fit = (uint32_t)A.max_budget - d0_above - d1_above - a2;
    const size_t first = (size_t)row * L.Hkv; // the batch item's first head
    uint32_t before = 0u, above = 0u, ties = 0u;
    for (int s = threadIdx.x; s < (g + 1) * ns; s += SEL_THREADS) {
        const size_t head = first + s / ns;
        const int slice = s % ns;
        const uint32_t *suf = A.slice_suf + (head * ns + slice) * 1025 + d2;
        const uint32_t gt = suf[1], t = suf[0] - gt;
        if (s >= g * ns) {
            const uint32_t *sl = A.slices + head * 3 * ns + slice;
            above += sl[ns] + sl[2 * ns] + gt;
            ties += t;
        } else {
            before += t;
        }
    }
    before = block_sum(sh, before);
    above = block_sum(sh, above);
    ties = block_sum(sh, ties);
    if (threadIdx.x == 0)
        L.budget_out[first + g] = min(L.n, L.floor_each + (int)(above + min(fit > before ? fit - before : 0u, ties)));
}

__global__ void allocate_floor_kernel(AllocArgs L, int heads)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < heads) L.budget_out[i] = min(L.n, L.floor_each);
}

hipError_t launch_allocate(const Dims &d, const float *attn, int total, float floor_frac, int32_t *budget_out,
                           uint32_t *keys2, uint32_t *scratch, int32_t *tmp, hipStream_t s)
{
    const int floor_each = (int)floor((double)floor_frac * (double)total / (double)d.Hkv);
    const int P = (int)min((long long)total - (long long)d.Hkv * floor_each, (long long)d.Hkv * d.n);
    AllocArgs L;
    L.budget_out = budget_out;
    L.above = (uint32_t *)tmp; // batch * Hkv of the batch * (2 + Hkv * ceil(P / Hkv)) words that are there when P > 0
    L.ties = keys2;
    L.Hkv = d.Hkv; L.n = d.n; L.floor_each = floor_each;
    if (P <= 0) {
        const int heads = d.batch * d.Hkv;
        hipLaunchKernelGGL(allocate_floor_kernel, dim3((heads + 255) / 256), dim3(256), 0, s, L, heads);
        return hipGetLastError();
    }
    const int N = d.Hkv * d.n;
    const SelArgs A = make_sel_args(d.batch, N, 0, attn, attn, nullptr, 1.0f, P, nullptr, nullptr, keys2, scratch);
    const int span = row_span(N);
    if (span <= SEL_ROW_MAX && d.Hkv <= 4 * SEL_BINS) {
        const dim3 grid(d.batch), block(ROW_THREADS);
        if (span <= 4 * ROW_THREADS) hipLaunchKernelGGL(allocate_row_kernel<4>, grid, block, 0, s, A, L);
        else if (span <= 8 * ROW_THREADS) hipLaunchKernelGGL(allocate_row_kernel<8>, grid, block, 0, s, A, L);
        else if (span <= 16 * ROW_THREADS) hipLaunchKernelGGL(allocate_row_kernel<16>, grid, block, 0, s, A, L);
        else hipLaunchKernelGGL(allocate_row_kernel<24>, grid, block, 0, s, A, L);
        return hipGetLastError();
    }
    // Heads of about a slice and more: slices of single heads, whose counts the histogram kernels keep, and five launches;
    // shorter ones share slices and are counted in a launch of their own.  us, launch of its own / kept
    // counts: 16 heads x 20011 in two rows 23.3 / 20.6, 8 x 131072 39.3 / 33.1, 64 rows of 8 x 8000 47.4 / 42.0, 24 x 1100 19.8 /
    // 19.5, 40 x 5000 22.4 / 21.7, 256 x 1024 22.9 / 24.3.
    if (d.n >= SEL_SLICE / 2 && d.Hkv <= ALLOC_MAX_HEADS) {
        SelArgs S = make_sel_args(d.batch * d.Hkv, d.n, 0, attn, attn, nullptr, 1.0f, P, nullptr, nullptr, keys2, scratch);
        S.share = d.Hkv;
        const size_t words = (size_t)d.batch * 2 * 3 * SEL_BINS;
        const dim3 slices(S.n_slices, d.batch * d.Hkv), threads(SEL_THREADS);
        hipLaunchKernelGGL(select_zero_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, scratch, words);
        hipLaunchKernelGGL((select_hist_kernel<0, 0, true>), slices, threads, 0, s, S);
        hipLaunchKernelGGL((select_hist_kernel<0, 1, true>), slices, threads, 0, s, S);
        hipLaunchKernelGGL((select_hist_kernel<0, 2, true>), slices, threads, 0, s, S);
        hipLaunchKernelGGL(allocate_total_kernel, dim3(d.Hkv, d.batch), threads, 0, s, S, L);
        return hipGetLastError();
    }
    const size_t hist_words = (size_t)d.batch * (2 * 3 * SEL_BINS + 2 * ST_WORDS);
    const size_t clear = std::max(hist_words, (size_t)d.batch * d.Hkv);
    const dim3 grid(A.n_slices, d.batch), block(SEL_THREADS);
    hipLaunchKernelGGL(allocate_clear_kernel, dim3((unsigned)((clear + 255) / 256)), dim3(256), 0, s, scratch, hist_words, L, d.batch);
    hipLaunchKernelGGL((select_hist_kernel<0, 0>), grid, block, 0, s, A);
    hipLaunchKernelGGL((select_hist_kernel<0, 1>), grid, block, 0, s, A);
    hipLaunchKernelGGL((select_hist_kernel<0, 2>), grid, block, 0, s, A);
    hipLaunchKernelGGL(allocate_count_kernel, grid, block, 0, s, A, L);
    hipLaunchKernelGGL(allocate_finish_kernel, dim3(d.batch), block, 0, s, A, L);
    return hipGetLastError();
}

} // namespace ckv
