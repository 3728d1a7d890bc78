// Exact per-tensor selection on ordered entries: sources, window / radix passes, ordered
// emission ("encode()" of Algorithms 1-3) with the state fix-up of Eq. 12 / Eq. 6, and the
// threshold hints.  Shared by the single-workgroup selection and the segmented chain.
#pragma once
#include "dgs_wave.h"

namespace dgs {

// ---------------------------------------------------------------------------
// select
// ---------------------------------------------------------------------------

// The value the selection ranks at flat index ix, read from the buffers themselves
// (dense sources, zero fill): the state / difference row, or model - sent_k.  WRITTEN: another workgroup
// of this launch may have stored the worker's state.
template <int OP, bool WRITTEN = false>
__device__ __forceinline__ float row_value(const float *state, const float *model, uint32_t ix)
{
    if (WRITTEN && OP == SEL_WORKER) return __uint_as_float(ld_dev((const uint32_t *)state + ix));
    return (OP == SEL_PULL_V) ? (model[ix] - state[ix]) : state[ix];
}

// What a sent entry leaves behind: worker m * a (Eq. 12, state stored as m u); pull on a
// difference row +0 (Eq. 6 as D_k -= G); pull on model - sent_k: sent_k += G (Eq. 6).
template <int OP>
__device__ __forceinline__ void fix_sent(float *state, uint32_t ix, float val, float m, bool later = false)
{
    if (OP == SEL_PULL_V && later) return;
    if (OP == SEL_WORKER) store_scattered(&state[ix], m * val);
    else if (OP == SEL_PULL) store_scattered(&state[ix], 0.0f);
    else store_scattered(&state[ix], state[ix] + val);
}

// An index that came out of a candidate list is used as an address: one outside the buffer
// (a corrupted list) is counted as an internal error and never dereferenced.
__device__ __forceinline__ bool index_ok(const SelectArgs &A, uint32_t ix)
{
    if (ix < A.n) return true;
    atomicAdd(&A.stats->internal_errors, 1ull);
    return false;
}

template <int OP, bool WRITTEN>
struct SrcDense {          // the tensor itself: position p <-> element off + p
    static constexpr bool AGG = false;
    const float *base;
    const float *model;
    uint32_t off;
    __device__ __forceinline__ uint32_t bits(uint32_t p) const
    {
        return __float_as_uint(row_value<OP, WRITTEN>(base, model, off + p));
    }
    __device__ __forceinline__ uint32_t index(uint32_t p) const { return off + p; }
};

struct SrcDenseLds {       // a small tensor staged in LDS: position p <-> element off + p
    static constexpr bool AGG = false;
    const uint32_t *v;
    uint32_t off;
    __device__ __forceinline__ uint32_t bits(uint32_t p) const { return v[p]; }
    __device__ __forceinline__ uint32_t index(uint32_t p) const { return off + p; }
};

struct SrcList {           // ordered candidates (index, value bits)
    static constexpr bool AGG = true;   // candidates share their top key bits: merge per wavefront
    const uint2 *list;
    __device__ __forceinline__ uint32_t bits(uint32_t p) const { return list[p].y; }
    __device__ __forceinline__ uint32_t index(uint32_t p) const { return list[p].x; }
};

struct SrcSplit {          // a list whose first SEL_LDS_LIST entries are in LDS, the rest in global scratch
    static constexpr bool AGG = true;
    const uint2 *llist;
    const uint2 *glist;
    __device__ __forceinline__ uint2 get(uint32_t p) const { return (p < SEL_LDS_LIST) ? llist[p] : glist[p]; }
    __device__ __forceinline__ uint32_t bits(uint32_t p) const { return get(p).y; }
    __device__ __forceinline__ uint32_t index(uint32_t p) const { return get(p).x; }
};

// The four consecutive elements e0 .. e0 + 3 (e0 a multiple of 4) of the ranked row as bit
// patterns, and which of them belong to the tensor [lo, hi): one 16-byte load per buffer where
// the quad lies inside the tensor, element by element at a tensor border.
// (All lanes of a wavefront call together, in the same tile.)
template <int OP, bool WRITTEN = false>
__device__ __forceinline__ uint32_t quad_bits(const SelectArgs &A, uint32_t e0, uint32_t lo, uint32_t hi,
                                              uint32_t (&bits)[4])
{
    const uint32_t base = (WRITTEN && OP == SEL_WORKER) ? uniform(e0 / TILE * TILE) : 0u;
    if (e0 >= lo && e0 + 3u < hi) {
        f32x4 v;
        if (WRITTEN && OP == SEL_WORKER) {
            v = load_through16(A.state + base, (e0 - base) * 4u);
        } else {
            v = *(const f32x4_any *)(A.state + e0);
        }
        if (OP == SEL_PULL_V) v = *(const f32x4_any *)(A.model + e0) - v;      // one fp32 subtraction per element
        bits[0] = __float_as_uint(v.x);
        bits[1] = __float_as_uint(v.y);
        bits[2] = __float_as_uint(v.z);
        bits[3] = __float_as_uint(v.w);
        return 0xFu;
    }
    uint32_t in = 0;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const uint32_t e = e0 + x;
        const bool ok = e >= lo && e < hi;
        bits[x] = ok ? __float_as_uint(row_value<OP, WRITTEN>(A.state, A.model, e)) : 0u;
        in |= ok ? (1u << x) : 0u;
    }
    return in;
}

// Candidate p of tile t.
__device__ __forceinline__ const uint2 *candidate(const SelectArgs &A, uint32_t t, uint32_t p)
{
    const uint32_t far = A.far0 + t * (CAPT - NEAR) + (p - NEAR), near = A.near0 + t * (NEAR - HEAD) + (p - HEAD);
    return A.heads + ((p < HEAD) ? t * HEAD + p : (p < NEAR ? near : far));      // (below 2^31: at most 2^22 tiles)
}

// What a tile's counter word says about tensor td's candidates in tile t: how many, and after
// how many of the previous tensor's (a first tile shared with it).  An overflowed tile, or a
// count beyond the slots (a corrupted word), sets ovf and counts as empty.
__device__ __forceinline__ void tile_counts(uint32_t w, uint32_t t, uint32_t tlo, bool head_shared, uint32_t &n_t,
                                            uint32_t &start, int &ovf)
{
    n_t = 0;
    start = 0;
    if (w == CNT_OVERFLOW) {
        ovf = 1;
    } else if (head_shared && t == tlo) {
        start = w & 0xFFFFu;      // the previous tensor's candidates come first in this tile
        n_t = w >> 16;
    } else {
        n_t = w & 0xFFFFu;
    }
    if (start + n_t > CAPT) {
        ovf = 1;
        n_t = 0;
        start = 0;
    }
}

// First bin (key >> SEG_LOWBITS) of the window histogram of a tensor that takes the chain.
// Candidates start at the collection threshold; when that lies far below the k-th key of the
// previous selection on this stream (a relaxed hint), the window is centred on that key
// instead, so that it reaches half an octave to either side of it.  Keys below the window are
// counted into bin 0, which then holds no usable rank.
__device__ __forceinline__ uint32_t seg_window_base(uint32_t tau_cur, uint32_t t_prev)
{
    const uint32_t b_tau = tau_cur >> SEG_LOWBITS;
    const uint32_t b_prev = t_prev >> SEG_LOWBITS;
    const uint32_t b_mid = (b_prev > SEG_WBINS / 2) ? (b_prev - SEG_WBINS / 2) : 0u;
    return max(b_tau, b_mid);
}

// Window histogram of part `sidx` of a tensor that takes the chain: in the ordered-list scratch of
// the tensor, which holds nothing until a failed prediction is collected again.  A part of at
// least SEG_TILES tiles (or the only one of at least 64) has room for the SEG_WBINS counters, the
// shorter last part uses what the others leave.
__device__ __forceinline__ uint32_t *part_hist(const SelectArgs &A, const TensorDesc &td, uint32_t j, uint32_t sidx)
{
    return (uint32_t *)(A.ord + (size_t)(td.off / TILE + j) * CAPT) + (size_t)sidx * SEG_WBINS;
}
static_assert(SEG_MIN_N / TILE * 2 * CAPT >= (SEG_MIN_N / TILE / SEG_TILES + 2) * SEG_WBINS, "part histograms fit");

// Window histogram of a list that one workgroup selects from: WIN_BINS buckets of key >> win_shift(op), which
// leaves that many low bits for a second histogram.  Half an octave for the worker, whose k-th key moves little
// from step to step; an octave for a pull: with half an octave the k-th key of a server's row that had
// waited long lay beyond the window, which costs three more passes over the list, 8 to 12 us (mean of the
// selection in the three server forms of 32 and 6 workers 28.5 -> 24.7, 29.7 -> 26.0, 31.8 -> 26.3 us;
// the wider second histogram costs 0.3 us where the window had served: a round on ResNet-50 shapes).
constexpr uint32_t WIN_BINS = 2048;
constexpr __host__ __device__ uint32_t win_shift(int op) { return op == SEL_WORKER ? 11u : 12u; }

// Its first bucket: the collection threshold or, when that lies far below (a relaxed hint), 1024 buckets
// under the previous k-th key.
template <int OP>
__device__ __forceinline__ uint32_t win_base_of(uint32_t tau_cur, uint32_t t_prev)
{
    return max(tau_cur >> win_shift(OP), max(t_prev >> win_shift(OP), WIN_BINS / 2) - WIN_BINS / 2);
}

constexpr uint32_t FEW = 256;

struct SelShared {
    alignas(16) uint32_t h[4096];      // (the join keeps its tiles in the upper half)
    uint32_t wsum[SEL_WAVES];
    uint32_t rowsum[64];
    int res[6];
    uint32_t kmin;
    uint32_t few, few_key[FEW], few_res[2];      // the keys that share the prefix of the k-th one, where they are few, and its rank
};

// Count into an LDS histogram.  With AGG (all 64 lanes must call this together), the
// lanes that hit the same bin as the first valid lane are merged into one atomic --
// candidate keys mostly share their top bits -- and the others add on their own.
template <bool AGG>
__device__ __forceinline__ void hist_add(uint32_t *h, uint32_t bin, bool valid)
{
    if (!AGG) {
        if (valid) atomicAdd(&h[bin], 1u);
        return;
    }
    const uint64_t todo = ballot64(valid);
    if (todo == 0) return;
    const int leader = __ffsll((unsigned long long)todo) - 1;
    const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)bin, leader);
    const uint64_t same = ballot64(valid && bin == b0);
    if ((int)lane_id() == leader) atomicAdd(&h[b0], (uint32_t)__popcll(same));
    else if (valid && bin != b0) atomicAdd(&h[bin], 1u);
}

// Window histogram of candidate keys: bucket (key >> win_shift(OP)) - win_base, everything at or
// below the base in bucket 0, everything beyond the window in the last one.
template <int OP>
__device__ __forceinline__ void window_count(uint32_t *h, uint32_t win_base, uint32_t key)
{
    const uint32_t hi = key >> win_shift(OP);
    const uint32_t w = (hi > win_base) ? (hi - win_base) : 0u;
    atomicAdd(&h[min(w, WIN_BINS - 1u)], 1u);
}

// Next threshold when fewer candidates (c) than the hinted rank R were collected, all at
// or above `kmin`: the lowest q of them span `width` keys; the same density is assumed
// below kmin (it is higher in fact, so this errs towards more candidates), with half as
// much again for safety, and never below half of the smallest candidate key.
__device__ __forceinline__ uint32_t hint_extrapolated(uint32_t kmin, uint32_t c, uint32_t R, uint32_t q,
                                                      uint32_t width)
{
    const float delta = 1.5f * (float)(R - c) * (float)width / (float)max(q, 1u);
    uint32_t tn = (delta < (float)kmin) ? (kmin - (uint32_t)delta) : 1u;
    if (kmin < 0x7F800000u) {
        const uint32_t half = __float_as_uint(__uint_as_float(kmin) * 0.5f) & 0x7FFFFFFFu;
        tn = max(tn, half);
    }
    return max(tn, 1u);
}

// The key of rank r2 (from the top) among the `sharing` keys in S.few_key, FEW at most, which differ in their `shift` low bits: those
// bits, and the rank among the keys equal to it.  One wavefront works it out for all; called behind the barrier that
// follows the last entry, and ends with one.
__device__ __forceinline__ void rank_few(SelShared &S, uint32_t sharing, uint32_t r2, uint32_t shift, uint32_t &low, uint32_t &rT)
{
    if (uniform(threadIdx.x >> 6) == 0) {
        const uint32_t lane = lane_id(), mask = (1u << shift) - 1u;
        const uint32_t mine = (lane < sharing) ? S.few_key[lane] & mask : 0u;
        uint32_t l = 0, r = 0;
        {
            uint32_t more[FEW / 64 - 1];
#pragma unroll
            for (uint32_t i = 0; i < FEW / 64 - 1; ++i) more[i] = (64u * (i + 1u) + lane < sharing) ? S.few_key[64u * (i + 1u) + lane] & mask : 0u;
            auto reach = [&](uint32_t bound) {      // how many are `bound` or more
                uint32_t m = (uint32_t)__popcll(ballot64(lane < sharing && mine >= bound));
                if (sharing > 64u) {
#pragma unroll
                    for (uint32_t i = 0; i < FEW / 64 - 1; ++i) m += (uint32_t)__popcll(ballot64(64u * (i + 1u) + lane < sharing && more[i] >= bound));
                }
                return m;
            };
#pragma unroll 1
            for (uint32_t bit = 1u << (shift - 1u); bit != 0; bit >>= 1)
                if (reach(l | bit) >= r2) l |= bit;      // (kept while at least r2 keys have it)
            r = r2 - reach(l + 1u);
        }
        if (lane == 0) {
            S.few_res[0] = l;
            S.few_res[1] = r;
        }
    }
    __syncthreads();
    low = S.few_res[0];
    rT = S.few_res[1];
}

// The next threshold as a window histogram shows it: its ranks R (bR, rR) and `third` (bE), see select_key.  lo: the first
// bucket that may hold a result.
template <int OP>
__device__ __forceinline__ void window_hint(const uint32_t *h, uint32_t base, int lo, int bR, uint32_t rR, int bE, bool measurable,
                                            uint32_t R, uint32_t cN, uint32_t qlow, uint32_t kmin, uint32_t *tau_next,
                                            uint32_t *expect, uint32_t *q_e)
{
    constexpr uint32_t SHIFT = win_shift(OP);
    if (measurable) {
        const uint32_t edge = (base + (uint32_t)bR) << SHIFT;
        *tau_next = edge ? edge : 1u;
        *expect = R - rR + h[bR];
        if (bE >= lo && bE < (int)WIN_BINS - 1) *q_e = (base + (uint32_t)bE) << SHIFT;
    } else if (R != 0 && bE >= lo && bE < (int)WIN_BINS - 1) {
        const uint32_t top = (base + (uint32_t)bE + 1u) << SHIFT;   // the lowest quarter ends below it
        *tau_next = hint_extrapolated(max(kmin, 1u), cN, R, qlow, top - min(kmin, top - 1u));
        *expect = R;
    }
}

// The k-th key of the `cN` ordered entries of `src` (T), and how many of the entries equal to it are taken
// (rT).  If R != 0 and R <= cN, also finds a key
// prefix of the entry of rank R -- 31 - win_shift(OP) bits where the window resolved
// it, 21 from the passes without one: *tau_next = its lower edge (>= 1) and
// *expect = how many entries lie at or above that edge; otherwise both 0.
// Candidate lists come with a window: win_base = first bucket (key >> win_shift(OP)), 0xFFFFFFFF for
// other sources; win_min = 1 if entries may lie below the base (bucket 0 is then mixed and
// cannot hold a result), else 0; win_ready: S.h already holds the window histogram of the
// entries (window_count); kmin = smallest key of the list.  With a window, R and Eq need be known to the first three
// wavefronts only, and what they lead to is thread 0's.  Returns whether it was found (it is, for cN >= k).
template <int OP, class Src>
__device__ __forceinline__ bool select_key(const Src src, const uint32_t cN, const uint32_t k,
                                           uint32_t R, const uint32_t Eq, const uint32_t win_base,
                                           const uint32_t win_min, const bool win_ready, const uint32_t kmin,
                                           SelShared &S, const SelectArgs &A, uint32_t *tau_next, uint32_t *expect,
                                           uint32_t *q_e, uint32_t &T, uint32_t &rT)
{
    const uint32_t tid = threadIdx.x;
    bool measurable = (R != 0) && (cN >= R);
    *tau_next = 0;
    *expect = 0;
    *q_e = 0;

    uint32_t pfx = 0;        // key prefix of the k-th entry, `lowbits` bits still unresolved
    uint32_t r2 = 0;         // its rank among the entries sharing that prefix
    uint32_t lowbits = 10;
    constexpr uint32_t SHIFT = win_shift(OP), LOW_BINS = Src::AGG ? (1u << SHIFT) : 2048u;
    static_assert(LOW_BINS <= sizeof(S.h) / 4, "low bits of a bucket");
    bool have_prefix = false;

    // ---- candidate lists: every key is >= the collection threshold, and the k-th key
    //      normally lies within a factor 1.4 (worker) or 2 of it, or close to the previous call's.
    //      One pass over a window of 2047 buckets (bucket 2047 = everything beyond) resolves all
    //      but SHIFT key bits at once.  A window that was placed by those hints
    //      and missed the k-th key is tried once more from the smallest key of the list.
    if (Src::AGG && win_base != 0xFFFFFFFFu) {
        uint32_t base = win_base, bmin = win_min;
        bool counted = win_ready;
        for (int attempt = 0; attempt < 2; ++attempt) {
            if (!counted) {   // otherwise the caller has counted the entries while it built the list
                for (uint32_t b = tid; b < WIN_BINS; b += SEL_THREADS) S.h[b] = 0;
                __syncthreads();
                for (uint32_t pb = 0; pb < cN; pb += 4 * SEL_THREADS) {
                    uint32_t kk[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t p = pb + i * SEL_THREADS + tid;
                        kk[i] = (p < cN) ? (src.bits(p) & 0x7FFFFFFFu) : 0u;
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (pb + i * SEL_THREADS + tid < cN) window_count<OP>(S.h, base, kk[i]);
                }
            }
            // third rank: the drift quantile if R is among the candidates; otherwise the entry
            // below which the lowest quarter of the candidates lies (for the extrapolated hint)
            const uint32_t qlow = max(cN / 4u, min(cN, 16u));
            const uint32_t third = measurable ? ((Eq <= cN) ? Eq : 0u) : ((R != 0) ? (cN - qlow + 1u) : 0u);
            find_ranks<WIN_BINS, SEL_WAVES>(S.h, k, measurable ? R : k, third, S.rowsum, S.res);
            const int bk = S.res[0], bR = S.res[2], bE = S.res[4];
            const uint32_t rk = (uint32_t)S.res[1], rR = (uint32_t)S.res[3];
            const int lo = (int)bmin;
            if (bk >= lo && bk < (int)WIN_BINS - 1 && bR >= lo && bR < (int)WIN_BINS - 1) {
                have_prefix = true;
                pfx = base + (uint32_t)bk;
                r2 = rk;
                lowbits = SHIFT;
                if (tid == 0)
                    window_hint<OP>(S.h, base, lo, bR, rR, bE, measurable, R, cN, qlow, kmin, tau_next, expect, q_e);
            }
            __syncthreads();
            if (have_prefix || base == (kmin >> SHIFT)) break;
            base = kmin >> SHIFT;
            bmin = 0;
            counted = false;
        }
    }

    if (!have_prefix) {
        if (Src::AGG && win_base != 0xFFFFFFFFu) {      // (R is known to the wavefronts that search only)
            if (tid == 0) S.kmin = R;
            __syncthreads();
            R = S.kmin;
            measurable = (R != 0) && (cN >= R);
        }
        // ---- pass 1: key bits [30:20]
        for (uint32_t b = tid; b < 2048; b += SEL_THREADS) S.h[b] = 0;
        __syncthreads();
        for (uint32_t pb = 0; pb < cN; pb += 4 * SEL_THREADS) {
            uint32_t kk[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t p = pb + i * SEL_THREADS + tid;
                kk[i] = (p < cN) ? (src.bits(p) & 0x7FFFFFFFu) : 0u;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                hist_add<Src::AGG>(S.h, kk[i] >> 20, pb + i * SEL_THREADS + tid < cN);
        }
        find_ranks<2048, SEL_WAVES>(S.h, k, measurable ? R : k, 0u, S.rowsum, S.res);
        const int b1 = S.res[0];
        const uint32_t r1 = (uint32_t)S.res[1];
        const int c1 = S.res[2];
        const uint32_t q1 = (uint32_t)S.res[3];
        __syncthreads();
        if (b1 < 0 || c1 < 0) {   // cannot happen for cN >= k
            if (tid == 0) atomicAdd(&A.stats->internal_errors, 1ull);
            return false;
        }

        // ---- pass 2: key bits [19:10] inside bucket b1 (and inside c1 for the hint)
        const bool two = measurable && (c1 != b1);
        for (uint32_t b = tid; b < 2048; b += SEL_THREADS) S.h[b] = 0;
        __syncthreads();
        for (uint32_t pb = 0; pb < cN; pb += 4 * SEL_THREADS) {
            uint32_t kk[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t p = pb + i * SEL_THREADS + tid;
                kk[i] = (p < cN) ? (src.bits(p) & 0x7FFFFFFFu) : 0xFFFFFFFFu;   // top bits match no bucket
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int top = (int)(kk[i] >> 20);
                if (top == b1) atomicAdd(&S.h[(kk[i] >> 10) & 1023u], 1u);
                else if (two && top == c1) atomicAdd(&S.h[1024u + ((kk[i] >> 10) & 1023u)], 1u);
            }
        }
        find_ranks<1024, SEL_WAVES>(S.h, r1, (measurable && !two) ? q1 : r1, 0u, S.rowsum, S.res);
        const int b2 = S.res[0];
        r2 = (uint32_t)S.res[1];
        int c2 = S.res[2];
        uint32_t q2 = (uint32_t)S.res[3];
        __syncthreads();
        if (two) {
            find_ranks<1024, SEL_WAVES>(S.h + 1024, q1, 0u, 0u, S.rowsum, S.res);
            c2 = S.res[0];
            q2 = (uint32_t)S.res[1];
            __syncthreads();
        }
        if (measurable && c2 >= 0) {
            const uint32_t edge = ((uint32_t)c1 << 20) | ((uint32_t)c2 << 10);
            *tau_next = edge ? edge : 1u;
            *expect = R - q2 + S.h[(two ? 1024 : 0) + c2];
        }
        if (b2 < 0) {
            if (tid == 0) atomicAdd(&A.stats->internal_errors, 1ull);
            return false;
        }
        pfx = ((uint32_t)b1 << 10) | (uint32_t)b2;
        lowbits = 10;
        __syncthreads();
    }

    // ---- last pass: the low key bits among the entries sharing the prefix
    const uint32_t lowmask = (1u << lowbits) - 1u;
    for (uint32_t b = tid; b < LOW_BINS; b += SEL_THREADS) S.h[b] = 0;
    __syncthreads();
    for (uint32_t pb = 0; pb < cN; pb += 4 * SEL_THREADS) {
        uint32_t kk[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t p = pb + i * SEL_THREADS + tid;
            kk[i] = (p < cN) ? (src.bits(p) & 0x7FFFFFFFu) : 0xFFFFFFFFu;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if ((kk[i] >> lowbits) == pfx) atomicAdd(&S.h[kk[i] & lowmask], 1u);
    }
    find_ranks<(int)LOW_BINS, SEL_WAVES>(S.h, r2, 0u, 0u, S.rowsum, S.res);
    const int b3 = S.res[0];
    rT = (uint32_t)S.res[1];
    __syncthreads();
    if (b3 < 0) {
        if (tid == 0) atomicAdd(&A.stats->internal_errors, 1ull);
        return false;
    }
    T = (pfx << lowbits) | (uint32_t)b3;
    return true;
}

// Exact selection: emits the k winners in order and applies the state fix-up.
template <int OP, int ITEMS, class Src>
__device__ __forceinline__ void select_emit(const Src src, const uint32_t cN, const uint32_t k,
                                            const uint32_t R, const uint32_t Eq, const uint32_t win_base,
                                            const uint32_t win_min, const bool win_ready, const uint32_t kmin,
                                            SelShared &S, const SelectArgs &A, const uint32_t outoff,
                                            uint32_t *tau_next, uint32_t *expect, uint32_t *q_e,
                                            uint32_t *t_out)
{
    const uint32_t tid = threadIdx.x;
    uint32_t T, rT;      // (ties: lowest index first)
    if (!select_key<OP>(src, cN, k, R, Eq, win_base, win_min, win_ready, kmin, S, A, tau_next, expect, q_e, T, rT)) return;
    *t_out = T;

    // ---- ordered emission
    uint32_t run_sel = 0, run_eq = 0;
    constexpr uint32_t CHUNK = SEL_THREADS * ITEMS;
    for (uint32_t cb = 0; cb < cN; cb += CHUNK) {
        const uint32_t p0 = cb + tid * ITEMS;
        uint32_t vb[ITEMS];
        uint32_t g = 0, q = 0;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t p = p0 + i;
            vb[i] = (p < cN) ? src.bits(p) : 0u;
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t p = p0 + i;
            const uint32_t key = vb[i] & 0x7FFFFFFFu;
            if (p < cN) {
                g += (key > T);
                q += (key == T);
            }
        }
        uint32_t total;
        const uint32_t before = block_excl_scan<SEL_WAVES>(g | (q << 16), S.wsum, total);
        const uint32_t g_before = before & 0xFFFFu, q_before = before >> 16;
        const uint32_t G = total & 0xFFFFu, Q = total >> 16;
        const uint32_t rem = (rT > run_eq) ? (rT - run_eq) : 0u;   // ties still to take
        uint32_t pos = run_sel + g_before + min(q_before, rem);
        uint32_t eq_seen = q_before;
        if (g | q) {
            // which of this thread's entries are sent, and where they go
            uint32_t ix[ITEMS], at[ITEMS];
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                const uint32_t p = p0 + i;
                const uint32_t key = vb[i] & 0x7FFFFFFFu;
                bool sel = (p < cN) && key > T;
                if (p < cN && key == T) {
                    sel = eq_seen < rem;
                    ++eq_seen;
                }
                at[i] = 0xFFFFFFFFu;
                ix[i] = 0;
                if (sel) {
                    if (pos < k) {
                        ix[i] = src.index(p);
                        if (index_ok(A, ix[i])) at[i] = pos;
                    }
                    ++pos;
                }
            }
            // sent_k += G reads the row: all of this thread's reads are issued before the first
            // is needed (one memory round trip instead of one per entry)
            float old[ITEMS];
            if (OP == SEL_PULL_V && !A.later) {
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) old[i] = (at[i] != 0xFFFFFFFFu) ? A.state[ix[i]] : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                if (at[i] != 0xFFFFFFFFu) {
                    const float v = __uint_as_float(vb[i]);
                    A.out_idx[outoff + at[i]] = ix[i];
                    A.out_val[outoff + at[i]] = v;
                    if (OP == SEL_WORKER) store_scattered(&A.state[ix[i]], A.m * v);
                    else if (OP == SEL_PULL) store_scattered(&A.state[ix[i]], 0.0f);
                    else if (!A.later) store_scattered(&A.state[ix[i]], old[i] + v);
                }
            }
        }
        run_sel += G + min(Q, rem);
        run_eq += Q;
    }
    if (run_sel != k && tid == 0) atomicAdd(&A.stats->internal_errors, 1ull);
}

// A small tensor (at most SMALL_N elements) straight from its buffer, 8 consecutive elements per thread in registers.
// Keys are counted only within an octave of the k-th key of the previous selection on this stream: one pass and one
// rank search give all but 12 bits of the new one, and the bucket it falls into mostly holds nothing but winners.
// (Counting every element, most lanes of a wavefront add to the same few counters, the zeros of a difference row
// all to one: 9 to 10 us on 7600 elements, which the whole launch waited for.)  Where the window has no answer -- no
// previous call, a k-th key that has moved further -- the nonzero keys are counted by their upper 12 bits, and those
// that share them with the k-th by the next 12.  us a call, generic passes over the elements in LDS / window / window
// that missed: worker steps on 60 tensors of 500 to 8192 elements 20.4 / 15.3 / 19.9, 200 of 8192 24.4 / 20.9 / 24.8, 20 of 1000
// 16.3 / 16.0 / 17.7; pulls on the printed state of the 60 23.3 / - / 21.1; first calls on the 60 27.0 / - / 21.0 (two
// kernels more).  A miss that left the registers and began again with the generic passes: 26.0, 30.5, 19.0; 29.5; 28.2.
// Returns whether the window held the k-th key (uniform; tests ask).
// STEP: the worker's accumulate comes first (no streaming pass has), and every element of the state is stored.
template <int OP, bool STEP = false>
__device__ __forceinline__ bool small_select(const SelectArgs &A, const TensorDesc &td, const PlanEntry &pe, uint32_t j,
                                             SelShared &S)
{
    constexpr uint32_t ITEMS = SMALL_N / SEL_THREADS, BINS = 4096, SHIFT = 12;
    static_assert(BINS * 4 <= sizeof(S.h) && (1u << SHIFT) == BINS && ITEMS % 4 == 0, "one histogram for all levels");
    static_assert(HSHIFT > SHIFT && HSHIFT - SHIFT <= SHIFT && HBINS == BINS, "two passes leave fewer bits than a window");
    const uint32_t tid = threadIdx.x, p0 = tid * ITEMS;
    const uint32_t t_prev = A.tprev[j];
    uint32_t bits[ITEMS];
    float row[OP == SEL_PULL_V ? ITEMS : 1];      // sent_k, which the values are not
#pragma unroll
    for (uint32_t x = 0; x < ITEMS; x += 4) {
        if (p0 + x + 4u <= td.n) {
            const f32x4 s = *(const f32x4_any *)(A.state + td.off + p0 + x);
            f32x4 v = s;
            if (OP == SEL_PULL_V) v = *(const f32x4_any *)(A.model + td.off + p0 + x) - s;
            if (STEP && OP == SEL_WORKER) {
                const f32x4 g = *(const f32x4_any *)(A.grad + td.off + p0 + x);
#pragma unroll
                for (int y = 0; y < 4; ++y) v[y] = __builtin_fmaf(A.lr, g[y], s[y]);
            }
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                bits[x + y] = __float_as_uint(v[y]);
                if (OP == SEL_PULL_V) row[x + y] = s[y];
            }
        } else {
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                const bool in = p0 + x + y < td.n;
                float s = in ? A.state[td.off + p0 + x + y] : 0.0f;
                if (STEP && OP == SEL_WORKER && in) s = __builtin_fmaf(A.lr, A.grad[td.off + p0 + x + y], s);
                bits[x + y] = __float_as_uint((OP == SEL_PULL_V && in) ? A.model[td.off + p0 + x + y] - s : s);
                if (OP == SEL_PULL_V) row[x + y] = s;
            }
        }
    }
    // f(key) for the nonzero keys of this thread (elements beyond the tensor read as 0), into cleared counters
    auto count = [&](auto f) {
        for (uint32_t b = tid; b < BINS; b += SEL_THREADS) S.h[b] = 0;
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < ITEMS; ++i) {
            const uint32_t key = bits[i] & 0x7FFFFFFFu;
            if (key != 0) f(key);
        }
    };
    const uint32_t base = max(t_prev >> SHIFT, BINS / 2) - BINS / 2;
    uint32_t seen = 0;                            // nonzero keys (low half), those in the window or above it
    count([&](uint32_t key) {
        ++seen;
        const uint32_t hi = key >> SHIFT;
        if (t_prev != 0 && hi >= base) {
            seen += 1u << 16;
            atomicAdd(&S.h[min(hi - base, BINS - 1u)], 1u);
        }
    });
    seen = block_sum<SEL_WAVES>(seen, S.wsum);
    const uint32_t nonzero = seen & 0xFFFFu;
    uint32_t T = 0, rT = pe.k - nonzero;          // (the message is completed with the lowest-index zeros)
    const bool near = (seen >> 16) >= pe.k && S.h[BINS - 1u] < pe.k;      // (the last bucket is open)
    if (nonzero >= pe.k) {
        // the k-th key is in bucket bk: its bits above the `low` lowest, its rank among the keys that share them
        uint32_t pfx, r2, low;
        int bk;
        if (near) {
            find_ranks<(int)BINS, SEL_WAVES>(S.h, pe.k, 0u, 0u, S.rowsum, S.res);
            bk = S.res[0];
            r2 = (uint32_t)S.res[1];
            pfx = base + (uint32_t)bk;
            low = SHIFT;
        } else {
            __syncthreads();
            count([&](uint32_t key) { atomicAdd(&S.h[key >> HSHIFT], 1u); });
            find_ranks<(int)BINS, SEL_WAVES>(S.h, pe.k, 0u, 0u, S.rowsum, S.res);
            const uint32_t top = (uint32_t)S.res[0], r1 = (uint32_t)S.res[1];
            low = HSHIFT - SHIFT;
            __syncthreads();
            count([&](uint32_t key) {
                if ((key >> HSHIFT) == top) atomicAdd(&S.h[(key >> low) & (BINS - 1u)], 1u);
            });
            find_ranks<(int)BINS, SEL_WAVES>(S.h, r1, 0u, 0u, S.rowsum, S.res);
            bk = S.res[0];
            r2 = (uint32_t)S.res[1];
            pfx = (top << SHIFT) | (uint32_t)bk;
        }
        if (S.h[bk] == r2 && pfx != 0) {
            T = (pfx << low) - 1u;                // the whole bucket is sent
            rT = 0;
        } else {
            __syncthreads();
            count([&](uint32_t key) {
                if ((key >> low) == pfx) atomicAdd(&S.h[key & ((1u << low) - 1u)], 1u);
            });
            find_ranks<(int)BINS, SEL_WAVES>(S.h, r2, 0u, 0u, S.rowsum, S.res);
            T = (pfx << low) | (uint32_t)S.res[0];
            rT = (uint32_t)S.res[1];
        }
    }
    uint32_t g = 0, q = 0;
#pragma unroll
    for (uint32_t i = 0; i < ITEMS; ++i) {
        const uint32_t key = bits[i] & 0x7FFFFFFFu;
        if (p0 + i < td.n) {
            g += key > T ? 1u : 0u;
            q += key == T ? 1u : 0u;
        }
    }
    uint32_t total;
    const uint32_t before = block_excl_scan<SEL_WAVES>(g | (q << 16), S.wsum, total);
    uint32_t eq = before >> 16, above = before & 0xFFFFu;      // ties: lowest index first, rT of them are taken
#pragma unroll
    for (uint32_t i = 0; i < ITEMS; ++i) {
        const uint32_t key = bits[i] & 0x7FFFFFFFu;
        const bool in = p0 + i < td.n, tie = in && key == T, over = in && key > T;
        const uint32_t pos = above + min(eq, rT);
        if ((over || (tie && eq < rT)) && pos < pe.k) {
            const uint32_t ix = td.off + p0 + i;
            const float v = __uint_as_float(bits[i]);
            A.out_idx[pe.outoff + pos] = ix;
            A.out_val[pe.outoff + pos] = v;
            if (STEP && OP == SEL_WORKER) bits[i] = __float_as_uint(A.m * v);
            else if (OP == SEL_WORKER) store_scattered(&A.state[ix], A.m * v);
            else if (OP == SEL_PULL) store_scattered(&A.state[ix], 0.0f);
            else if (!A.later) store_scattered(&A.state[ix], row[i] + v);
        }
        above += over ? 1u : 0u;
        eq += tie ? 1u : 0u;
    }
    if (STEP && OP == SEL_WORKER) {
#pragma unroll
        for (uint32_t x = 0; x < ITEMS; x += 4) {
            if (p0 + x + 4u <= td.n) {
                f32x4 o;
#pragma unroll
                for (int y = 0; y < 4; ++y) o[y] = __uint_as_float(bits[x + y]);
                *(f32x4_any *)(A.state + td.off + p0 + x) = o;
            } else {
#pragma unroll
                for (int y = 0; y < 4; ++y)
                    if (p0 + x + y < td.n) A.state[td.off + p0 + x + y] = __uint_as_float(bits[x + y]);
            }
        }
    }
    if (tid == 0) {
        if ((total & 0xFFFFu) + min(total >> 16, rT) != pe.k) atomicAdd(&A.stats->internal_errors, 1ull);
        A.tprev[j] = T;
    }
    return near;
}

// Rank (from the top) whose key becomes the next predicted threshold, and how the
// drift since the current threshold was set is measured.
//   c: candidates collected at the current threshold; E: candidates that threshold was
//   expected to collect when it was set (0 = unknown); `drift`: the two are comparable.
// Worker: sent entries stay large (they keep m * a) and unsent ones keep growing, so
// the keys of the tail move from step to step.  If the tail grew (c >= E), *Eq = E asks
// for the key of rank E among the present candidates: the old threshold's quantile has
// moved there, and the next threshold is scaled by the same ratio (hint_scaled).  If it
// shrank, the quantile lies below every candidate and cannot be read off: the rank is
// widened by the ratio of the counts instead.
template <int OP>
__device__ __forceinline__ uint32_t hint_rank(const TensorDesc &td, const PlanEntry &pe, bool drift,
                                              uint32_t c, uint32_t E, float m, uint32_t young, uint32_t *Eq)
{
    *Eq = 0;
    // a pull, or a worker without momentum: sent entries vanish, so even with nothing new
    // before the next call k entries must remain above the hinted key: about 2k for the worker, whose
    // steps follow each other, and for a pull what the plan and the age of the row say
    uint32_t R = (OP != SEL_WORKER) ? (young ? pe.k2_zero : pe.k2_pull) : (m == 0.0f ? pe.k2_zero : pe.k2);
    if (OP == SEL_WORKER && drift && E != 0) {
        if (c >= E) {
            *Eq = E;
        } else {
            const float d = fmaxf((float)c / (float)E, 0.5f);
            R = (uint32_t)((float)R / d);
        }
    }
    const uint32_t rmin = max(1u, pe.k / 4u);
    return min(max(R, rmin), td.n);
}

// Threshold for the next step: the key `edge` of the hinted rank, moved by half of the
// relative shift that the previous threshold's quantile showed (q_e / tau_cur, between 1
// and 2).  Half: growth usually slows down, and a threshold that is too high costs a
// dense re-selection while one that is too low only costs extra candidates.
__device__ __forceinline__ uint32_t hint_scaled(uint32_t edge, uint32_t q_e, uint32_t tau_cur)
{
    if (q_e <= tau_cur || tau_cur < 0x00800000u || q_e >= 0x7F800000u) return edge;   // no growth / not normal
    const float f = 1.0f + 0.5f * (fminf(__uint_as_float(q_e) / __uint_as_float(tau_cur), 2.0f) - 1.0f);
    const float x = __uint_as_float(edge) * f;
    const uint32_t t = __float_as_uint(x) & 0x7FFFFFFFu;
    return (t > edge && t < 0x7F800000u) ? t : edge;
}

// Next threshold when rank R was not among the candidates: relax the current one by a
// quarter, but not below half of the smallest candidate key (all of them already pass).
__device__ __forceinline__ uint32_t hint_relaxed(uint32_t tau_cur, uint32_t kmin)
{
    const float f = __uint_as_float(tau_cur & 0x7FFFFFFFu) * 0.75f;
    uint32_t tn = __float_as_uint(f) & 0x7FFFFFFFu;
    if (!(tau_cur > 1u) || tn == 0) tn = 1;
    if (kmin != 0xFFFFFFFFu && kmin < 0x7F800000u) {
        const uint32_t half = __float_as_uint(__uint_as_float(kmin) * 0.5f) & 0x7FFFFFFFu;
        if (half > tn) tn = half;
    }
    return tn;
}

// Fewer candidates than k although every nonzero key was collected: the message is
// completed with the tensor's lowest-index zero-key entries.  With z = k - c zeros to
// add and candidate i (in index order) at x_i, the zeros below x_i number x_i - off - i;
// the P candidates for which that is < z lie inside the leading run [off, off + z + P),
// which is sent whole (z zeros and P candidates); the other candidates follow.
template <int OP, bool WRITTEN, class Src>
__device__ __forceinline__ void zero_fill_emit(const Src src, const uint32_t c, const TensorDesc &td,
                                               const PlanEntry &pe, const SelectArgs &A, uint32_t *wsum)
{
    const uint32_t tid = threadIdx.x;
    const uint32_t z = pe.k - c;
    uint32_t mine = 0;
    for (uint32_t p = tid; p < c; p += SEL_THREADS) mine += ((src.index(p) - td.off - p) < z) ? 1u : 0u;
    const uint32_t P = block_sum<SEL_WAVES>(mine, wsum);
    const uint32_t X = z + P;
    for (uint32_t q = tid; q < X; q += SEL_THREADS) {
        const uint32_t ix = td.off + q;
        const float v = row_value<OP, WRITTEN>(A.state, A.model, ix);
        A.out_idx[pe.outoff + q] = ix;
        A.out_val[pe.outoff + q] = v;
        fix_sent<OP>(A.state, ix, v, A.m, A.later != 0);
    }
    for (uint32_t p = P + tid; p < c; p += SEL_THREADS) {
        const uint32_t ix = src.index(p);
        const float v = __uint_as_float(src.bits(p));
        A.out_idx[pe.outoff + z + p] = ix;
        A.out_val[pe.outoff + z + p] = v;
        if (index_ok(A, ix)) fix_sent<OP>(A.state, ix, v, A.m, A.later != 0);
    }
}

// Minimum over the 64 lanes of a wavefront (DPP, same pattern as the scan);
// the result is valid in lane 63.
__device__ __forceinline__ uint32_t wave_min_to_last(uint32_t v)
{
    int x = (int)v;
    const int id = (int)0xFFFFFFFFu;
#define DGS_MIN_STEP(ctrl, rmask)                                                             \
    x = (int)min((uint32_t)x, (uint32_t)__builtin_amdgcn_update_dpp(id, x, ctrl, rmask, 0xf, false))
    DGS_MIN_STEP(0x111, 0xf);
    DGS_MIN_STEP(0x112, 0xf);
    DGS_MIN_STEP(0x114, 0xf);
    DGS_MIN_STEP(0x118, 0xf);
    DGS_MIN_STEP(0x142, 0xa);
    DGS_MIN_STEP(0x143, 0xc);
#undef DGS_MIN_STEP
    return (uint32_t)x;
}

// Ordered-list entry: LDS while it fits, global scratch beyond (an ordinary cached store: the
// list is read back by this workgroup; see release_dev() for the one case where another
// workgroup writes to the same place later in the launch).
__device__ __forceinline__ void put_entry(uint2 *llist, uint2 *glist, uint32_t pos, uint2 e)
{
    if (pos < SEL_LDS_LIST) {
        llist[pos] = e;
    } else {
        glist[pos] = e;
        // keeps the two stores apart: merged into one store through a generic pointer they
        // would take the slow flat path into LDS
        asm volatile("" ::: "memory");
    }
}

}  // namespace dgs
