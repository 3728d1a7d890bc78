// What the workgroups of a selection launch do with one tensor: joins of the candidates that the streaming pass has left in its
// tiles, the exact selection from a list, and what follows a failed prediction.  Used by k_select and k_step.
#pragma once
#include "dgs_chain.h"

namespace dgs {

// The launch a workgroup is part of: the selection kernel, the same with the chain's workgroups in it, or a whole call (k_step).
enum Form { FORM_SELECT = 0, FORM_CHAIN = 1, FORM_STEP = 2 };
// Whether the rows that the selection ranks have been stored by other workgroups of the same launch.
template <int OP, int FORM>
constexpr bool written() { return FORM == FORM_STEP && OP == SEL_WORKER; }

// h: HBINS counters in LDS.  Thread 0 receives the threshold whose candidates number at
// least pe.k2 (or every nonzero when there are fewer), and the middle of the bucket that holds
// the k-th key (anchors the window histograms).  Contains find_ranks' three barriers.
template <int NW>
__device__ __forceinline__ void pick_from_hist(const uint32_t *h, const PlanEntry &pe, uint32_t *rowsum, int *res,
                                               uint32_t &tau_out, uint32_t &tprev_out)
{
    find_ranks<HBINS, NW>(h, pe.k2, pe.k, 0u, rowsum, res);
    const int b2 = res[0], b1 = res[2];
    // the histogram holds the nonzero keys only: a rank beyond its total means
    // "fewer nonzeros than that", and every nonzero is collected
    uint32_t t;
    if (b2 < 0 && b1 < 0) {
        t = 1;
    } else if (b2 < 0) {
        t = (b1 > 0) ? (1u << HSHIFT) : 1u;
    } else if (b2 > 0) {
        t = (uint32_t)b2 << HSHIFT;
    } else if (b1 > 0) {
        t = 1u << HSHIFT;
    } else {
        t = 1;   // the k-th key is tiny or zero: collect every nonzero
    }
    tau_out = t;
    tprev_out = (b1 >= 0) ? (((uint32_t)b1 << HSHIFT) + (1u << (HSHIFT - 1))) : 0u;
}

constexpr uint32_t B_GROUP_MAX = 8;   // most parts one re-collecting workgroup looks after

struct PartShared {
    SelShared S;
    uint32_t pbase[SEG_MAX_PER_TENSOR + 1];   // first list position of every part of the tensor
    uint32_t pofs[SEG_MAX_PER_TENSOR];        // where every part's global list starts (entries into ord)
    uint32_t wtot[SEL_WAVES];
    uint32_t vbuf[B_GROUP_MAX];               // verdicts of the tensors of a re-collecting workgroup's parts
    uint32_t start0;                          //       entries of the previous tensor in a shared first tile
    uint32_t crowd_slot[SEL_THREADS];         //       the round's crowded tiles (which lane has them)
    uint32_t bc;
    uint32_t pair[2];
    uint32_t wmax[SEL_WAVES];
    uint32_t all, least;                      // (the entries of all units; the complement of the most of one)
};

// JOIN of a run of tiles: the candidates of tensor j in tiles [sd.tile0, sd.tile0 + sd.ntiles),
// in index order, through `put(position, entry)`.  Returns the count; `ovf` is set if a tile had
// overflowed its slots.  Rounds of SEL_THREADS tiles.  Every lane takes one tile's count; a
// workgroup scan of the counts gives every tile its list position.  The tiles' first lines (8
// candidates, 64 bytes) are fetched as the contiguous stretch they are -- four lanes per line,
// four lines per lane -- and put in place with the positions read back from LDS; what crowded
// tiles hold behind theirs, and a first tile shared with the previous tensor, go to a worklist that
// the wavefronts then copy, a tile at a time each or four.
template <class Put>
__device__ __forceinline__ uint32_t join_part(const SelectArgs &A, const TensorDesc &td, const SegDesc &sd,
                                              PartShared &P, bool &ovf_out, Put put)
{
    const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63u;
    const uint32_t tlo = td.off / TILE;
    const bool head_shared = (td.off % TILE) != 0;
    // list position and count of every tile of the round (bit 31: its first line begins with another
    // tensor's candidates); the window is counted below them meanwhile
    static_assert((WIN_BINS + 2 * SEL_THREADS) * 4 <= sizeof(P.S.h), "room for the tiles of a round");
    uint32_t *tile_pos = P.S.h + WIN_BINS, *tile_n = tile_pos + SEL_THREADS;
    uint32_t base = 0;
    int ovf = 0;
    // lines of this wavefront's 64 tiles: load v covers tiles 16 v .. 16 v + 15.  A round's are fetched as soon as
    // those before are in place, while the crowded tiles are copied: a round on ResNet-50 shapes 111.1 -> 110.0 us, an
    // event of a server with 12 sent rows 59.5 -> 59.1 (each side as two copies, whose medians agreed to 0.2).  A second
    // set of registers, fetched a whole round ahead, brought no more: one compute unit takes in 29 bytes a ns at most.
    uint4 pf[4];
    uint32_t w;
    auto fetch = [&](uint32_t r0) {
#pragma unroll
        for (uint32_t v = 0; v < 4; ++v) {
            const uint32_t tl = r0 + wave * 64u + v * 16u + (lane >> 2);
            pf[v] = (tl < sd.ntiles) ? ((const uint4 *)(A.heads + (size_t)(sd.tile0 + tl) * HEAD))[lane & 3u]
                                     : make_uint4(0, 0, 0, 0);
        }
        w = (r0 + tid < sd.ntiles) ? A.tile_cnt[sd.tile0 + r0 + tid] : 0u;
    };
    fetch(0);
    for (uint32_t r0 = 0; r0 < sd.ntiles; r0 += SEL_THREADS) {
        const uint32_t t = sd.tile0 + r0 + tid;
        uint32_t n_t, start;
        tile_counts(w, t, tlo, head_shared, n_t, start, ovf);
        // one scan for both: list positions (low 19 bits: at most 2^18 candidates a round) and the
        // number of crowded tiles (the bits above)
        const bool crowded = n_t != 0 && (start != 0 || n_t > HEAD);
        uint32_t total;
        const uint32_t excl = block_excl_scan<SEL_WAVES>(n_t | (crowded ? 1u << 19 : 0u), P.S.wsum, total);
        const uint32_t pos = base + (excl & 0x7FFFFu);
        const uint32_t round_n = total & 0x7FFFFu;
        uint32_t nc = total >> 19;
        tile_pos[tid] = pos;
        tile_n[tid] = n_t | (start != 0 ? 0x80000000u : 0u);
        if (crowded) P.crowd_slot[excl >> 19] = tid;
        if (head_shared && t == tlo) P.start0 = start;      // (the tensor's first tile, shared with the one before)
        __syncthreads();
#pragma unroll
        for (uint32_t v = 0; v < 4; ++v) {
            const uint32_t slot = wave * 64u + v * 16u + (lane >> 2);
            const uint32_t nv = tile_n[slot], p = tile_pos[slot], e0 = 2u * (lane & 3u);
            const uint32_t n = (nv >> 31) ? 0u : nv;
            if (e0 < n) put(p + e0, make_uint2(pf[v].x, pf[v].y));
            if (e0 + 1 < n) put(p + e0 + 1, make_uint2(pf[v].z, pf[v].w));
        }
        if (r0 + SEL_THREADS < sd.ntiles) fetch(r0 + SEL_THREADS);
        // What the first lines do not hold: the candidates behind them in crowded tiles, and all of a first
        // tile shared with the previous tensor.
        if (nc != 0 && nc <= 2 * SEL_WAVES) {
            // a few: a wavefront copies one at a time (a round on ResNet-50 shapes, 20 of them in 1024 tiles: the
            // worker's selection 21.5 us, 22.3 the other way)
            for (uint32_t q = wave; q < nc; q += SEL_WAVES) {
                const uint32_t slot = P.crowd_slot[q], nv = tile_n[slot], tc = sd.tile0 + r0 + slot;
                const uint32_t skip = (nv >> 31) ? 0u : HEAD, from = skip ? HEAD : P.start0;
                for (uint32_t i = skip + lane; i < (nv & 0x7FFFFFFFu); i += 64)
                    put(tile_pos[slot] + i, *candidate(A, tc, from + i - skip));
            }
            nc = 0;
        }
        // Many: 16 lanes take a tile, CU tiles each, and step along them together, so that a wavefront has
        // 4 CU stretches of 128 bytes in flight.  (Every list position searching its tile in LDS and
        // fetching its own entry: a step without momentum at 1 % on ResNet-50 shapes, 25 candidates a tile,
        // 21.8 us instead of 17.9; the selections of servers 1.3 to 3 us more.)
        constexpr uint32_t CU = 4;
        for (uint32_t q0 = wave * 4u; q0 < nc; q0 += 4u * SEL_WAVES * CU) {      // (wave-uniform)
            uint32_t tile[CU], from[CU], at[CU], left[CU], most = 0;
#pragma unroll
            for (uint32_t u = 0; u < CU; ++u) {
                const uint32_t q = q0 + u * 4u * SEL_WAVES + (lane >> 4);
                tile[u] = sd.tile0;
                from[u] = at[u] = left[u] = 0;
                if (q < nc) {
                    const uint32_t slot = P.crowd_slot[q], nv = tile_n[slot];
                    const uint32_t skip = (nv >> 31) ? 0u : HEAD;
                    tile[u] = sd.tile0 + r0 + slot;
                    from[u] = skip ? HEAD : P.start0;
                    at[u] = tile_pos[slot] + skip;
                    left[u] = (nv & 0x7FFFFFFFu) - skip;
                }
                most = max(most, left[u]);
            }
            for (uint32_t i = lane & 15u; ballot64(i < most) != 0; i += 16u) {
                uint2 e[CU];
#pragma unroll
                for (uint32_t u = 0; u < CU; ++u)
                    if (i < left[u])
                        e[u] = *candidate(A, tile[u], from[u] + i);
#pragma unroll
                for (uint32_t u = 0; u < CU; ++u)
                    if (i < left[u]) put(at[u] + i, e[u]);
            }
        }
        base += round_n;
        // (the next round rewrites the positions behind the two barriers of its scan)
    }
    ovf_out = __syncthreads_or(ovf) != 0;
    return base;
}

// Elements of tensor j inside the part, as rows of 256 consecutive elements per wavefront
// (4 per lane): the wavefronts take the part's tiles in equal consecutive runs, so that the
// order of wavefronts is the order of indices.
struct DenseRun {
    uint32_t t0, t1;     // this wavefront's tiles [t0, t1) of the flat buffer
    uint32_t lo, hi;     // the tensor's elements [lo, hi)
};

__device__ __forceinline__ DenseRun dense_run(const TensorDesc &td, const SegDesc &sd)
{
    const uint32_t wave = threadIdx.x >> 6;
    const uint32_t per = (sd.ntiles + SEL_WAVES - 1) / SEL_WAVES;
    DenseRun r;
    r.t0 = sd.tile0 + min(wave * per, sd.ntiles);
    r.t1 = sd.tile0 + min((wave + 1) * per, sd.ntiles);
    r.lo = td.off;
    r.hi = td.off + td.n;
    return r;
}

// RE-HISTOGRAM of one part: key bits [30:19] of the tensor's nonzero elements in the part,
// into lh (HBINS counters in LDS, zeroed here).  Ends with a barrier.
template <int OP, bool WRITTEN>
__device__ __forceinline__ void dense_hist(const SelectArgs &A, const TensorDesc &td, const SegDesc &sd, uint32_t *lh)
{
    for (uint32_t b = threadIdx.x; b < HBINS; b += SEL_THREADS) lh[b] = 0;
    __syncthreads();
    const DenseRun r = dense_run(td, sd);
    const uint32_t lane = lane_id();
    // two tiles per turn, all of their loads issued before the first counter is touched (the odd
    // last turn reads its one tile twice and counts it once)
    for (uint32_t t = r.t0; t < r.t1; t += 2) {
        const bool two = t + 1 < r.t1;
        uint32_t bits[2][4][4];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int row = 0; row < 4; ++row)
                quad_bits<OP, WRITTEN>(A, (u && two ? t + 1 : t) * TILE + row * 256 + lane * 4, r.lo, r.hi, bits[u][row]);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int row = 0; row < 4; ++row)
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const uint32_t key = bits[u][row][x] & 0x7FFFFFFFu;      // elements outside the tensor read as 0
                    if (key != 0 && (u == 0 || two)) atomicAdd(&lh[key >> HSHIFT], 1u);
                }
    }
    __syncthreads();
}

// RE-COLLECTION of one part: the tensor's elements in the part with key >= tau, in index
// order, through `put(position, entry)`; nothing is written when there are more than `cap`.
// Two passes over the part (count, then place).  Returns the count.
template <int OP, bool WRITTEN, class Put>
__device__ __forceinline__ uint32_t dense_compact(const SelectArgs &A, const TensorDesc &td, const SegDesc &sd,
                                                  uint32_t tau, uint32_t cap, PartShared &P, Put put)
{
    const DenseRun r = dense_run(td, sd);
    const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
    uint32_t mine = 0;
    for (uint32_t t = r.t0; t < r.t1; t += 2) {      // two tiles in flight, as in dense_hist
        const bool two = t + 1 < r.t1;
        uint32_t bits[2][4][4], in[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int row = 0; row < 4; ++row)
                in[u][row] = quad_bits<OP, WRITTEN>(A, (u && two ? t + 1 : t) * TILE + row * 256 + lane * 4, r.lo, r.hi,
                                           bits[u][row]);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int row = 0; row < 4; ++row)
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    if ((u == 0 || two) && ((in[u][row] >> x) & 1u) && (bits[u][row][x] & 0x7FFFFFFFu) >= tau) ++mine;
    }
    const uint32_t wsum_ = wave_sum(mine);
    __syncthreads();
    if (lane == 0) P.wtot[wave] = wsum_;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (uint32_t x = 0; x < SEL_WAVES; ++x) {
        const uint32_t v = P.wtot[x];
        if (x < wave) before += v;
        total += v;
    }
    if (total > cap) return total;
    uint32_t run = before;
    for (uint32_t t = r.t0; t < r.t1; ++t) {
        uint32_t tbits[4][4], tin[4];
#pragma unroll
        for (int row = 0; row < 4; ++row) tin[row] = quad_bits<OP, WRITTEN>(A, t * TILE + row * 256 + lane * 4, r.lo, r.hi, tbits[row]);
#pragma unroll
        for (int row = 0; row < 4; ++row) {
            const uint32_t e0 = t * TILE + row * 256 + lane * 4;
            const uint32_t (&bits)[4] = tbits[row];
            bool f[4];
            uint64_t mk[4];
            const uint32_t in = tin[row];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                f[x] = ((in >> x) & 1u) && (bits[x] & 0x7FFFFFFFu) >= tau;
                mk[x] = ballot64(f[x]);
            }
            if ((mk[0] | mk[1] | mk[2] | mk[3]) != 0) {
                uint32_t p = run + mbcnt64(mk[0]) + mbcnt64(mk[1]) + mbcnt64(mk[2]) + mbcnt64(mk[3]);
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    if (f[x]) {
                        put(p, make_uint2(e0 + x, bits[x]));
                        ++p;
                    }
                }
                run += (uint32_t)(__popcll(mk[0]) + __popcll(mk[1]) + __popcll(mk[2]) + __popcll(mk[3]));
            }
        }
    }
    // the two passes must have seen the same elements
    if (lane == 0 && run - before != wsum_) atomicAdd(&A.stats->internal_errors, 1ull);
    return total;
}

// A tensor on the chain whose window missed the k-th key (a row that has waited long), but whose candidates are all there: this
// workgroup counts them again alone, first by 12 leading bits, then in a window around the bucket found.  Nine events in ten of a
// server with 2 workers, 8 tensors of 1.2M elements and lists of 11 K, selection in us: within 60, and 157 with such tensors
// collected again by their parts; an event 50.8 / 65.9 on average, 59.8 with one workgroup per tensor.  (Where the chain has
// launches of its own the parts collect again: this code costs a selection 0.5 to 1 %.)
__device__ __forceinline__ uint32_t window_again(const SelectArgs &A, const TensorDesc &td, const PlanEntry &pe, uint32_t j,
                                                 uint32_t c, uint32_t R, uint32_t tau_cur, PartShared &P)
{
    uint32_t *h = P.S.h;
    const uint32_t tlo = td.off / TILE, nt = (td.off + td.n - 1u) / TILE - tlo + 1u;
    const bool measurable = (R != 0) && (c >= R);
    bool over;
    __syncthreads();
    count_tiles(A, td, tlo, nt, h, HBINS, P.S.wsum, over, [](uint32_t key) { return key >> HSHIFT; });
    find_ranks<HBINS, SEL_WAVES>(h, pe.k, measurable ? R : pe.k, 0u, P.S.rowsum, P.S.res);
    const uint32_t top = (uint32_t)P.S.res[0];
    uint32_t tn = hint_relaxed(tau_cur, 0xFFFFFFFFu), expect = 0;
    if (measurable) {
        tn = max((uint32_t)P.S.res[2] << HSHIFT, 1u);
        expect = R - (uint32_t)P.S.res[3] + h[P.S.res[2]];
    }
    const uint32_t win = max(top << (HSHIFT - SEG_LOWBITS), 1u) - 1u;      // (below the bucket: the first one counts what lies lower, too)
    __syncthreads();
    window_tiles(A, td, tlo, nt, win, h, P.S.wsum, over);
    find_ranks<SEG_WBINS, SEL_WAVES>(h, pe.k, 0u, 0u, P.S.rowsum, P.S.res);
    if (threadIdx.x == 0) {
        SegState *st = &A.segstate[j];
        st->pfx = win + (uint32_t)P.S.res[0];
        st->r2 = (uint32_t)P.S.res[1];
        st_dev(&st->chain, make_uint2(st->r2, ((uint32_t)SEG_ACTIVE << CHAIN_STATUS_SHIFT) | st->pfx));
        atomicAdd(&A.stats->candidates, (unsigned long long)c);
        atomicAdd(&A.stats->segmented_tensors, 1ull);
        atomicAdd(&A.stats->repaired_tensors, 1ull);
        if (A.write_hint) {
            A.tau[j] = min(tn, 0x7F7FFFFFu);
            A.hint2[j] = expect;
        }
    }
    __syncthreads();
    return (uint32_t)SEG_ACTIVE;
}

// A tensor that takes the chain: its window histogram (c candidates in all; the sum of its parts'
// own, or, collected again, the one the parts have added to in ghist) -> the 19-bit prefix of the
// k-th key, its rank among the entries sharing it, and the next hint.  Returns the tensor's status (SEG_ACTIVE / SEG_LISTS, or 0 = failed);
// thread 0 writes segstate / hints.
template <int OP, bool HERE>
__device__ __forceinline__ uint32_t window_step(const SelectArgs &A, const TensorDesc &td, const PlanEntry &pe,
                                                uint32_t j, uint32_t &c, bool &ovf, uint32_t tau_cur, uint32_t tprev_cur,
                                                uint32_t hint2_cur, bool exact_mode, bool lists, PartShared &P)
{
    const uint32_t tid = threadIdx.x;
    uint32_t *h = P.S.h;
    uint32_t *gh = A.ghist + (size_t)j * HBINS;
    uint32_t mylow = 0xFFFFFFFFu, cnt = 0;
    if (tid == 0) P.S.kmin = 0xFFFFFFFFu;
    if (HERE && !lists && tid < window_blocks(td.nseg, A.window_max)) cnt = ld_dev(&A.segcnt[td.seg_first + tid * window_parts(td.nseg, A.window_max)]);
    if (!lists) {
        // four counters per load, every other part: a tensor of 90 parts costs a thread 45 loads
        static_assert(SEG_WBINS == 2 * SEL_THREADS, "two threads per four counters");
        const uint32_t b4 = tid & (SEL_THREADS / 2 - 1u), half = tid / (SEL_THREADS / 2);
        const uint4 *ph = (const uint4 *)part_hist(A, td, j, 0) + b4;
        uint4 sum = make_uint4(0, 0, 0, 0);
        const uint32_t nh = HERE ? window_blocks(td.nseg, A.window_max) : td.nseg;
#pragma unroll 8
        for (uint32_t s = half; s < nh; s += 2) {
            uint4 v;
            if (HERE) {      // written in this launch
                const uint2 *p = (const uint2 *)(ph + (size_t)s * (SEG_WBINS / 4));
                const uint2 a = ld_dev(p), b = ld_dev(p + 1);
                v = make_uint4(a.x, a.y, b.x, b.y);
            } else {
                v = ph[(size_t)s * (SEG_WBINS / 4)];
            }
            sum.x += v.x;
            sum.y += v.y;
            sum.z += v.z;
            sum.w += v.w;
        }
        if (half == 0) ((uint4 *)h)[b4] = sum;
        __syncthreads();
        if (half != 0) {
            uint4 t = ((uint4 *)h)[b4];
            ((uint4 *)h)[b4] = make_uint4(t.x + sum.x, t.y + sum.y, t.z + sum.z, t.w + sum.w);
        }
    }
    __syncthreads();
    for (uint32_t b = tid; b < SEG_WBINS; b += SEL_THREADS) {
        uint32_t v = h[b];
        if (lists) {
            v = ld_dev(&gh[b]);
            if (v) st_dev(&gh[b], 0u);   // clean for the next use
            h[b] = v;
        }
        if (v && mylow == 0xFFFFFFFFu) mylow = b;
    }
    mylow = wave_min_to_last(mylow);
    if (lane_id() == 63 && mylow != 0xFFFFFFFFu) atomicMin(&P.S.kmin, mylow);
    if (HERE && !lists) {
        c = block_sum<SEL_WAVES>(cnt & 0x7FFFFFFFu, P.S.wsum);
        ovf = __syncthreads_or((int)(cnt >> 31)) != 0;
    }
    const uint32_t win_base = seg_window_base(tau_cur, tprev_cur);
    const int bin_min = (win_base > (tau_cur >> SEG_LOWBITS)) ? 1 : 0;   // bin 0 mixes in lower keys
    uint32_t R = 0, Eq = 0;
    if (A.write_hint) R = hint_rank<OP>(td, pe, !exact_mode, c, hint2_cur, A.m, A.young, &Eq);
    const bool measurable = (R != 0) && (c >= R);
    const uint32_t qlow = max(c / 4u, min(c, 16u));
    const uint32_t third = measurable ? Eq : ((R != 0 && c != 0) ? (c - qlow + 1u) : 0u);
    find_ranks<SEG_WBINS, SEL_WAVES>(h, pe.k, measurable ? R : pe.k, third, P.S.rowsum, P.S.res);
    const int bk = P.S.res[0], bR = P.S.res[2];
    const uint32_t lowest = P.S.kmin;
    const bool ok = !ovf && (c >= pe.k) && bk >= bin_min && bk < (int)SEG_WBINS - 1;
    if (HERE && !lists && !ok && !ovf && c >= pe.k && td.n <= GROUP_TILES * TILE)
        return window_again(A, td, pe, j, c, R, tau_cur, P);
    if (tid == 0 && ok) {
        SegState *st = &A.segstate[j];
        st->pfx = win_base + (uint32_t)bk;
        st->r2 = (uint32_t)P.S.res[1];
        // (the slabs go on while the hint is worked out)
        if (HERE && !lists) st_dev(&st->chain, make_uint2(st->r2, ((uint32_t)SEG_ACTIVE << CHAIN_STATUS_SHIFT) | st->pfx));
        atomicAdd(&A.stats->candidates, (unsigned long long)c);
        atomicAdd(&A.stats->segmented_tensors, 1ull);
        if (A.write_hint) {
            uint32_t tn = 0, expect = 0;
            if (measurable && bR >= bin_min && bR < (int)SEG_WBINS - 1) {
                const uint32_t edge = (win_base + (uint32_t)bR) << SEG_LOWBITS;
                tn = edge ? edge : 1u;
                expect = R - (uint32_t)P.S.res[3] + h[bR];
                const int bE = P.S.res[4];
                if (bE >= bin_min && bE < (int)SEG_WBINS - 1)
                    tn = hint_scaled(tn, (win_base + (uint32_t)bE) << SEG_LOWBITS, tau_cur);
            }
            if (tn == 0 && !measurable && R != 0 && lowest != 0xFFFFFFFFu && (int)lowest >= bin_min &&
                P.S.res[4] >= (int)lowest && P.S.res[4] < (int)SEG_WBINS - 1) {
                const uint32_t kmin = max((win_base + lowest) << SEG_LOWBITS, tau_cur);
                tn = hint_extrapolated(kmin, c, R, qlow, ((uint32_t)P.S.res[4] - lowest + 1u) << SEG_LOWBITS);
                expect = R;
            }
            if (tn == 0) {
                const uint32_t kmin = (lowest == 0xFFFFFFFFu || (int)lowest < bin_min) ? 0xFFFFFFFFu
                                                             : max((win_base + lowest) << SEG_LOWBITS, tau_cur);
                tn = hint_relaxed(tau_cur, kmin);
                expect = 0;
            }
            if (tn >= 0x7F800000u) tn = 0x7F7FFFFFu;
            A.tau[j] = tn;
            A.hint2[j] = expect;
        }
    }
    __syncthreads();
    return !ok ? 0u : (lists ? (uint32_t)SEG_LISTS : (uint32_t)SEG_ACTIVE);
}

// Selection of a whole tensor straight from the buffers by this one workgroup:
// dense requests on tensors outside the chain, and whatever the re-collection could not
// resolve.  Exact for any data; slow on large tensors.
template <int OP, bool WRITTEN>
__device__ __forceinline__ void dense_select(const SelectArgs &A, const TensorDesc &td, const PlanEntry &pe, uint32_t j,
                                             uint32_t tau_cur, PartShared &P, uint2 *llist)
{
    const uint32_t tid = threadIdx.x;
    uint32_t R = 0, Eq = 0;
    if (td.big && A.write_hint) R = hint_rank<OP>(td, pe, false, 0u, 0u, A.m, A.young, &Eq);
    uint32_t tau_next = 0, expect = 0, q_e = 0, t_k = 0;
    if (td.n <= 2 * SEL_LDS_LIST) {
        uint32_t *lv = (uint32_t *)llist;
        __syncthreads();
        for (uint32_t p = tid; p < td.n; p += SEL_THREADS)
            lv[p] = __float_as_uint(row_value<OP, WRITTEN>(A.state, A.model, td.off + p));
        __syncthreads();
        // Entries per thread, 2 / 3 / 4 of them, us a dense call: 300 tensors of 20 K at 0.1, worker 85.4 / 82.3 / 81.3,
        // difference row 67.3 / 64.8 / 63.5, printed state 73.9 / 71.5 / 70.4; at 0.5 76.8 / 77.4 / 79.9, 68.4 / 68.7 / 71.2,
        // 74.9 / 74.0 / 74.8; 200 of 30 K at 0.5 60.0 / 60.3 / 62.8, 52.7 / 52.7 / 55.3, 56.5 / 54.6 / 56.7.  (1: 3 to 10 us
        // more, 8: up to 24 us more at 0.5.)
        SrcDenseLds src{lv, td.off};
        select_emit<OP, OP == SEL_PULL_V ? 4 : 3>(src, td.n, pe.k, R, 0u, 0xFFFFFFFFu, 0u, false, 0xFFFFFFFFu, P.S, A, pe.outoff,
                           &tau_next, &expect, &q_e, &t_k);
    } else {
        // (4 / 8 a thread: 8 tensors of 60 K at 0.1, worker 102.9 / 116.2, printed state 109.7 / 134.1; one of 2.4M that
        // falls back 833.7 / 924.5)
        SrcDense<OP, WRITTEN> src{A.state, A.model, td.off};
        select_emit<OP, 4>(src, td.n, pe.k, R, 0u, 0xFFFFFFFFu, 0u, false, 0xFFFFFFFFu, P.S, A, pe.outoff,
                           &tau_next, &expect, &q_e, &t_k);
    }
    if (td.big && A.write_hint && tid == 0) {
        uint32_t tn = tau_next;
        if (tn == 0) {
            tn = hint_relaxed(tau_cur, 0xFFFFFFFFu);
            expect = 0;
        }
        if (tn >= 0x7F800000u) tn = 0x7F7FFFFFu;
        A.tau[j] = tn;
        A.hint2[j] = expect;
        A.tprev[j] = t_k;
    }
}

// What a selection from a list leaves for the next call.
__device__ __forceinline__ void list_hints(const SelectArgs &A, uint32_t j, uint32_t tau_next, uint32_t expect, uint32_t q_e,
                                           uint32_t t_k, uint32_t tau_cur, uint32_t kmin)
{
    if (!A.write_hint || threadIdx.x != 0) return;
    uint32_t tn = tau_next;
    if (tn == 0) {
        tn = hint_relaxed(tau_cur, kmin);
        expect = 0;
    } else if (q_e != 0) {
        tn = hint_scaled(tn, q_e, tau_cur);
    }
    if (tn >= 0x7F800000u) tn = 0x7F7FFFFFu;   // keep the hint finite
    A.tau[j] = tn;
    A.hint2[j] = expect;
    A.tprev[j] = t_k;
}

// The tensor's candidates are in `llist` (first SEL_LDS_LIST) and `glist` (beyond): exact
// selection, emission, fix-up and the next hint.  win_*: the window histogram in P.S.h counted
// while the list was built (single-part tensors), see select_emit.  KEY: the k-th key alone, for the workgroups that await it.
template <int OP, bool KEY = false>
__device__ __forceinline__ void list_select(const SelectArgs &A, const TensorDesc &td, const PlanEntry &pe, uint32_t j,
                                            uint32_t c, uint32_t kmin, uint32_t tau_cur, uint32_t hint2_cur,
                                            uint32_t win_join, bool win_counted, bool exact_mode, PartShared &P,
                                            uint2 *llist, uint2 *glist)
{
    // the window placed by the hints serves if no candidate lies below the threshold (none can);
    // a histogram counted on the way then stands as it is
    const bool anchored = (win_join != 0xFFFFFFFFu) && (kmin != 0xFFFFFFFFu) && (kmin >> win_shift(OP)) >= (tau_cur >> win_shift(OP));
    const bool win_ready = win_counted && anchored;
    const uint32_t win_base = (kmin == 0xFFFFFFFFu) ? 0xFFFFFFFFu : (anchored ? win_join : (kmin >> win_shift(OP)));
    const uint32_t win_min = (anchored && win_join > (kmin >> win_shift(OP))) ? 1u : 0u;   // entries below the window
    uint32_t R = 0, Eq = 0;
    if (A.write_hint && (threadIdx.x < 3u * 64u || win_base == 0xFFFFFFFFu)) R = hint_rank<OP>(td, pe, !exact_mode, c, hint2_cur, A.m, A.young, &Eq);
    uint32_t tau_next = 0, expect = 0, q_e = 0, t_k = 0;
    if (KEY) {
        uint32_t rT;
        if (select_key<OP>(SrcSplit{llist, glist}, c, pe.k, R, Eq, win_base, win_min, win_ready, kmin, P.S, A, &tau_next, &expect, &q_e, t_k, rT) &&
            threadIdx.x == 0)
            st_dev(&A.segstate[j].key, make_uint2(rT, KEY_READY | t_k));
    } else if (c <= SEL_LDS_LIST) {
        // Entries per thread, 2 / 3 / 4 of them: a round on ResNet-50 shapes 111.0 / 109.8 / 111.2 us, an event of a server with
        // 32 sent rows 59.8 / 59.5 / 59.9, with difference rows 83.0 / 82.8 / 83.2; 70 odd tensors, 6 workers 45.4 / 45.1 /
        // 45.6.  (Every instance of the emission costs the kernel scalar registers, which it spills: 194 to 243 of them,
        // 400 to 431 with 4, 8, 4 and 8 here and in the other three, where the round takes 115.0.)
        SrcList src{llist};
        select_emit<OP, 3>(src, c, pe.k, R, Eq, win_base, win_min, win_ready, kmin, P.S, A, pe.outoff,
                           &tau_next, &expect, &q_e, &t_k);
    } else {
        // The list outgrew LDS: its tail is read from global scratch.  (4 / 8 a thread: 1.2M elements at 1 % by one workgroup,
        // worker 53.6 / 56.5, printed state 88.0 / 92.3)
        SrcSplit src{llist, glist};
        select_emit<OP, 4>(src, c, pe.k, R, Eq, win_base, win_min, win_ready, kmin, P.S, A, pe.outoff,
                           &tau_next, &expect, &q_e, &t_k);
    }
    list_hints(A, j, tau_next, expect, q_e, t_k, tau_cur, kmin);
}

// ---------------------------------------------------------------------------
// the lists of a whole call in one launch (dgs_step.h)
// ---------------------------------------------------------------------------

// A unit's list, values and indices apart (the ranking of a long list reads the values alone): their first words in ord.
__device__ __forceinline__ uint32_t step_val(const StepUnit &u) { return 2u * u.ord0 + STEP_LINE; }
__device__ __forceinline__ uint32_t step_idx(const StepUnit &u) { return step_val(u) + u.cap; }
__device__ __forceinline__ uint2 *step_word(const SelectArgs &A, uint32_t ord0) { return A.ord + ord0 + 1u; }

// Whether a tensor of n elements has emitting workgroups in the launch.
__device__ __forceinline__ bool step_emits(const SelectArgs &A, uint32_t n) { return A.nemit != 0 && n >= SEG_MIN_N; }

// Where the ranking workgroup puts what does not fit its LDS list (as SrcSplit's tail: entry SEL_LDS_LIST comes first): the
// streaming pass's slots, which lie before ord and which nobody uses in such a launch, of the tiles that are wholly the tensor's.
// There are CAPT a tile, and the units' lists have fewer entries than that for all tiles but the tensor's two outer ones, so
// that what they hold always fits.
__device__ __forceinline__ uint2 *step_tail(const SelectArgs &A, const TensorDesc &td)
{
    static_assert(SEL_LDS_LIST >= 2u * CAPT, "the outer tiles");
    return A.ord - (size_t)(A.ntiles - (td.off + TILE - 1u) / TILE) * CAPT - SEL_LDS_LIST;
}

// put(position, index, value) for every entry of a tensor's lists (KEYS: the index is not read), in any order.  16 lanes take a
// unit, a lane four entries with one load past the L2: such a load takes a compute unit some 20 ns whatever its width
// (16 K keys of 256 units, a wavefront per unit and 4 bytes a lane: 11 us; so 3 to 4).
template <bool KEYS, class Put>
__device__ __forceinline__ void step_gather(const SelectArgs &A, uint32_t first, uint32_t units, const uint32_t *pbase, Put put)
{
    constexpr uint32_t C = 2;                 // chunks of 64 entries of each of them in flight
    const uint32_t quarter = threadIdx.x >> 4, lane = threadIdx.x & 15u;
    const StepUnit u_first = A.steptab[first], u_last = A.steptab[first + units - 1u];
    const uint32_t *words = (const uint32_t *)A.ord;
    for (uint32_t u0 = 0; u0 < units; u0 += SEL_THREADS / 16u) {
        const uint32_t u = u0 + quarter;
        if (u >= units) break;
        const uint32_t at = pbase[u], n = pbase[u + 1u] - at;
        // (the lists of a tensor are equally far apart, and equally long but for the last)
        const uint32_t val = step_val(u_first) + 2u * u * u_first.rows * 4u * CAPT, idx = val + (u + 1u < units ? u_first.cap : u_last.cap);
        for (uint32_t q0 = 4u * lane; q0 < n; q0 += 64u * C) {
            uint4 v[C], x[C];
#pragma unroll
            for (uint32_t c = 0; c < C; ++c) {
                v[c] = x[c] = make_uint4(0u, 0u, 0u, 0u);
                if (q0 + 64u * c >= n) continue;      // (the last load of a list may read up to three words behind it: there is room)
                v[c] = ld_dev16(words, val + q0 + 64u * c);
                if (!KEYS) x[c] = ld_dev16(words, idx + q0 + 64u * c);
            }
#pragma unroll
            for (uint32_t c = 0; c < C; ++c) {
                const uint32_t q = q0 + 64u * c;
                if (q < n) put(at + q, x[c].x, v[c].x);
                if (q + 1u < n) put(at + q + 1u, x[c].y, v[c].y);
                if (q + 2u < n) put(at + q + 2u, x[c].z, v[c].z);
                if (q + 3u < n) put(at + q + 3u, x[c].w, v[c].w);
            }
        }
    }
}

// A pull of a tensor with emitting workgroups whose list its ranking workgroup cannot hold, or whose k-th key lies beyond the hinted
// window (a row that has waited long): the keys are read three times, for 12 bits, 11 and 8, and the exact
// one goes on to those workgroups.  21 K keys: 10 us.  (Cut down to what fits, or collected again by the tensor's parts, 100.)
template <int OP>
__device__ __forceinline__ void step_rank(const SelectArgs &A, const TensorDesc &td, const PlanEntry &pe, uint32_t j, uint32_t first, uint32_t units,
                                          uint32_t c, uint32_t tau_cur, uint32_t hint2_cur, PartShared &P)
{
    const uint32_t tid = threadIdx.x;
    constexpr uint32_t MID = 11, LOW = HSHIFT - MID;       // bits of the second pass, for the k-th key and the hinted rank, and of the third
    static_assert(HBINS <= sizeof(P.S.h) / 4 && 2u << MID <= HBINS, "a histogram for each pass");
    auto count = [&](auto f) {                       // f(key), into cleared counters
        __syncthreads();
        for (uint32_t b = tid; b < HBINS; b += SEL_THREADS) P.S.h[b] = 0;
        __syncthreads();
        step_gather<true>(A, first, units, P.pbase, [&](uint32_t, uint32_t, uint32_t v) { f(v & 0x7FFFFFFFu); });
    };
    uint32_t Eq = 0;
    const uint32_t R = hint_rank<OP>(td, pe, false, c, hint2_cur, A.m, A.young, &Eq);
    const bool measurable = R != 0 && c >= R;
    count([&](uint32_t key) { atomicAdd(&P.S.h[key >> HSHIFT], 1u); });
    find_ranks<HBINS, SEL_WAVES>(P.S.h, pe.k, measurable ? R : pe.k, 0u, P.S.rowsum, P.S.res);
    const uint32_t top = (uint32_t)P.S.res[0], r1 = (uint32_t)P.S.res[1], edge = (uint32_t)P.S.res[2], r1_hint = (uint32_t)P.S.res[3];
    count([&](uint32_t key) {
        const uint32_t hi = key >> HSHIFT, mid = (key >> LOW) & ((1u << MID) - 1u);
        if (hi == top) atomicAdd(&P.S.h[mid], 1u);
        else if (hi == edge) atomicAdd(&P.S.h[(1u << MID) + mid], 1u);
    });
    find_ranks<(1 << MID), SEL_WAVES>(P.S.h, r1, (measurable && edge == top) ? r1_hint : r1, 0u, P.S.rowsum, P.S.res);
    const uint32_t pfx = (top << MID) | (uint32_t)P.S.res[0], r2 = (uint32_t)P.S.res[1];
    uint32_t bin = (uint32_t)P.S.res[2], rank = (uint32_t)P.S.res[3], *hist = P.S.h;
    if (edge != top) {
        __syncthreads();
        hist += 1u << MID;
        find_ranks<(1 << MID), SEL_WAVES>(hist, r1_hint, 0u, 0u, P.S.rowsum, P.S.res);
        bin = (uint32_t)P.S.res[0];
        rank = (uint32_t)P.S.res[1];
    }
    const uint32_t expect = measurable ? R - rank + hist[bin] : 0u;
    count([&](uint32_t key) {
        if ((key >> LOW) == pfx) atomicAdd(&P.S.h[key & ((1u << LOW) - 1u)], 1u);
    });
    find_ranks<(1 << LOW), SEL_WAVES>(P.S.h, r2, 0u, 0u, P.S.rowsum, P.S.res);
    const uint32_t T = (pfx << LOW) | (uint32_t)P.S.res[0], rT = (uint32_t)P.S.res[1];
    if (tid == 0) {
        st_dev(&A.segstate[j].key, make_uint2(rT, KEY_READY | T));
        atomicAdd(&A.stats->candidates, (unsigned long long)c);
        if (c > SEL_LIST_HARD) atomicAdd(&A.stats->repaired_tensors, 1ull);
    }
    list_hints(A, j, measurable ? max((edge << HSHIFT) | (bin << LOW), 1u) : 0u, expect, 0u, T, tau_cur, 0xFFFFFFFFu);
}

// The candidates of a tensor of several parts, addressed by list position through the parts'
// global lists (pbase: first position of every part, in LDS).
struct SrcParts {
    static constexpr bool AGG = true;
    const uint2 *ord;
    const uint32_t *pbase;     // LDS: first list position of every part
    const uint32_t *pofs;      // LDS: where every part's list starts in ord
    uint32_t nseg;
    __device__ __forceinline__ uint2 get(uint32_t p) const
    {
        uint32_t lo = 0, hi = nseg;       // last part whose first position is <= p
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (pbase[mid] <= p) lo = mid;
            else hi = mid;
        }
        return ld_dev(&ord[(size_t)pofs[lo] + (p - pbase[lo])]);
    }
    __device__ __forceinline__ uint32_t bits(uint32_t p) const { return get(p).y; }
    __device__ __forceinline__ uint32_t index(uint32_t p) const { return get(p).x; }
};

// TRIM: a candidate list that is complete but too long for one workgroup is cut down to what a
// fresh collection would have found.  The list's own key histogram (bits [30:20]) gives the
// threshold -- the lower edge of the bucket that holds rank pe.k2 -- and the entries at or above
// it are moved up in list order into llist / glist.  No second pass over the tensor.  Returns the
// new count, or 0 (nothing moved) if that is still beyond list_max; tau is raised to the new
// threshold.  A success is published to `verdict` before the entries are moved.
//   In place: an entry never moves to a later position, and every turn has read its entries
//   before it writes any, so both an LDS list and the tail that spills into the first unit's
//   global list are only ever written where they have been read.
template <class Src>
__device__ __forceinline__ uint32_t trim_list(const SelectArgs &A, const Src &src, uint32_t c, uint32_t list_max,
                                              const PlanEntry &pe, uint32_t *verdict, PartShared &P, uint2 *llist,
                                              uint2 *glist, uint32_t &tau)
{
    const uint32_t tid = threadIdx.x;
    constexpr uint32_t GU = 8;      // entries per thread in flight
    for (uint32_t b = tid; b < 2048; b += SEL_THREADS) P.S.h[b] = 0;
    __syncthreads();
    for (uint32_t q0 = 0; q0 < c; q0 += GU * SEL_THREADS) {
        uint32_t key[GU];
#pragma unroll
        for (uint32_t u = 0; u < GU; ++u) {
            const uint32_t q = q0 + u * SEL_THREADS + tid;
            key[u] = (q < c) ? (src.bits(q) & 0x7FFFFFFFu) : 0u;
        }
#pragma unroll
        for (uint32_t u = 0; u < GU; ++u)
            if (key[u] != 0) atomicAdd(&P.S.h[key[u] >> 20], 1u);
    }
    find_ranks<2048, SEL_WAVES>(P.S.h, pe.k2, pe.k, 0u, P.S.rowsum, P.S.res);
    const int b2 = P.S.res[0];
    // (rank k2 beyond the nonzero keys of the list: nothing to cut, the count below says so)
    const uint32_t t = max((b2 > 0) ? ((uint32_t)b2 << 20) : 1u, tau);    // nothing below tau is in the list
    uint32_t reach = 0;      // entries at or above t: whole buckets, by construction
    for (uint32_t b = tid; b < 2048; b += SEL_THREADS)
        if (b >= (t >> 20)) reach += P.S.h[b];
    __syncthreads();
    const uint32_t c2 = block_sum<SEL_WAVES>(reach, P.S.wsum);
    __syncthreads();
    if (c2 < pe.k || c2 > list_max) return 0u;
    if (verdict && tid == 0) st_dev(verdict, 0x100u | (uint32_t)SEG_DONE);
    uint32_t run = 0;
    for (uint32_t q0 = 0; q0 < c; q0 += GU * SEL_THREADS) {      // GU consecutive entries per thread
        uint2 e[GU];
        uint32_t keep = 0;
#pragma unroll
        for (uint32_t u = 0; u < GU; ++u) {
            const uint32_t q = q0 + tid * GU + u;
            e[u] = (q < c) ? src.get(q) : make_uint2(0, 0);
        }
#pragma unroll
        for (uint32_t u = 0; u < GU; ++u) {
            const uint32_t q = q0 + tid * GU + u;
            if (q < c && (e[u].y & 0x7FFFFFFFu) >= t) keep |= 1u << u;
        }
        uint32_t tot;
        uint32_t pos = run + block_excl_scan<SEL_WAVES>((uint32_t)__popcll((unsigned long long)keep), P.S.wsum, tot);
#pragma unroll
        for (uint32_t u = 0; u < GU; ++u) {
            if ((keep >> u) & 1u) {
                if (pos < c2) put_entry(llist, glist, pos, e[u]);
                ++pos;
            }
        }
        run += tot;
    }
    wait_mem();
    __syncthreads();
    if (tid == 0 && run != c2) atomicAdd(&A.stats->internal_errors, 1ull);      // the two passes disagree
    tau = t;
    return c2;
}

// What the workgroup that completes a tensor's candidate lists does with them (`round` 0: the
// streaming pass's candidates, 1: re-collected with a fresh threshold).  Returns the tensor's
// status: SEG_DONE, SEG_ACTIVE / SEG_LISTS / SEG_ZERO (the chain kernels go on), or SEG_PENDING (round 0
// only: collect again).
//   multi: the lists are global lists of several units -- the tensor's parts (by_parts: counts
//   in segcnt) or its join groups (counts in grpcnt) -- and are gathered here; otherwise the
//   one list is in llist / glist (or, for a tensor that takes the chain, still in its tiles, and
//   in round 1 in its global list only) with count c0, overflow ovf0, smallest key (or a lower bound of it) kmin0, and --
//   win_counted -- the window histogram counted on the way.
//   verdict: where the outcome is published for the re-collecting workgroups of the launch
//   (null: nobody waits); a success is published as soon as it is certain, before the work.
//   tau_cur, tprev_cur: the threshold the lists were collected with and the anchor of the window
//   histograms (handed in: in round 1 they were published by another workgroup of this launch).
template <int OP, int FORM>
__device__ __forceinline__ uint32_t tensor_select(const SelectArgs &A, const TensorDesc &td, const PlanEntry &pe,
                                                  uint32_t j, int round, bool multi, bool by_parts, uint32_t c0,
                                                  bool ovf0, uint32_t kmin0, uint32_t tau_cur, uint32_t tprev_cur,
                                                  uint32_t win_join, bool win_counted, uint32_t *verdict,
                                                  PartShared &P, uint2 *llist)
{
    constexpr bool HERE = FORM == FORM_CHAIN;
    const uint32_t tid = threadIdx.x;
    const uint32_t tlo = td.off / TILE;
    uint2 *glist = A.ord + (size_t)(tlo + j) * CAPT;      // = the first part's list
    const bool exact_mode = A.exact_mode || round != 0;
    const uint32_t hint2_cur = A.write_hint ? A.hint2[j] : 0u;
    const uint32_t nunits = by_parts ? td.nseg : td.ngrp;
    const SegDesc *units = by_parts ? A.segtab + td.seg_first : A.grptab + td.grp_first;
    const uint32_t *ucnt = by_parts ? A.segcnt + td.seg_first : A.grpcnt + td.grp_first;
    const bool have_pbase = nunits <= SEG_MAX_PER_TENSOR;
    // The longest list this workgroup selects from.  A tensor of several parts is gathered in
    // place: what does not fit the LDS list goes to the first part's global list, which must
    // end before the second part's begins.
    const uint32_t list_max = multi ? max(SEL_LDS_LIST, min(SEL_LIST_HARD, units[0].ntiles * CAPT))
                                    : SEL_LIST_HARD;
    uint32_t c = c0, kmin = kmin0;
    bool ovf = ovf0;
    if (multi) {
        // counts of the units -> list positions
        uint32_t o = 0;
        c = 0;
        for (uint32_t s0 = 0; s0 < nunits; s0 += SEL_THREADS) {
            const uint32_t s = s0 + tid;
            uint32_t cnt = (s < nunits) ? ld_dev(&ucnt[s]) : 0u;
            if (cnt >> 31) o = 1;
            cnt &= 0x7FFFFFFFu;
            uint32_t tot;
            const uint32_t ex = block_excl_scan<SEL_WAVES>(cnt, P.S.wsum, tot);
            if (s < nunits && have_pbase) {
                P.pbase[s] = c + ex;
                P.pofs[s] = (units[s].tile0 + j) * CAPT;   // below 2^32: n < 2^32
            }
            c += tot;
        }
        if (tid == 0 && have_pbase) P.pbase[nunits] = c;
        ovf = __syncthreads_or((int)o) != 0;
    }
    uint32_t status = 0;
    bool early = false;      // the verdict went out before the work
    if (pe.seg) status = window_step<OP, HERE>(A, td, pe, j, c, ovf, tau_cur, tprev_cur, hint2_cur, exact_mode, round != 0, P);
    // every nonzero is in the lists
    const bool zerofill = !ovf && c < pe.k && tau_cur <= 1u && (!multi || have_pbase);
    if (status == 0 && zerofill) {
        // the message is completed with the tensor's lowest-index zeros
        early = true;
        status = SEG_DONE;
        if (verdict && tid == 0) st_dev(verdict, 0x100u | (uint32_t)SEG_DONE);
        if (pe.seg && round == 0) {
            // the candidates are still in their tiles, and the chain's emission goes through those anyway
            status = SEG_ZERO;
            if (tid == 0) {
                SegState *st = &A.segstate[j];
                st->r2 = pe.k - c;
                st->pfx = 0;
                atomicAdd(&A.stats->segmented_tensors, 1ull);
            }
        } else if (multi) {
            zero_fill_emit<OP, written<OP, FORM>()>(SrcParts{A.ord, P.pbase, P.pofs, nunits}, c, td, pe, A, P.S.wsum);
        } else if (pe.seg) {
            zero_fill_emit<OP, written<OP, FORM>()>(SrcList{glist}, c, td, pe, A, P.S.wsum);
        } else if (c > SEL_LDS_LIST) {
            zero_fill_emit<OP, written<OP, FORM>()>(SrcSplit{llist, glist}, c, td, pe, A, P.S.wsum);
        } else {
            zero_fill_emit<OP, written<OP, FORM>()>(SrcList{llist}, c, td, pe, A, P.S.wsum);
        }
        if (A.write_hint && tid == 0) {
            A.tau[j] = 1u;
            A.hint2[j] = 0u;
            A.tprev[j] = 0u;
        }
        if (tid == 0) atomicAdd(&A.stats->candidates, (unsigned long long)c);
    } else if (!pe.seg && !ovf && c >= pe.k && c <= list_max && (!multi || have_pbase)) {
        early = true;
        if (verdict && tid == 0) st_dev(verdict, 0x100u | (uint32_t)SEG_DONE);
        if (multi) {
            // gather the parts' lists into one (positions beyond the LDS list land in the first
            // part's global list: on dead space, or on the very entry that is being moved)
            const bool count_win = (win_join != 0xFFFFFFFFu);   // the hinted window is counted on the way
            for (uint32_t b = tid; b < WIN_BINS; b += SEL_THREADS) P.S.h[b] = 0;
            if (tid == 0) P.S.kmin = 0xFFFFFFFFu;
            __syncthreads();
            const SrcParts src{A.ord, P.pbase, P.pofs, nunits};
            uint32_t km = 0xFFFFFFFFu;
            constexpr uint32_t GU = 8;      // entries per thread in flight
            for (uint32_t q0 = 0; q0 < c; q0 += GU * SEL_THREADS) {
                uint2 e[GU];
#pragma unroll
                for (uint32_t u = 0; u < GU; ++u) {
                    const uint32_t q = q0 + u * SEL_THREADS + tid;
                    e[u] = (q < c) ? src.get(q) : make_uint2(0, 0);
                }
#pragma unroll
                for (uint32_t u = 0; u < GU; ++u) {
                    const uint32_t q = q0 + u * SEL_THREADS + tid;
                    if (q < c) {
                        put_entry(llist, glist, q, e[u]);
                        km = min(km, e[u].y & 0x7FFFFFFFu);
                        if (count_win) window_count<OP>(P.S.h, win_join, e[u].y & 0x7FFFFFFFu);
                    }
                }
            }
            km = wave_min_to_last(km);
            if (lane_id() == 63) atomicMin(&P.S.kmin, km);
            wait_mem();
            __syncthreads();
            kmin = P.S.kmin;
        }
        list_select<OP>(A, td, pe, j, c, kmin, tau_cur, hint2_cur, win_join,
                        multi ? (win_join != 0xFFFFFFFFu) : win_counted, exact_mode, P, llist, glist);
        if (tid == 0) atomicAdd(&A.stats->candidates, (unsigned long long)c);
        status = SEG_DONE;
    }
    if (status == 0 && !pe.seg && !ovf && (!multi || have_pbase) && c >= pe.k && c > list_max) {
        // Every candidate is in the lists, there are only too many of them for one workgroup
        // (the threshold has fallen behind a scale that grew): trimmed on the spot.
        uint32_t tau_new = tau_cur;
        const uint32_t c2 = multi ? trim_list(A, SrcParts{A.ord, P.pbase, P.pofs, nunits}, c, list_max, pe, verdict, P,
                                              llist, glist, tau_new)
                                  : trim_list(A, SrcSplit{llist, glist}, c, list_max, pe, verdict, P, llist, glist, tau_new);
        if (c2 != 0) {
            early = true;
            if (tid == 0) {
                atomicAdd(&A.stats->candidates, (unsigned long long)c2);
                if (round == 0) atomicAdd(&A.stats->repaired_tensors, 1ull);
            }
            // (smallest key unknown: the threshold is a lower bound of it, and the window is
            // counted from the list)
            list_select<OP>(A, td, pe, j, c2, tau_new, tau_new, hint2_cur, 0xFFFFFFFFu, false, true, P, llist, glist);
            status = SEG_DONE;
        }
    }
    if (status == 0) status = (round == 0 && A.repair) ? (uint32_t)SEG_PENDING : (uint32_t)SEG_FALLBACK;
    if (status == SEG_FALLBACK) {
        if (tid == 0) {
            atomicAdd(&A.stats->fallback_tensors, 1ull);
            atomicAdd(&A.stats->fallback_elems, (unsigned long long)td.n);
        }
        dense_select<OP, written<OP, FORM>()>(A, td, pe, j, tau_cur, P, llist);
        status = SEG_DONE;
    } else if (round != 0 && tid == 0) {
        atomicAdd(&A.stats->repaired_tensors, 1ull);
    }
    if (tid == 0) A.segstate[j].status = status;
    if (HERE && pe.seg && status != SEG_PENDING && status != SEG_ACTIVE) {      // the slabs of this launch go on
        wait_mem();
        __syncthreads();
        if (tid == 0) {
            SegState *st = &A.segstate[j];
            const bool done = status == SEG_DONE;
            st_dev(&st->chain, make_uint2(done ? 0u : st->r2, (status << CHAIN_STATUS_SHIFT) | (done ? 0u : st->pfx)));
        }
    }
    if (verdict && !early) {
        wait_mem();
        __syncthreads();
        if (tid < 64) {
            // A rejected join may have spilled list entries with cached stores into the very
            // lists that other workgroups now fill again: written back before they start, so
            // that no older copy in this L2 shadows theirs.
            if (status == SEG_PENDING) release_dev();
            if (tid == 0) st_dev(verdict, 0x100u | status);
        }
    }
    return status;
}

// RE-HISTOGRAM (role 1) or RE-COLLECTION (role 2) of one part of a tensor that the JOIN left
// pending (the caller has seen that verdict).
template <int OP, int FORM>
__device__ __forceinline__ void recollect_part(const SelectArgs &A, uint32_t role, uint32_t part, PartShared &P,
                                               uint2 *llist)
{
    const uint32_t tid = threadIdx.x;
    const SegDesc sd = A.segtab[part];
    const uint32_t j = sd.j;
    const TensorDesc td = A.tdesc[j];
    PlanEntry pe = A.plan[j];
    if (FORM == FORM_STEP) pe.seg = 0;
    const bool multi = td.nseg > 1;
    SegState *st = &A.segstate[j];
    uint2 *plist = A.ord + (size_t)(sd.tile0 + j) * CAPT;       // this part's list
    const uint32_t part_cap = sd.ntiles * CAPT;
    if (!multi) return;
    uint32_t *gh = A.ghist + (size_t)j * HBINS;
    if (role == 1) {
        uint32_t *lh = (uint32_t *)llist;
        dense_hist<OP, written<OP, FORM>()>(A, td, sd, lh);
        for (uint32_t b = tid; b < HBINS; b += SEL_THREADS) {
            const uint32_t v = lh[b];
            if (v) atomicAdd(&gh[b], v);
        }
        if (!arrive_last(&st->arrive[1], td.nseg, &P.bc)) return;
        for (uint32_t b = tid; b < HBINS; b += SEL_THREADS) {
            const uint32_t v = ld_dev(&gh[b]);
            lh[b] = v;
            if (v) st_dev(&gh[b], 0u);
        }
        uint32_t tau_new = 0, tprev_new = 0;
        pick_from_hist<SEL_WAVES>(lh, pe, P.S.rowsum, P.S.res, tau_new, tprev_new);
        if (tid == 0) {
            st_dev(&A.tau[j], tau_new);
            st_dev(&A.tprev[j], tprev_new);
        }
        wait_mem();
        __syncthreads();
        if (tid == 0) st_dev(&st->tau_ready, 1u);
        return;
    }
    const uint32_t ready = wait_word(&st->tau_ready, A.spin_limit, &P.bc);
    if (tid == 0) {
        if (ready == 0) atomicAdd(&A.stats->internal_errors, 1ull);
        reader_done(&st->seen[1], td.nseg, 1u, &st->tau_ready);
    }
    if (ready == 0) return;
    const uint32_t tau_new = ld_dev(&A.tau[j]);
    const uint32_t tprev_new = ld_dev(&A.tprev[j]);
    const uint32_t win2 = seg_window_base(tau_new, tprev_new);
    for (uint32_t b = tid; b < 2048; b += SEL_THREADS) P.S.h[b] = 0;
    __syncthreads();
    uint32_t c2;
    if (pe.seg) {
        c2 = dense_compact<OP, written<OP, FORM>()>(A, td, sd, tau_new, part_cap, P, [&](uint32_t pos, uint2 e) {
            st_dev(&plist[pos], e);
            const uint32_t hi12 = (e.y & 0x7FFFFFFFu) >> SEG_LOWBITS;
            const uint32_t w = (hi12 > win2) ? (hi12 - win2) : 0u;
            atomicAdd(&P.S.h[min(w, SEG_WBINS - 1u)], 1u);
        });
        __syncthreads();
        if (c2 <= part_cap) {
            for (uint32_t b = tid; b < SEG_WBINS; b += SEL_THREADS) {
                const uint32_t v = P.S.h[b];
                if (v) atomicAdd(&gh[b], v);
            }
        }
    } else {
        c2 = dense_compact<OP, written<OP, FORM>()>(A, td, sd, tau_new, part_cap, P, [&](uint32_t pos, uint2 e) { st_dev(&plist[pos], e); });
    }
    if (tid == 0) {
        st_dev(&A.segcnt[part], min(c2, 0x7FFFFFFFu) | (c2 > part_cap ? 0x80000000u : 0u));
    }
    if (!arrive_last(&st->arrive[2], td.nseg, &P.bc)) return;
    tensor_select<OP, FORM>(A, td, pe, j, 1, true, true, 0u, false, 0xFFFFFFFFu, tau_new, tprev_new, 0xFFFFFFFFu, false,
                      nullptr, P, llist);
}

// One RE-HISTOGRAM or RE-COLLECTION workgroup, number b of 2 nb.
template <int OP, int FORM>
__device__ __forceinline__ void standby_block(const SelectArgs &A, uint32_t b, uint32_t nb, PartShared &P, uint2 *llist)
{
    const uint32_t tid = threadIdx.x;
    const uint32_t role = (b < nb) ? 1u : 2u;
    const uint32_t first = (role == 1) ? b : b - nb;
    // the verdicts of the tensors these parts belong to: lane i waits for part i's tensor and
    // signs off for that part
    if (tid < B_GROUP_MAX) P.vbuf[tid] = 0;
    __syncthreads();
    const uint32_t mypart = first + tid * nb;
    if (tid < A.bgroup && mypart < A.nparts) {
        const SegDesc sd = A.segtab[mypart];
        if (A.tdesc[sd.j].nseg > 1) {
            SegState *st = &A.segstate[sd.j];
            uint32_t v = 0;
            for (uint32_t spin = 0; spin < A.spin_limit; ++spin) {
                v = ld_dev(&st->verdict);
                if (v != 0) break;
                __builtin_amdgcn_s_sleep(4);
            }
            if (v == 0) atomicAdd(&A.stats->internal_errors, 1ull);   // gave up waiting
            reader_done(&st->seen[0], 2u * A.tdesc[sd.j].nseg, 1u, &st->verdict);
            P.vbuf[tid] = v;
        }
    }
    __syncthreads();
    for (uint32_t i = 0; i < A.bgroup; ++i)
        if (__builtin_expect((P.vbuf[i] & 0xFFu) == SEG_PENDING, 0)) recollect_part<OP, FORM>(A, role, first + i * nb, P, llist);
}

// A tensor of one part whose prediction failed: its workgroup collects again on the spot.
template <int OP, int FORM>
__device__ __forceinline__ void recollect_here(const SelectArgs &A, const TensorDesc &td, const PlanEntry &pe, uint32_t j, PartShared &P,
                                               uint2 *llist)
{
    const uint32_t tid = threadIdx.x;
    const SegDesc sd = A.segtab[td.seg_first];
    uint2 *plist = A.ord + (size_t)(sd.tile0 + j) * CAPT;
    const uint32_t part = td.seg_first, part_cap = sd.ntiles * CAPT;
    uint32_t *lh = (uint32_t *)llist;
    dense_hist<OP, written<OP, FORM>()>(A, td, sd, lh);
    uint32_t tau_new = 0, tprev_new = 0;
    pick_from_hist<SEL_WAVES>(lh, pe, P.S.rowsum, P.S.res, tau_new, tprev_new);
    if (tid == 0) {
        A.tau[j] = tau_new;
        st_dev(&A.tprev[j], tprev_new);      // (the chain's ranking writes this word in the same launch)
        P.bc = tau_new;
    }
    __syncthreads();
    tau_new = P.bc;
    for (uint32_t b = tid; b < 2048; b += SEL_THREADS) P.S.h[b] = 0;
    __syncthreads();
    const uint32_t win2 = seg_window_base(tau_new, tprev_new);
    const uint32_t cap = pe.seg ? part_cap : min(part_cap, SEL_LIST_HARD);
    uint32_t c2;
    if (pe.seg) {
        c2 = dense_compact<OP, written<OP, FORM>()>(A, td, sd, tau_new, cap, P, [&](uint32_t pos, uint2 e) {
            st_dev(&plist[pos], e);
            const uint32_t hi12 = (e.y & 0x7FFFFFFFu) >> SEG_LOWBITS;
            const uint32_t w = (hi12 > win2) ? (hi12 - win2) : 0u;
            atomicAdd(&P.S.h[min(w, SEG_WBINS - 1u)], 1u);
        });
        __syncthreads();
        if (c2 <= cap) {
            uint32_t *gh = A.ghist + (size_t)j * HBINS;
            for (uint32_t b = tid; b < SEG_WBINS; b += SEL_THREADS) {
                const uint32_t v = P.S.h[b];
                if (v) atomicAdd(&gh[b], v);
            }
            if (tid == 0) st_dev(&A.segcnt[part], c2);
        }
    } else {
        uint2 *glist = plist;
        c2 = dense_compact<OP, written<OP, FORM>()>(A, td, sd, tau_new, cap, P, [&](uint32_t pos, uint2 e) { put_entry(llist, glist, pos, e); });
    }
    wait_mem();
    __syncthreads();
    // kmin unknown (0 keeps the window honest: it is counted again from the list)
    tensor_select<OP, FORM>(A, td, pe, j, 1, false, true, c2, c2 > cap, tau_new, tau_new, tprev_new, 0xFFFFFFFFu, false,
                      nullptr, P, llist);
}

// The chain's first part inside the selection's launch: the window histogram of a run of parts of a tensor.  The
// workgroup that arrives last for the tensor returns true.
__device__ __forceinline__ bool window_run(const SelectArgs &A, const SegDesc &run, const TensorDesc &td, uint32_t tau_cur,
                                           uint32_t tprev_cur, PartShared &P)
{
    const uint32_t tid = threadIdx.x, per = window_parts(td.nseg, A.window_max), nb = window_blocks(td.nseg, A.window_max);
    bool ovf;
    const uint32_t c = window_tiles(A, td, run.tile0, run.ntiles, seg_window_base(tau_cur, tprev_cur), P.S.h, P.S.wsum, ovf);
    uint2 *out = (uint2 *)part_hist(A, td, run.j, run.sidx / per);
    for (uint32_t b = tid; b < SEG_WBINS / 2; b += SEL_THREADS) st_dev(&out[b], make_uint2(P.S.h[2 * b], P.S.h[2 * b + 1]));
    if (tid == 0) st_dev(&A.segcnt[td.seg_first + run.sidx], c | (ovf ? 0x80000000u : 0u));
    return arrive_last(&A.segstate[run.j].arrive[0], nb, &P.bc);
}

}  // namespace dgs
