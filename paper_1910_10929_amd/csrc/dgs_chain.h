// The chain: tensors whose candidate lists are too long for one workgroup to join and select from.
// The candidates stay where the streaming pass has left them, tile by tile; one wavefront takes 8 or
// 16 tiles, all of their first 64 candidates in flight together, four tiles to an instruction, and the work is cut into
// slabs of CSLAB_TILES tiles, so that it fills the chip for any number of tensors.  Joining the
// candidates into one ordered list first, one workgroup per 4096 tiles, was bound by that
// workgroup: 92 us of a call on ResNet-50 shapes at 1 % without momentum (the whole selection now
// 31), 232 us at 1 % of 1e9 parameters.  At that size each pass reads 240 MB of
// candidates and the emission is bound by its scattered 4-byte stores (1e7 of them: 420 us).
//   window  per run of parts: window histogram of the candidates, in a slot of its own -- no atomics
//           between workgroups; one workgroup of the selection kernel adds a tensor's histograms up and leaves
//           the 19-bit prefix of the k-th key and its rank below it
//   finish  two workgroups per slab.  RANK counts the low 12 bits of the entries that share the
//           prefix; the one arriving last for a tensor ranks: the exact k-th key and how many of the
//           entries equal to it are taken.  EMIT awaits that, counts its winners, adds up what the
//           slabs before it have published, and writes its stretch of the message ("encode()" of
//           Algorithms 1-3) and the state fix-up (Eq. 12 / Eq. 6).  Ties need no list and no case
//           of their own.
// Waiting is for blocks with lower indices only.  The chip deals a launch's blocks out to its eight dies in turn and each die
// starts its share in order, so the lowest block that has not ended either runs, and waits for nobody, or is the next to
// start on a die whose earlier blocks of this launch have all ended.  That is progress as long as the die has room, which
// another launch may take: two at once stand still only if each fills a die with waiting blocks and holds
// back one that the other needs.  The bound on every wait (A.spin_limit) then ends it, counted as an internal error.
// Where there are few enough slabs all of that is part of the selection's launch (CHAIN_HERE), beside the joins of the
// other tensors; otherwise window and finish are launches of their own, before and behind it.
// A tensor whose prediction failed was collected again into one list per part by the selection
// kernel (SEG_LISTS); its slabs then take equal shares of those lists in place of their tiles.  A tensor
// with fewer nonzeros than k (SEG_ZERO) has its message completed with zeros by its slabs.
#pragma once
#include "dgs_slab.h"

namespace dgs {

constexpr uint32_t WINDOW_TPW = 16;       // tiles of one wavefront of k_list_window at a time

// The candidates of up to 64 consecutive tiles: lane i describes tile i.
struct WaveTiles {
    uint32_t t0;         // the first of them
    uint32_t n, start;   // candidates of the tensor, and where they start: in the tile (after those of a
                         // previous tensor), or in the ordered lists
    bool lists;
    int ovf;
};

__device__ __forceinline__ WaveTiles wave_tiles(const SelectArgs &A, const TensorDesc &td, uint32_t t0, uint32_t nt,
                                                bool lists, uint32_t part)
{
    const uint32_t lane = lane_id();
    WaveTiles w;
    w.t0 = t0;
    w.lists = lists;
    w.n = w.start = 0;
    w.ovf = 0;
    if (!lists) {
        const uint32_t cnt = (lane < nt) ? A.tile_cnt[t0 + lane] : 0u;
        tile_counts(cnt, t0 + lane, td.off / TILE, (td.off % TILE) != 0, w.n, w.start, w.ovf);
    } else if (lane < nt) {
        const SegDesc ps = A.segtab[part];
        const uint64_t cnt = ld_dev(&A.segcnt[part]) & 0x7FFFFFFFu, i = t0 + lane - ps.tile0;
        const uint64_t lo = cnt * i / ps.ntiles, hi = cnt * (i + 1) / ps.ntiles;
        w.n = (uint32_t)(hi - lo);
        w.start = (ps.tile0 + ps.j) * CAPT + (uint32_t)lo;      // below 2^32: n < 2^32
    }
    return w;
}

__device__ __forceinline__ uint32_t tile_n(const WaveTiles &w, uint32_t i)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)w.n, (int)i);
}

// Candidate q of tile i (q below its count).
__device__ __forceinline__ uint2 tile_get(const SelectArgs &A, const WaveTiles &w, uint32_t i, uint32_t start, uint32_t q)
{
    const uint32_t p = start + q;
    if (w.lists) return ld_dev(&A.ord[p]);
    return *candidate(A, w.t0 + i, p);
}

// A wavefront takes four tiles at a time, 16 lanes each, and a lane two of a tile's candidates: one 16-byte load for
// the first NEAR of each, and one for as many more where one of the four tiles has more.  (64 lanes on one tile, a
// candidate each: every instruction of these passes works on the 10 to 30 candidates of one tile then, and
// they are bound by instructions: a round on one tensor of 2^20 elements at 1 % 85.0 us, 73.4 so; the window histogram of
// 1e9 parameters at 1 % 122 us, 73 so.)
static_assert(NEAR == 32 && HEAD % 2 == 0, "16 lanes, two candidates each");
constexpr uint32_t PAIRS = 2 * NEAR;      // candidates of a tile that are held in registers

__device__ __forceinline__ uint32_t shuffle(uint32_t v, uint32_t from)
{
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * from), (int)v);
}

// This lane's candidates of tile 4 i + lane / 16: positions at, at + 1, NEAR + at and NEAR + at + 1 of its list, of which
// n are the tensor's from `start` on (for the ordered lists: start 0, positions count from the share's first).
struct LanePair {
    uint32_t n, start, at;
    __device__ __forceinline__ bool has(uint32_t x) const { return at + x - start < n; }
};

__device__ __forceinline__ LanePair lane_pair(const WaveTiles &w, uint32_t i)
{
    const uint32_t lane = lane_id(), t = 4u * i + (lane >> 4);
    LanePair p;
    p.n = shuffle(w.n, t);
    p.start = w.lists ? 0u : shuffle(w.start, t);
    p.at = 2u * (lane & 15u);
    return p;
}

// The tiles (bit i: tile i) that hold candidates at position `from` or behind it.
__device__ __forceinline__ uint64_t deep_tiles(const WaveTiles &w, uint32_t from)
{
    return ballot64(w.n != 0 && (w.lists ? 0u : w.start) + w.n > from);
}
__device__ __forceinline__ bool deep_group(uint64_t deep, uint32_t i) { return ((deep >> (4u * i)) & 0xFull) != 0; }

// Those candidates for NT tiles: e[i][0] the first NEAR positions, e[i][1] the next.
template <uint32_t NT>
__device__ __forceinline__ void tile_firsts(const SelectArgs &A, const WaveTiles &w, uint4 (&e)[NT / 4][2])
{
    const uint32_t lane = lane_id();
    static_assert(NT % 4 == 0, "four tiles at a time");
    const uint64_t deep = deep_tiles(w, NEAR);
#pragma unroll
    for (uint32_t i = 0; i < NT / 4; ++i) {
        LanePair p = lane_pair(w, i);
        const uint32_t from = w.lists ? shuffle(w.start, 4u * i + (lane >> 4)) : 0u;
#pragma unroll
        for (uint32_t u = 0; u < 2; ++u, p.at += NEAR) {
            e[i][u] = make_uint4(0u, 0u, 0u, 0u);
            if (u == 1 && !deep_group(deep, i)) continue;
            if (w.lists) {
                const uint2 a = p.has(0) ? ld_dev(&A.ord[from + p.at]) : make_uint2(0u, 0u);
                const uint2 b = p.has(1) ? ld_dev(&A.ord[from + p.at + 1u]) : make_uint2(0u, 0u);
                e[i][u] = make_uint4(a.x, a.y, b.x, b.y);
            } else if (p.has(0) || p.has(1)) {
                e[i][u] = *(const uint4 *)candidate(A, w.t0 + 4u * i + (lane >> 4), p.at);      // (both in the same line)
            }
        }
    }
}

// f(entry) for every candidate, in no particular order (lanes diverge inside f).
template <uint32_t NT, class F>
__device__ __forceinline__ void each_candidate(const SelectArgs &A, const WaveTiles &w, const uint4 (&e)[NT / 4][2], F f)
{
    const uint32_t lane = lane_id();
    const uint64_t deep = deep_tiles(w, NEAR);
#pragma unroll
    for (uint32_t i = 0; i < NT / 4; ++i) {
        LanePair p = lane_pair(w, i);
        if (p.has(0)) f(make_uint2(e[i][0].x, e[i][0].y));
        if (p.has(1)) f(make_uint2(e[i][0].z, e[i][0].w));
        if (!deep_group(deep, i)) continue;
        p.at += NEAR;
        if (p.has(0)) f(make_uint2(e[i][1].x, e[i][1].y));
        if (p.has(1)) f(make_uint2(e[i][1].z, e[i][1].w));
    }
    for (uint64_t m = deep_tiles(w, PAIRS); m != 0; m &= m - 1ull) {
        const uint32_t i = (uint32_t)__ffsll((unsigned long long)m) - 1u, n = tile_n(w, i);
        const uint32_t start = (uint32_t)__builtin_amdgcn_readlane((int)w.start, (int)i);
        const uint32_t skip = w.lists ? PAIRS : PAIRS - min(start, PAIRS);
        for (uint32_t q = skip + lane; q < n; q += 64) f(tile_get(A, w, i, start, q));
    }
}

// How many of the candidates in tiles [tile0, tile0 + ntiles) of a tensor fall into each of `bins` buckets, into h (counters
// in LDS, zeroed here): bin(key).  Returns their number; `over`: a tile had overflowed.
template <class Bin>
__device__ __forceinline__ uint32_t count_tiles(const SelectArgs &A, const TensorDesc &td, uint32_t tile0, uint32_t ntiles,
                                                uint32_t *h, uint32_t bins, uint32_t *wsum, bool &over, Bin bin)
{
    const uint32_t tid = threadIdx.x, wave = uniform(tid >> 6);
    for (uint32_t b = tid; b < bins; b += SEL_THREADS) h[b] = 0;
    __syncthreads();
    uint32_t mine = 0;
    int ovf = 0;
    for (uint32_t t = wave * WINDOW_TPW; t < ntiles; t += SEL_WAVES * WINDOW_TPW) {
        const WaveTiles w = wave_tiles(A, td, tile0 + t, min(WINDOW_TPW, ntiles - t), false, 0u);
        mine += w.n;
        ovf |= w.ovf;
        uint4 e[WINDOW_TPW / 4][2];
        tile_firsts<WINDOW_TPW>(A, w, e);
        each_candidate<WINDOW_TPW>(A, w, e, [&](uint2 x) { atomicAdd(&h[bin(x.y & 0x7FFFFFFFu)], 1u); });
    }
    const uint32_t c = block_sum<SEL_WAVES>(mine, wsum);
    over = __syncthreads_or(ovf) != 0;
    return c;
}

// The window histogram: SEG_WBINS buckets of key >> SEG_LOWBITS from `win` on, what lies below in the first, beyond in the last.
__device__ __forceinline__ uint32_t window_tiles(const SelectArgs &A, const TensorDesc &td, uint32_t tile0, uint32_t ntiles,
                                                 uint32_t win, uint32_t *h, uint32_t *wsum, bool &over)
{
    return count_tiles(A, td, tile0, ntiles, h, SEG_WBINS, wsum, over, [&](uint32_t key) {
        const uint32_t hi = key >> SEG_LOWBITS;
        return min((hi > win) ? (hi - win) : 0u, SEG_WBINS - 1u);
    });
}

// Tiles of one wavefront of a slab.
constexpr uint32_t slab_tpw(uint32_t threads) { return CSLAB_TILES / (threads / 64) < 4 ? 4u : CSLAB_TILES / (threads / 64); }

struct FinishShared {
    alignas(8) uint32_t h[SEG_LBINS];      // (an emission stages its winners there)
    uint32_t rowsum[64];
    int res[6];
    uint32_t wtot[SEL_WAVES];
    uint32_t g, q, limit, bc;
    uint32_t pair[2];
};

// RANK (blocks below A.ncslabs): the low key bits of the slab's entries that share the prefix.
template <uint32_t THREADS>
__device__ __forceinline__ void rank_slab(const SelectArgs &A, uint32_t slab, const SegDesc &sd, const TensorDesc &td,
                                          SegState *st, uint32_t pfx, uint32_t r2, const WaveTiles &w,
                                          const uint4 (&e)[slab_tpw(THREADS) / 4][2], FinishShared &C)
{
    const uint32_t tid = threadIdx.x;
    uint32_t *glow = A.ghist + (size_t)sd.j * HBINS;
    if (tid == 0) slab_publish<false>(&A.slabs_done[slab], 0u, 0u, 0u);      // nothing published yet (complete before the arrival below)
    each_candidate<slab_tpw(THREADS)>(A, w, e, [&](uint2 x) {
        if (((x.y & 0x7FFFFFFFu) >> SEG_LOWBITS) == pfx) atomicAdd(&glow[x.y & (SEG_LBINS - 1u)], 1u);
    });
    if (!arrive_last(&st->arrive[3], td.ncs, &C.bc)) return;
    // the tensor's last slab: exact k-th key and tie budget
    for (uint32_t b = 2u * tid; b < SEG_LBINS; b += 2u * THREADS) {
        const uint2 v = ld_dev((const uint2 *)&glow[b]);
        C.h[b] = v.x;
        C.h[b + 1] = v.y;
        if (v.x | v.y) st_dev((uint2 *)&glow[b], make_uint2(0u, 0u));      // clean for the next use
    }
    find_ranks<SEG_LBINS, (int)(THREADS / 64)>(C.h, r2, 0u, 0u, C.rowsum, C.res);
    if (tid == 0) {
        // (a rank beyond what the slabs counted cannot happen: nothing is sent then, and it is reported)
        if (C.res[0] < 0) atomicAdd(&A.stats->internal_errors, 1ull);
        const uint32_t T = (C.res[0] < 0) ? 0x7FFFFFFFu : ((pfx << SEG_LOWBITS) | (uint32_t)C.res[0]);
        st_dev(&st->key, make_uint2((C.res[0] < 0) ? 0u : (uint32_t)C.res[1], KEY_READY | T));
        st_dev(&A.tprev[sd.j], T);
    }
}

// EMIT (the other blocks): ordered emission of the slab and the state fix-up.  A slab that gives up
// a wait, and every slab of the tensor behind it, emits nothing and leaves the state as it is.
template <int OP, uint32_t THREADS>
__device__ __forceinline__ void emit_slab(const SelectArgs &A, uint32_t slab, const SegDesc &sd, const TensorDesc &td,
                                          const PlanEntry &pe, SegState *st, const WaveTiles &w,
                                          const uint4 (&e)[slab_tpw(THREADS) / 4][2], FinishShared &C)
{
    constexpr uint32_t WAVES = THREADS / 64, CTPW = slab_tpw(THREADS);
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = uniform(tid >> 6);
    const uint2 key = wait_pair(&st->key, A.spin_limit, C.pair);
    if (key.y == 0) {
        if (tid == 0) {
            slab_publish<false>(&A.slabs_done[slab], SLAB_FAIL, 0u, 0u);
            atomicAdd(&A.stats->internal_errors, 1ull);
        }
        return;
    }
    const uint32_t T = uniform(key.y & ~KEY_READY), rT = uniform(key.x);
    // entries above T (low half) and equal to it (high half) of this wavefront: a few thousand at most
    uint32_t mine = 0;
    each_candidate<CTPW>(A, w, e, [&](uint2 x) {
        const uint32_t key = x.y & 0x7FFFFFFFu;
        mine += (key > T ? 1u : 0u) + (key == T ? 0x10000u : 0u);
    });
    const uint32_t sum = wave_sum(mine);
    if (lane == 0) C.wtot[wave] = sum;
    __syncthreads();
    uint32_t all;
    const uint32_t before = sum_waves<(int)WAVES>(C.wtot, all);
    if (wave == 0) {
        const bool head = (slab == td.cs_first);
        if (lane == 0) slab_publish<false>(&A.slabs_done[slab], head ? SLAB_SUM : SLAB_OWN, all & 0xFFFFu, all >> 16);
        uint32_t g, q;
        const bool known = slab_look_back<false>(A, slab, td.cs_first, [&](uint32_t i) { return &A.slabs_done[i]; }, g, q);
        if (lane == 0) {
            if (!head) slab_publish<false>(&A.slabs_done[slab], known ? SLAB_SUM : SLAB_FAIL, g + (all & 0xFFFFu), q + (all >> 16));
            C.limit = known ? pe.k : 0u;
            C.g = g;
            C.q = q;
            if (known && slab + 1 == td.cs_first + td.ncs &&                                        // the tensor's last slab
                (g + (all & 0xFFFFu) + rT != pe.k || q + (all >> 16) < rT))
                atomicAdd(&A.stats->internal_errors, 1ull);
        }
    }
    __syncthreads();
    uint32_t eq = C.q + (before >> 16);              // the tensor's ties seen so far: lowest index first, rT of them are taken
    uint32_t pos = C.g + (before & 0xFFFFu) + min(eq, rT);
    const uint32_t limit = C.limit;
    auto write = [&](uint32_t p, uint2 x, float was) {
        if (p >= limit) return;
        const float v = __uint_as_float(x.y);
        A.out_idx[pe.outoff + p] = x.x;
        A.out_val[pe.outoff + p] = v;
        if (!index_ok(A, x.x)) return;
        if (OP == SEL_WORKER) store_scattered(&A.state[x.x], A.m * v);
        else if (OP == SEL_PULL) store_scattered(&A.state[x.x], 0.0f);
        else store_scattered(&A.state[x.x], was + v);
    };
    constexpr uint32_t STAGED = SEG_LBINS / 2 / WAVES;            // entries of a wavefront in C.h
    uint2 *stage = (uint2 *)C.h + wave * STAGED;
    const uint64_t deep = deep_tiles(w, NEAR), deeper = deep_tiles(w, PAIRS);
#pragma unroll
    for (uint32_t i = 0; i < CTPW / 4; ++i) {                     // (wave-uniform, like all of this loop)
        if (!deep_group(deeper, i)) {
            // four tiles; in each, the lanes' pairs of the first NEAR positions come before those of the next
            const bool more = deep_group(deep, i);
            LanePair p = lane_pair(w, i);
            const uint64_t low = (1ull << (lane & 48u)) - 1ull, up = low | (0xFFFFull << (lane & 48u));
            bool v[4], f[4];
            uint64_t mk[4];
#pragma unroll
            for (uint32_t x = 0; x < 4; ++x) {
                const uint32_t bits = (x & 1u) ? e[i][x / 2].w : e[i][x / 2].y;
                if (x == 2) p.at += NEAR;
                v[x] = (x < 2 || more) && p.has(x & 1u);
                f[x] = v[x] && (bits & 0x7FFFFFFFu) == T;
                mk[x] = ballot64(f[x]);
            }
            auto rank = [&](uint32_t x) {                         // marked entries before entry x of this lane
                uint32_t r;
                if (x < 2) r = mbcnt64(mk[0]) + mbcnt64(mk[1]) + (uint32_t)(__popcll(mk[2] & low) + __popcll(mk[3] & low));
                else r = mbcnt64(mk[2]) + mbcnt64(mk[3]) + (uint32_t)(__popcll(mk[0] & up) + __popcll(mk[1] & up));
                return r + ((x & 1u) && f[x - 1] ? 1u : 0u);
            };
            uint32_t tied[4] = {0, 0, 0, 0};
            const bool ties = (mk[0] | mk[1] | mk[2] | mk[3]) != 0;
            if (ties) {
#pragma unroll
                for (uint32_t x = 0; x < 4; ++x) tied[x] = eq + rank(x);
                eq += (uint32_t)(__popcll(mk[0]) + __popcll(mk[1]) + __popcll(mk[2]) + __popcll(mk[3]));
            }
#pragma unroll
            for (uint32_t x = 0; x < 4; ++x) {
                const uint32_t bits = (x & 1u) ? e[i][x / 2].w : e[i][x / 2].y;
                f[x] = v[x] && ((bits & 0x7FFFFFFFu) > T || (f[x] && tied[x] < rT));
                mk[x] = ballot64(f[x]);
            }
            // The winners meet in LDS and leave 64 at a time: neighbours in the message by neighbouring lanes, and winners
            // of one line of the state in one store (1 % of 1e9 parameters: 524 / 439 us, and 584 / 508 straight from
            // the registers).
            const uint32_t won = (uint32_t)(__popcll(mk[0]) + __popcll(mk[1]) + __popcll(mk[2]) + __popcll(mk[3]));
            const bool fits = won <= STAGED;
#pragma unroll
            for (uint32_t x = 0; x < 4; ++x) {
                if (x >= 2 && !more) break;
                const uint2 c = (x & 1u) ? make_uint2(e[i][x / 2].z, e[i][x / 2].w) : make_uint2(e[i][x / 2].x, e[i][x / 2].y);
                if (!f[x]) continue;
                const uint32_t r = rank(x);
                if (fits) stage[r] = c;
                else write(pos + r, c, (OP == SEL_PULL_V && c.x < A.n) ? A.state[c.x] : 0.0f);
            }
            __builtin_amdgcn_wave_barrier();
            for (uint32_t r = lane; fits && r < won; r += 64) {
                const uint2 c = stage[r];
                write(pos + r, c, (OP == SEL_PULL_V && c.x < A.n) ? A.state[c.x] : 0.0f);
            }
            __builtin_amdgcn_wave_barrier();
            pos += won;
            continue;
        }
#pragma unroll 1
        for (uint32_t t = 4u * i; t < 4u * i + 4u; ++t) {         // one of the four has more than that: a tile at a time
            const uint32_t n = tile_n(w, t), start = (uint32_t)__builtin_amdgcn_readlane((int)w.start, (int)t);
            for (uint32_t q0 = 0; q0 < n; q0 += 64) {
                const bool valid = q0 + lane < n;
                const uint2 x = valid ? tile_get(A, w, t, start, q0 + lane) : make_uint2(0u, 0u);
                const float was = (OP == SEL_PULL_V && valid && x.x < A.n) ? A.state[x.x] : 0.0f;
                const uint32_t key = x.y & 0x7FFFFFFFu;
                const uint64_t mt = ballot64(valid && key == T);
                const bool f = valid && (key > T || (key == T && eq + mbcnt64(mt) < rT));
                eq += (uint32_t)__popcll(mt);
                const uint64_t mf = ballot64(f);
                if (f) write(pos + mbcnt64(mf), x, was);
                pos += (uint32_t)__popcll(mf);
            }
        }
    }
}

// SEG_ZERO, both roles: there is nothing to rank, and the emission completes the message with the
// tensor's z lowest-index zeros.  Candidate i of the tensor (in index order), at local index x, has x - i zeros below
// it.  While fewer than z, everything up to x is sent, and its position is x; from then on it is z + i.
// The candidates of a tile that begins with at least z zeros below it come from its list; a tile before
// that is read element by element, and those are dealt out to the wavefronts one at a time.  Bound by
// its loads and stores.  Pulls from an empty row / one with 0.9 k nonzeros, us: flat tensor of 1.2e6 at 1 %
// 30 / 40, of 2^23 at 1 % 62 / 50, of 1e9 at 0.1 % 967 / 1030.  All tiles joined and all pairs written by one
// workgroup: 30 / 54, 81 / 217, 3030 / 4500; joined by one per 4096 tiles, written by one: 20 / 42 (one launch
// less), 72 / 236, 1160 / 3150.
template <int OP, uint32_t THREADS>
__device__ __forceinline__ void zero_slab(const SelectArgs &A, bool emit, uint32_t slab, const SegDesc &sd,
                                          const TensorDesc &td, const PlanEntry &pe, SegState *st, uint32_t z, FinishShared &C)
{
    constexpr uint32_t WAVES = THREADS / 64, CTPW = slab_tpw(THREADS);
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = uniform(tid >> 6), end = td.off + td.n;
    if (!emit) {
        if (tid == 0) slab_publish<false>(&A.slabs_done[slab], 0u, 0u, 0u);
        if (arrive_last(&st->arrive[3], td.ncs, &C.bc) && tid == 0) st_dev(&st->key, make_uint2(0u, KEY_READY));
        return;
    }
    const uint32_t first = min(wave * CTPW, sd.ntiles), nt = min(CTPW, sd.ntiles - first);
    const WaveTiles w = wave_tiles(A, td, sd.tile0 + first, nt, false, sd.sidx);
    const uint32_t upto = wave_incl_scan(w.n);
    if (lane == 63) C.wtot[wave] = upto;
    const bool ready = wait_pair(&st->key, A.spin_limit, C.pair).y != 0;
    uint32_t i0 = 0, all = 0;
#pragma unroll
    for (uint32_t x = 0; x < WAVES; ++x) {
        i0 += (x < wave) ? C.wtot[x] : 0u;
        all += C.wtot[x];
    }
    if (wave == 0) {
        const bool head = (slab == td.cs_first);
        if (ready && lane == 0) slab_publish<false>(&A.slabs_done[slab], head ? SLAB_SUM : SLAB_OWN, all, 0u);
        uint32_t g = 0, q = 0;
        const bool known = ready && slab_look_back<false>(A, slab, td.cs_first, [&](uint32_t i) { return &A.slabs_done[i]; }, g, q);
        if (lane == 0) {
            if (!head || !known) slab_publish<false>(&A.slabs_done[slab], known ? SLAB_SUM : SLAB_FAIL, g + all, 0u);
            C.limit = known ? pe.k : 0u;
            C.g = g;
            if (!ready || (known && slab + 1 == td.cs_first + td.ncs && g + all + z != pe.k))
                atomicAdd(&A.stats->internal_errors, 1ull);
        }
    }
    __syncthreads();
    i0 += C.g;
    const uint32_t limit = C.limit;
    auto put = [&](uint32_t p, uint32_t ix, float v, float was) {
        if (p >= limit) return;
        A.out_idx[pe.outoff + p] = ix;
        A.out_val[pe.outoff + p] = v;
        if (!index_ok(A, ix)) return;
        if (OP == SEL_WORKER) store_scattered(&A.state[ix], A.m * v);
        else if (OP == SEL_PULL) store_scattered(&A.state[ix], 0.0f);
        else store_scattered(&A.state[ix], was + v);
    };
    auto behind_the_run = [&](uint32_t base, uint32_t before) { return max(base, td.off) - td.off - before >= z; };
    uint32_t *at = C.h;                              // candidates before every tile of the slab
    if (lane < nt) at[first + lane] = i0 + upto - w.n;
#pragma unroll 1
    for (uint32_t i = 0; i < nt; ++i) {
        const uint32_t n = tile_n(w, i);
        if (n != 0 && behind_the_run((w.t0 + i) * TILE, i0)) {
            const uint32_t start = (uint32_t)__builtin_amdgcn_readlane((int)w.start, (int)i);
            for (uint32_t q = lane; q < n; q += 64) {
                const uint2 e = tile_get(A, w, i, start, q);
                put(z + i0 + q, e.x, __uint_as_float(e.y), (OP == SEL_PULL_V && e.x < A.n) ? A.state[e.x] : 0.0f);
            }
        }
        i0 += n;
    }
    __syncthreads();
#pragma unroll 1
    for (uint32_t i = wave; i < sd.ntiles; i += WAVES) {
        const uint32_t base = (sd.tile0 + i) * TILE;
        uint32_t before0 = at[i];
        if (behind_the_run(base, before0)) break;
        // 64 consecutive elements at a time (their pairs leave as whole lines), all loads in flight together
        constexpr uint32_t ROWS = TILE / 64;
        float was[ROWS], model[ROWS];
#pragma unroll
        for (uint32_t u = 0; u < ROWS; ++u) {
            const uint32_t ix = min(max(base + u * 64 + lane, td.off), end - 1u);      // (one outside the tensor is not used)
            was[u] = A.state[ix];
            if (OP == SEL_PULL_V) model[u] = A.model[ix];
        }
#pragma unroll
        for (uint32_t u = 0; u < ROWS; ++u) {
            const uint32_t ix = base + u * 64 + lane, local = ix - td.off;
            const float v = (OP == SEL_PULL_V) ? model[u] - was[u] : was[u];
            const bool in = ix >= td.off && ix < end, nonzero = in && (__float_as_uint(v) & 0x7FFFFFFFu) != 0;
            const uint64_t m = ballot64(nonzero);
            const uint32_t before = before0 + mbcnt64(m);
            if (in && (nonzero || local - before < z)) put(nonzero ? min(local, z + before) : local, ix, v, was[u]);
            before0 += (uint32_t)__popcll(m);
        }
    }
}

// One workgroup of the chain's last part: RANK of slab `slab` or (emit) EMIT.  HERE: in the selection's own launch,
// behind the workgroups that decide what becomes of the tensor; the slab's candidates are fetched while that is
// awaited.
template <int OP, uint32_t THREADS, bool HERE>
__device__ __forceinline__ void finish_slab(const SelectArgs &A, bool emit, uint32_t slab, FinishShared &C)
{
    constexpr uint32_t CTPW = slab_tpw(THREADS);
    const SegDesc sd = A.cslabs[slab];               // (its sidx is the part it lies in)
    const PlanEntry pe = A.plan[sd.j];
    if (!HERE && !pe.seg) return;
    SegState *st = &A.segstate[sd.j];
    uint32_t status = HERE ? (uint32_t)SEG_ACTIVE : st->status;
    if (status != SEG_ACTIVE && status != SEG_LISTS && status != SEG_ZERO) return;
    const TensorDesc td = A.tdesc[sd.j];
    uint32_t pfx = HERE ? 0u : st->pfx, r2 = HERE ? 0u : st->r2;
    const uint32_t first = min(uniform(threadIdx.x >> 6) * CTPW, sd.ntiles), nt = min(CTPW, sd.ntiles - first);
    WaveTiles w = wave_tiles(A, td, sd.tile0 + first, nt, status == SEG_LISTS, sd.sidx);
    uint4 e[CTPW / 4][2];
    tile_firsts<CTPW>(A, w, e);                      // (on their way while what follows is awaited)
    if (HERE) {
        const uint2 v = wait_pair(&st->chain, A.spin_limit, C.pair);
        status = uniform(v.y >> CHAIN_STATUS_SHIFT);
        pfx = uniform(v.y & ((1u << CHAIN_STATUS_SHIFT) - 1u));
        r2 = uniform(v.x);
        if (status == SEG_IDLE) {                    // gave up waiting
            if (threadIdx.x == 0) {
                if (emit) slab_publish<false>(&A.slabs_done[slab], SLAB_FAIL, 0u, 0u);
                atomicAdd(&A.stats->internal_errors, 1ull);
            }
            return;
        }
        if (status == SEG_LISTS) {                   // collected again meanwhile
            w = wave_tiles(A, td, sd.tile0 + first, nt, true, sd.sidx);
            tile_firsts<CTPW>(A, w, e);
        }
    }
    if (__builtin_expect(status == SEG_ZERO, 0)) zero_slab<OP, THREADS>(A, emit, slab, sd, td, pe, st, r2, C);
    else if (status != SEG_ACTIVE && status != SEG_LISTS) {}      // (one workgroup has selected it after all)
    else if (emit) emit_slab<OP, THREADS>(A, slab, sd, td, pe, st, w, e, C);
    else rank_slab<THREADS>(A, slab, sd, td, st, pfx, r2, w, e, C);
    // The last of the tensor's workgroups clears what they have read for the next launch.  (Where the emission has awaited
    // the ranking, every slab's RANK is through before, and the EMIT counts for both.)
    const bool ranked = status == SEG_ACTIVE || status == SEG_LISTS || status == SEG_ZERO;
    if (threadIdx.x == 0 && (emit || !ranked)) {
        const uint32_t count = ranked ? 2u : 1u;
        const uint32_t old = __hip_atomic_fetch_add(&st->chain_seen, count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (old + count == 2u * td.ncs) {
            if (HERE) st_dev(&st->chain, make_uint2(0u, 0u));
            st_dev(&st->key, make_uint2(0u, 0u));
            st_dev(&st->chain_seen, 0u);
        }
    }
}

}  // namespace dgs
