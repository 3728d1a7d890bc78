#include "dgs_chain.h"

namespace dgs {

__global__ __launch_bounds__(SEL_THREADS) void k_list_window(const SelectArgs A)
{
    __shared__ uint32_t h[SEG_WBINS];
    __shared__ uint32_t wsum[SEL_WAVES];
    const uint32_t part = blockIdx.x;
    const SegDesc sd = A.segtab[part];
    if (!A.plan[sd.j].seg) return;
    const TensorDesc td = A.tdesc[sd.j];
    const uint32_t tid = threadIdx.x;
    bool over;
    const uint32_t c = window_tiles(A, td, sd.tile0, sd.ntiles, seg_window_base(A.tau[sd.j], A.tprev[sd.j]), h, wsum, over);
    uint32_t *out = part_hist(A, td, sd.j, sd.sidx);
    for (uint32_t b = tid; b < SEG_WBINS; b += SEL_THREADS) out[b] = h[b];
    if (tid == 0) A.segcnt[part] = c | (over ? 0x80000000u : 0u);
}

template <int OP, uint32_t THREADS>
__global__ __launch_bounds__(THREADS) void k_list_finish(const SelectArgs A)
{
    __shared__ FinishShared C;
    const bool emit = blockIdx.x >= A.ncslabs;
    finish_slab<OP, THREADS, false>(A, emit, emit ? blockIdx.x - A.ncslabs : blockIdx.x, C);
}

void launch_window(const SelectArgs &a, void *stream, void *ev0)
{
    if (a.nparts == 0) return;
    launch_k(k_list_window, dim3(a.nparts), dim3(SEL_THREADS), (hipStream_t)stream, ev0, nullptr, a);
}

template <uint32_t THREADS>
static void launch_finish(int op, const SelectArgs &a, hipStream_t st, void *ev0, void *ev1)
{
    const dim3 grid(2 * a.ncslabs), block(THREADS);
    if (op == SEL_WORKER) launch_k(k_list_finish<SEL_WORKER, THREADS>, grid, block, st, ev0, ev1, a);
    else if (op == SEL_PULL) launch_k(k_list_finish<SEL_PULL, THREADS>, grid, block, st, ev0, ev1, a);
    else launch_k(k_list_finish<SEL_PULL_V, THREADS>, grid, block, st, ev0, ev1, a);
}

void launch_chain(int op, const SelectArgs &a, void *stream, void *ev0, void *ev1)
{
    hipStream_t st = (hipStream_t)stream;
    if (a.ncslabs == 0) return;
    // While all slabs run at once (or nearly so) the depth of a workgroup counts: 8 tiles per wavefront.
    // Many rounds of workgroups are better served by twice as many workgroups per compute unit with 16
    // tiles per wavefront.  Rounds with 1024 / 512 threads, us: transformer shapes (about 900 slabs) 394 / 408; one flat
    // tensor at 0.3 / 1 % with 1530 slabs 954 / 942 and 1199 / 1208, 1980 1206 / 1212 and 1554 / 1579,
    // 3050 1796 / 1781 and 2365 / 2375; 25 equal tensors with 1530 830 / 775 and 1080 / 1047, 3050 1655 / 1535 and
    // 2209 / 2131; 1e9 parameters (7.8 K) at 1 % 5596 / 5338.
    if (a.ncslabs < 2048u) launch_finish<1024>(op, a, st, ev0, ev1);
    else launch_finish<512>(op, a, st, ev0, ev1);
}

// ---------------------------------------------------------------------------
// dense requests
// ---------------------------------------------------------------------------
//
// Above density 1/32 candidates stop paying off, and the tensors themselves are read again.  The
// accumulate pass has counted bits [30:19] of every key of the big tensors and k_pick_dense has
// found the bucket that holds the k-th one; then, one workgroup per slab of SLAB_TILES tiles of a
// tensor (a small tensor is one slab, and that workgroup counts its leading bits too),
//   refine 1  counts bits [18:11] of the keys in that bucket and writes those keys down, slab by slab;
//             the slab arriving last for a tensor ranks: 20 leading bits of the k-th key
//   refine 2  counts the low 11 bits of the keys that share them, among the keys written down (a slab
//             with too many of them reads its elements again); the slab arriving last ranks: the exact
//             key, and how many of the entries equal to it are taken
//   emit      counts its winners, adds up what the slabs before it have published (the chain's
//             look-back), ordered emission and state fix-up.  Ties need no case of their own.
// Each pass is bound by memory (4 B/param, mostly from the last-level cache up to a few 1e7
// parameters), by having enough of the chip at work, and refine 1 by the device-wide atomics that
// add the slabs' counters up: 256 bins keep those at 200 per slab of 32 tiles (2048 bins per slab
// of 16 tiles: 400 K on 25.6M parameters, 56 instead of 41 us).  ResNet-50 shapes at density 0.1:
// one workgroup per part (256 tiles and more, element by element) took 1070 + 72 + 361 us for a
// worker step; these three 41 + 37 + 80 us on a grid of (parts) x (slabs of the longest part), mostly
// empty workgroups on such a layout, 32 + 28 + 66 us with one workgroup per slab, and 33 + 13 + 57 us since
// refine 2 goes through the keys that refine 1 has written down (1.6 % of the elements; writing them costs
// refine 1 what holding two tiles a wavefront instead of four gains it) and the emission has 128 registers.
// Where the bucket is the one that it was in the last two calls, the accumulate pass has listed its keys (tile_keys) and the refinements
// read nothing else.  us a pull on Gaussian rows, elements read / keys listed: ResNet-50 shapes at 0.1 137 / 129, 24 tensors of 10M
// 860 / 718, one of 64M 290 / 254, one of 240M 864 / 717; a round of ResNet-50 shapes, where seven tensors in eight keep their bucket
// from one call to the next (and have three times as many keys in it), 450 / 439: the refinements 23 + 11 us instead of 33 + 13.

constexpr uint32_t SLAB_WAVES = SLAB_THREADS / 64;
constexpr uint32_t TPW = 4;                              // consecutive tiles of one wavefront
// The emission takes half slabs: its staging area is 8 KB of LDS per wavefront, and workgroups of four
// wavefronts leave more of them on a compute unit (80 against 97 us, figures as above).
constexpr uint32_t EMIT_TILES = SLAB_TILES / 2, EMIT_WAVES = EMIT_TILES / TPW, EMIT_THREADS = 64 * EMIT_WAVES;
constexpr uint32_t REF1_SHIFT = 11, REF1_BINS = 256;     // refine 1: key bits [18:11]
constexpr uint32_t REF2_BINS = 2048;                     // refine 2: key bits [10:0]
// Copies of refine 1's counters, and of the count of finished slabs where a tensor has many: adds of the whole device
// to one word follow each other at 11 ns.  us a pull on one tensor of 64M / 240M at 0.1, one copy / 8: elements read 314 / 290
// and 938 / 864; the refinements and the emission of 240M from listed keys 681 / 506, of 24 tensors of 10M 533 / 509.
constexpr uint32_t COPIES = 8;
static_assert(COPIES * REF1_BINS <= REF2_BINS, "the copies");

struct Slab {
    TensorDesc td;
    uint32_t j, tlo;          // its tensor, and that tensor's first tile
    uint32_t idx, count;      // which slab of the tensor it is, of how many (in units of TILES tiles)
    uint32_t tile0, ntiles;
};

// One block per slab and nothing else: a layout may hold one tensor of a thousand slabs and a
// hundred thousand of one.  false: the second half of a tensor's last slab is empty.
template <uint32_t TILES>
__device__ __forceinline__ bool find_slab(const SelectArgs &A, Slab &s)
{
    constexpr uint32_t PER = SLAB_TILES / TILES;
    s.j = A.dslabs[blockIdx.x / PER];
    s.td = A.tdesc[s.j];
    s.tlo = s.td.off / TILE;
    const uint32_t nt = (s.td.off + s.td.n - 1u) / TILE - s.tlo + 1u;
    s.idx = blockIdx.x - s.td.ds_first * PER;
    s.count = (nt + TILES - 1u) / TILES;
    if (s.idx >= s.count) return false;
    s.tile0 = s.tlo + s.idx * TILES;
    s.ntiles = min(TILES, nt - s.idx * TILES);
    return true;
}

// Where a slab of the emission publishes (two words): in the ordered-list scratch of its first tile.
__device__ __forceinline__ uint2 *dense_word(const SelectArgs &A, uint32_t tile0, uint32_t j)
{
    return A.ord + (size_t)(tile0 + j) * CAPT;
}

// The keys that refine 1 hands to refine 2: a stretch of its own for every wavefront that has tiles, in the
// scratch of the slab's first half (the second half begins with a word of the emission), behind one count
// each.  The bucket of 1/16 octave around the k-th key of a Gaussian tensor holds 2 % of its elements at
// density 0.1; there is room for half of a wavefront's elements in slabs of up to 16 tiles (2 CAPT words for
// the TILE elements of a tile), falling to a quarter in a full slab of 32.
constexpr uint32_t KEYS_AT = 16, ROUTE_AT = 4;
static_assert(KEYS_AT >= 4 + SLAB_WAVES, "two words of the emission and the counts");
struct SlabKeys {
    uint32_t *count;          // per wavefront
    uint32_t *mine;           // this wavefront's keys
    uint32_t waves, room;     // wavefronts that have tiles, keys of one of them
};
__device__ __forceinline__ SlabKeys slab_keys(const SelectArgs &A, const Slab &s)
{
    uint32_t *words = (uint32_t *)dense_word(A, s.tile0, s.j);
    SlabKeys k;
    k.count = words + KEYS_AT - SLAB_WAVES;
    k.waves = (s.ntiles + TPW - 1u) / TPW;
    k.room = (min(s.ntiles, EMIT_TILES) * (2u * CAPT) - KEYS_AT) / k.waves;
    k.mine = words + KEYS_AT + (threadIdx.x >> 6) * k.room;
    return k;
}

// NT of this wavefront's tiles of the slab, from its tile `first` on, 16 values per lane and tile; bit 4 r + x
// of in[i] says that value x of row r belongs to the tensor.  All loads are in flight together.
template <int OP, uint32_t NT>
__device__ __forceinline__ void load_slab(const SelectArgs &A, const Slab &s, uint32_t first, uint32_t (&bits)[NT][4][4],
                                          uint32_t (&in)[NT])
{
    const uint32_t lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const uint32_t lo = s.td.off, hi = s.td.off + s.td.n;
#pragma unroll
    for (uint32_t i = 0; i < NT; ++i) {
        const uint32_t ti = wave * TPW + first + i;
        in[i] = 0;
        if (ti >= s.ntiles) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int x = 0; x < 4; ++x) bits[i][r][x] = 0;
            continue;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            in[i] |= quad_bits<OP>(A, (s.tile0 + ti) * TILE + r * 256 + lane * 4, lo, hi, bits[i][r]) << (4 * r);
    }
}

// f(key, belongs) for every element of this wavefront's tiles, 64 at a time (all lanes call), in any order.
// Two tiles at a time: a kernel that holds all four needs 82 registers and leaves two workgroups on a
// compute unit, for 800 of them on ResNet-50 shapes one full round and a half.
template <int OP, class F>
__device__ __forceinline__ void each_key(const SelectArgs &A, const Slab &s, F f)
{
    constexpr uint32_t NT = 2;
#pragma unroll 1
    for (uint32_t first = 0; first < TPW; first += NT) {
        uint32_t bits[NT][4][4], in[NT];
        load_slab<OP, NT>(A, s, first, bits, in);
#pragma unroll
        for (uint32_t i = 0; i < NT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int x = 0; x < 4; ++x) f(bits[i][r][x] & 0x7FFFFFFFu, ((in[i] >> (4 * r + x)) & 1u) != 0);
    }
}

template <int OP, int LEVEL>
__global__ __launch_bounds__(SLAB_THREADS, 8) void k_dense_refine(const SelectArgs A)
{
    constexpr uint32_t BINS = (LEVEL == 1) ? REF1_BINS : REF2_BINS;
    constexpr uint32_t SHIFT = (LEVEL == 1) ? HSHIFT : REF1_SHIFT;       // the prefix known so far
    constexpr uint32_t LOW = (LEVEL == 1) ? REF1_SHIFT : 0u;
    __shared__ __align__(16) uint32_t h[LEVEL == 1 ? HBINS : BINS];
    __shared__ uint32_t rowsum[64];
    __shared__ int res[6];
    __shared__ uint32_t bc;
    const uint32_t tid = threadIdx.x;
    if (LEVEL == 2) {      // (before anything that has to be waited for)
        for (uint32_t b = 4u * tid; b < BINS; b += 4u * SLAB_THREADS) *(uint4 *)&h[b] = make_uint4(0, 0, 0, 0);
        __syncthreads();
    }
    Slab s;
    if (!find_slab<SLAB_TILES>(A, s)) return;
    const uint32_t j = s.j;
    SegState *st = &A.segstate[j];
    const bool leading = (LEVEL == 1) && !s.td.big;       // the leading bits are still to be counted
    const uint32_t k = A.plan[j].k;
    if (leading) {
        if (tid == 0) st->status = (k == s.td.n) ? SEG_ALL : SEG_ACTIVE;
        if (k == s.td.n) return;
    } else if (st->status != SEG_ACTIVE) {
        return;
    }
    uint32_t pfx = st->pfx, r2 = st->r2;
    uint32_t *g = A.ghist + (size_t)j * HBINS;
    const SlabKeys keys = slab_keys(A, s);
    const uint32_t wave = uniform(tid >> 6);
    // What the accumulate pass has listed, if that was the right bucket and no tile of the slab has had more than there is room
    // for.  (Refinement 1 uses the scratch for its own lists otherwise, and says which it was.)
    uint32_t *route = (uint32_t *)dense_word(A, s.tile0, j) + ROUTE_AT;
    bool listed = s.td.big && st->T == 1u;
    if (LEVEL == 1 && listed) {
        const uint32_t *cnt = (const uint32_t *)dense_word(A, s.tile0 + lane_id(), j) + TKEYS_COUNT;
        listed = ballot64(lane_id() < s.ntiles && *cnt > TKEYS_ROOM) == 0;
    }
    if (LEVEL == 2 && listed) listed = *route != 0;
    if (LEVEL == 1) {
        for (uint32_t b = tid; b < (leading ? HBINS : BINS); b += SLAB_THREADS) h[b] = 0;
        __syncthreads();
        if (tid == 0 && s.td.big) *route = listed ? 1u : 0u;
    }
    bool from_keys = (LEVEL == 2) && !listed;
    if (from_keys)
        for (uint32_t w = 0; w < keys.waves; ++w) from_keys &= keys.count[w] <= keys.room;
    if (listed) {
        // 16 lanes a tile, the wavefront's TPW at once
        const uint32_t ti = wave * TPW + (lane_id() >> 4);
        const uint32_t *words = (const uint32_t *)dense_word(A, s.tile0 + min(ti, s.ntiles - 1u), j);
        const uint32_t c = (ti < s.ntiles) ? words[TKEYS_COUNT] : 0u;
        for (uint32_t q = lane_id() & 15u; q < c; q += 16) {
            const uint32_t key = words[TKEYS_AT + q];
            if (LEVEL == 1 || (key >> SHIFT) == pfx) atomicAdd(&h[(key >> LOW) & (BINS - 1u)], 1u);
        }
    } else if (from_keys) {
        // A smooth tensor has a few keys per slab that share the prefix (one in 256 of those written down), but
        // all of them do where keys are tied: quantised ones, or ones that had 16 bits.  So they are counted in LDS
        // and a slab adds at most once to a word: adds of the whole device to one word follow each other at 11 ns
        // (64M parameters with 1 % ties, all three passes: 7485 us with an add per key, 262 so).
        const uint32_t listed = (wave < keys.waves) ? keys.count[wave] : 0u;
        for (uint32_t q = lane_id(); q < listed; q += 64) {
            const uint32_t key = keys.mine[q];
            if ((key >> SHIFT) == pfx) atomicAdd(&h[key & (BINS - 1u)], 1u);
        }
    } else {
        if (leading) {
            each_key<OP>(A, s, [&](uint32_t key, bool in) {
                if (in) atomicAdd(&h[key >> HSHIFT], 1u);
            });
            find_ranks<(int)HBINS, (int)SLAB_WAVES>(h, k, 0u, 0u, rowsum, res);
            pfx = (uint32_t)res[0];
            r2 = (uint32_t)res[1];
            __syncthreads();
            for (uint32_t b = tid; b < BINS; b += SLAB_THREADS) h[b] = 0;
            __syncthreads();
        }
        uint32_t run = 0;
        each_key<OP>(A, s, [&](uint32_t key, bool in) {
            const bool hit = in && (key >> SHIFT) == pfx;
            const uint64_t m = ballot64(hit);
            if (m == 0) return;
            if (hit) {
                atomicAdd(&h[(key >> LOW) & (BINS - 1u)], 1u);
                const uint32_t at = run + mbcnt64(m);
                if (LEVEL == 1 && at < keys.room) keys.mine[at] = key;
            }
            run += (uint32_t)__popcll(m);
        });
        if (LEVEL == 1 && wave < keys.waves && lane_id() == 0) keys.count[wave] = run;
    }
    // (the emission's slabs have published nothing yet)
    if (LEVEL == 2 && tid < SLAB_TILES / EMIT_TILES && tid * EMIT_TILES < s.ntiles)
        slab_publish<true>(dense_word(A, s.tile0 + tid * EMIT_TILES, j), 0u, 0u, 0u);
    __syncthreads();
    // (16 bytes a thread: with 2048 counters read and cleared one by one this pass takes 15 us instead of 13)
    static_assert(LEVEL == 2 || BINS <= SLAB_THREADS, "a counter each");
    if (LEVEL == 1 && tid < BINS && h[tid]) atomicAdd(&g[(s.idx % COPIES) * BINS + tid], h[tid]);
    for (uint32_t b = 4u * tid; LEVEL == 2 && b < BINS; b += 4u * SLAB_THREADS) {
        const uint4 v = *(const uint4 *)&h[b];
        if (v.x) atomicAdd(&g[b], v.x);
        if (v.y) atomicAdd(&g[b + 1], v.y);
        if (v.z) atomicAdd(&g[b + 2], v.z);
        if (v.w) atomicAdd(&g[b + 3], v.w);
    }
    // Counted in far from the words that every slab begins with (the status and the prefix): a line that is
    // added to all the time has to be fetched anew by every reader.  On one flat tensor of 64M / 250M / 1e9
    // parameters refine 1 (elements read, one copy of everything) takes 67 / 212 / 786 us; with the count beside the status
    // 107 / 484 / 2007, and 87 / 298 / 1122 with half as many slabs on a compute unit and no keys written down.
    static_assert(REF2_BINS + (COPIES + 1u) * 32u <= HBINS, "words that neither refinement counts in, on lines of their own");
    if (s.count > COPIES * 64u &&
        !arrive_last(&g[HBINS - 1u - (1u + s.idx % COPIES) * 32u], (s.count - s.idx % COPIES + COPIES - 1u) / COPIES, &bc)) return;
    if (!arrive_last(&g[HBINS - 1u], s.count > COPIES * 64u ? COPIES : s.count, &bc)) return;

    // ------------------------------------------------------------------ the tensor's last slab
    for (uint32_t b = tid; b < BINS; b += SLAB_THREADS) {
        constexpr uint32_t N = (LEVEL == 1) ? COPIES : 1u;
        uint32_t v[N], sum = 0;
#pragma unroll
        for (uint32_t x = 0; x < N; ++x) v[x] = ld_dev(&g[x * BINS + b]);
#pragma unroll
        for (uint32_t x = 0; x < N; ++x) {
            sum += v[x];
            if (v[x]) st_dev(&g[x * BINS + b], 0u);   // clean for the next use
        }
        h[b] = sum;
    }
    find_ranks<(int)BINS, (int)SLAB_WAVES>(h, r2, 0u, 0u, rowsum, res);
    const int bin = res[0];
    const uint32_t rank = (uint32_t)res[1];
    if (bin < 0) {                  // the pass before has counted other elements: cannot happen
        if (tid == 0) {
            st->status = SEG_FALLBACK;
            atomicAdd(&A.stats->internal_errors, 1ull);
        }
        return;
    }
    if (tid == 0) {
        const uint32_t key = (pfx << (SHIFT - LOW)) | (uint32_t)bin;
        if (LEVEL == 1) {
            st->pfx = key;
            st->r2 = rank;
        } else {
            st->T = key;
            st->rT = rank;
        }
    }
}

// Winners are staged per tile in LDS and leave as coalesced runs; the state is written by whole
// 64-byte lines wherever a line has a winner (at these densities most lines that have one would
// otherwise be read, merged and written back by the memory side for every 4-byte store).
// 128 registers let four workgroups share a compute unit (148 by themselves: three, 66 instead of 57 us
// on ResNet-50 shapes at density 0.1); the printed state's emission would spill 176 of them and keeps its own.
template <int OP>
__global__ __launch_bounds__(EMIT_THREADS, OP == SEL_PULL_V ? 3 : 4) void k_dense_emit(const SelectArgs A)
{
    __shared__ uint2 stage_all[EMIT_WAVES][TILE];
    __shared__ uint32_t wtot[EMIT_WAVES];
    __shared__ uint32_t g_before, q_before, known_before;
    Slab s;
    if (!find_slab<EMIT_TILES>(A, s)) return;
    const SegState *st = &A.segstate[s.j];
    const uint32_t status = st->status;
    if (status != SEG_ACTIVE && status != SEG_ALL) return;
    const PlanEntry pe = A.plan[s.j];
    const uint32_t lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const bool all = (status == SEG_ALL);
    // (density 1: everything is sent, at its own position)
    const uint32_t T = all ? 0u : st->T, rT = all ? 0u : st->rT;
    uint32_t bits[TPW][4][4], in[TPW];
    load_slab<OP, TPW>(A, s, 0u, bits, in);
    uint32_t mine = 0;
#pragma unroll
    for (uint32_t i = 0; i < TPW; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const bool ok = (in[i] >> (4 * r + x)) & 1u;
                const uint32_t key = bits[i][r][x] & 0x7FFFFFFFu;
                if (ok && (all || key > T)) ++mine;
                else if (ok && key == T) mine += 1u << 16;
            }
    const uint32_t sum = wave_sum(mine);         // at most 4096 of either kind, EMIT_TILES / 4 times that in all
    if (lane == 0) wtot[wave] = sum;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (uint32_t w = 0; w < EMIT_WAVES; ++w) {
        before += (w < wave) ? wtot[w] : 0u;
        total += wtot[w];
    }
    if (wave == 0) {
        uint32_t g = max(s.tile0 * TILE, s.td.off) - s.td.off, q = 0;
        bool known = true;
        if (!all) {
            uint2 *word = dense_word(A, s.tile0, s.j);
            if (lane == 0) slab_publish<true>(word, s.idx == 0 ? SLAB_SUM : SLAB_OWN, total & 0xFFFFu, total >> 16);
            known = slab_look_back<true>(A, s.idx, 0u, [&](uint32_t i) { return dense_word(A, s.tlo + i * EMIT_TILES, s.j); },
                                         g, q);
            if (lane == 0) {
                if (s.idx != 0) slab_publish<true>(word, known ? SLAB_SUM : SLAB_FAIL, g + (total & 0xFFFFu), q + (total >> 16));
                if (known && s.idx + 1 == s.count &&
                    (g + (total & 0xFFFFu) + rT != pe.k || q + (total >> 16) < rT))
                    atomicAdd(&A.stats->internal_errors, 1ull);
            }
        }
        if (lane == 0) {
            g_before = g;
            q_before = q;
            known_before = known ? 1u : 0u;
        }
    }
    __syncthreads();
    if (known_before == 0) return;
    uint32_t eq = q_before + (before >> 16);     // the tensor's ties before this row: lowest index first, rT of them are taken
    uint32_t pos = g_before + (before & 0xFFFFu) + min(eq, rT);
    uint2 *stage = stage_all[wave];
#pragma unroll
    for (uint32_t i = 0; i < TPW; ++i) {
        const uint32_t ti = wave * TPW + i;
        if (ti >= s.ntiles) break;               // wave-uniform
        const uint32_t base = (s.tile0 + ti) * TILE;
        uint32_t run = 0;                        // winners of this tile so far
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t e0 = base + r * 256 + lane * 4;
            bool f[4], q[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const bool ok = (in[i] >> (4 * r + x)) & 1u;
                const uint32_t key = bits[i][r][x] & 0x7FFFFFFFu;
                f[x] = ok && (all || key > T);
                q[x] = !all && ok && key == T;
            }
            const uint64_t anyq = ballot64(q[0] | q[1] | q[2] | q[3]);
            if (anyq != 0) {
                uint32_t er = eq;
                uint32_t cnt = 0;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const uint64_t m = ballot64(q[x]);
                    er += mbcnt64(m);
                    cnt += (uint32_t)__popcll(m);
                }
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    if (q[x]) {
                        f[x] = er < rT;
                        ++er;
                    }
                eq += cnt;
            }
            uint64_t mk[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) mk[x] = ballot64(f[x]);
            const uint64_t any = mk[0] | mk[1] | mk[2] | mk[3];
            if (any == 0) continue;
            uint32_t p = run + mbcnt64(mk[0]) + mbcnt64(mk[1]) + mbcnt64(mk[2]) + mbcnt64(mk[3]);
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if (f[x]) stage[p++] = make_uint2(e0 + x, bits[i][r][x]);
            run += (uint32_t)(__popcll(mk[0]) + __popcll(mk[1]) + __popcll(mk[2]) + __popcll(mk[3]));
            const bool quad = ((in[i] >> (4 * r)) & 0xFu) == 0xFu;
            if (quad) {
                if (((any >> (lane & ~3u)) & 0xFull) != 0) {
                    f32x4 o;
                    if (OP == SEL_PULL_V) o = *(const f32x4_any *)(A.state + e0);
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const float v = __uint_as_float(bits[i][r][x]);
                        if (OP == SEL_PULL_V) {
                            if (f[x]) o[x] = o[x] + v;
                        } else {
                            o[x] = !f[x] ? v : (OP == SEL_WORKER ? A.m * v : 0.0f);
                        }
                    }
                    __builtin_nontemporal_store((f32x4_any)o, (f32x4_any *)(A.state + e0));
                }
            } else {
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    if (f[x]) fix_sent<OP>(A.state, e0 + x, __uint_as_float(bits[i][r][x]), A.m);
            }
        }
        __builtin_amdgcn_wave_barrier();
        for (uint32_t w = lane; w < run; w += 64) {
            const uint2 e = stage[w];
            if (pos + w < pe.k) {
                A.out_idx[pe.outoff + pos + w] = e.x;
                A.out_val[pe.outoff + pos + w] = __uint_as_float(e.y);
            }
        }
        __builtin_amdgcn_wave_barrier();
        pos += run;
    }
}

void launch_dense(int op, const SelectArgs &a, void *stream, void *ev0, void *ev1)
{
    hipStream_t st = (hipStream_t)stream;
    const dim3 grid(a.ndslabs), block(SLAB_THREADS);
    const dim3 egrid(a.ndslabs * (SLAB_TILES / EMIT_TILES)), eblock(EMIT_THREADS);
    if (op == SEL_PULL_V) {
        launch_k(k_dense_refine<SEL_PULL_V, 1>, grid, block, st, ev0, nullptr, a);
        launch_k(k_dense_refine<SEL_PULL_V, 2>, grid, block, st, nullptr, nullptr, a);
        launch_k(k_dense_emit<SEL_PULL_V>, egrid, eblock, st, nullptr, ev1, a);
    } else {      // worker and difference row rank the same buffer
        launch_k(k_dense_refine<SEL_PULL, 1>, grid, block, st, ev0, nullptr, a);
        launch_k(k_dense_refine<SEL_PULL, 2>, grid, block, st, nullptr, nullptr, a);
        if (op == SEL_WORKER) launch_k(k_dense_emit<SEL_WORKER>, egrid, eblock, st, nullptr, ev1, a);
        else launch_k(k_dense_emit<SEL_PULL>, egrid, eblock, st, nullptr, ev1, a);
    }
}

}  // namespace dgs
