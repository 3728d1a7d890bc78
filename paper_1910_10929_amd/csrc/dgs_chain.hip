// The chain: what follows the selection kernel for tensors whose candidate lists are too long
// for one workgroup.  The selection kernel has left, per tensor, the 19-bit prefix of the k-th key and
// its rank among the entries sharing that prefix; here
//   prefix  per part   : counts the entries above the prefix, appends those sharing it to the
//                        tensor's prefix list and counts their low 12 bits; the part that
//                        arrives last for a tensor RANKS: exact k-th key, tie budget, and every
//                        part's output position
//   emit    per part   : ordered emission ("encode()" of Algorithms 1-3) and the state fix-up
//                        (Eq. 12 / Eq. 6).
// Dense requests have no candidate lists; their passes over the tensors themselves are at the end
// of this file.
#include "dgs_select.h"

namespace dgs {

// The entries one part contributes: its stretch of the tensor's candidate lists, in index order.
struct PartSource {
    const uint2 *list;
    uint32_t count;
};

__device__ __forceinline__ PartSource part_source(const SelectArgs &A, uint32_t part)
{
    return PartSource{A.ord + A.segstart[part], A.segcnt[part] & 0x7FFFFFFFu};
}

constexpr uint32_t PFX_STAGE = 1024;   // entries sharing the prefix that one part can stage in LDS

struct ChainShared {
    uint32_t h[SEG_LBINS];
    uint32_t sG[SEG_MAX_PER_TENSOR];
    uint32_t sQ[SEG_MAX_PER_TENSOR];
    uint32_t rowsum[64];
    int res[6];
    uint32_t wsum[SEL_WAVES];
    uint2 stage[PFX_STAGE];
    uint32_t nstage, base, bc;
};

__global__ __launch_bounds__(SEL_THREADS) void k_chain_prefix(const SelectArgs A)
{
    __shared__ ChainShared C;
    const uint32_t part = blockIdx.x;
    const SegDesc sd = A.segtab[part];
    const uint32_t j = sd.j;
    const PlanEntry pe = A.plan[j];
    if (!pe.seg) return;
    SegState *st = &A.segstate[j];
    if (st->status != SEG_ACTIVE) return;
    const TensorDesc td = A.tdesc[j];
    const PartSource src = part_source(A, part);
    const uint32_t cs = src.count;
    const uint32_t tid = threadIdx.x;
    const uint32_t pfx = st->pfx;
    uint4 *plist = A.pfxlist + (size_t)td.pfx_slot * PFX_CAP;
    uint32_t *glow = A.ghist + (size_t)j * HBINS;   // low key bits of the entries sharing the prefix
    if (tid == 0) C.nstage = 0;
    __syncthreads();
    uint32_t g1 = 0;
    for (uint32_t eb = 0; eb < cs; eb += 4 * SEL_THREADS) {
        uint2 ent[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t e = eb + u * SEL_THREADS + tid;
            ent[u] = (e < cs) ? src.list[e] : make_uint2(0, 0);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t e = eb + u * SEL_THREADS + tid;
            if (e < cs) {
                const uint32_t hi12 = (ent[u].y & 0x7FFFFFFFu) >> SEG_LOWBITS;
                if (hi12 > pfx) {
                    ++g1;
                } else if (hi12 == pfx) {
                    atomicAdd(&glow[ent[u].y & (SEG_LBINS - 1u)], 1u);
                    const uint32_t p = atomicAdd(&C.nstage, 1u);
                    if (p < PFX_STAGE) C.stage[p] = ent[u];
                }
            }
        }
    }
    const uint32_t G1 = block_sum(g1, C.wsum, SEL_WAVES);   // its barriers also complete `stage`
    const uint32_t ns = C.nstage;
    if (tid == 0) {
        st_dev(&A.segG1[part], G1);
        // one reservation per part in the tensor's prefix list; a part that could not stage all
        // of its entries pushes the count past the capacity, and the ranking counts instead
        if (ns) C.base = __hip_atomic_fetch_add(&st->pfxcount, ns > PFX_STAGE ? PFX_CAP + 1u : ns,
                                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (ns && ns <= PFX_STAGE) {
        const uint32_t b0 = C.base;
        for (uint32_t i = tid; i < ns; i += SEL_THREADS)
            if (b0 + i < PFX_CAP) {
                // (index, value bits) and (part, 0) as two 8-byte device-scope stores
                uint2 *dst = (uint2 *)&plist[b0 + i];
                st_dev(&dst[0], C.stage[i]);
                st_dev(&dst[1], make_uint2(sd.sidx, 0u));
            }
    }
    if (!arrive_last(&st->arrive[3], td.nseg, &C.bc)) return;

    // ------------------------------------------------------------------ RANK (last part)
    const uint32_t m = ld_dev(&st->pfxcount);
    const uint32_t r2 = st->r2;
    for (uint32_t s = tid; s < td.nseg; s += SEL_THREADS) { C.sG[s] = 0; C.sQ[s] = 0; }
    for (uint32_t b = tid; b < SEG_LBINS; b += SEL_THREADS) {
        const uint32_t v = ld_dev(&glow[b]);
        C.h[b] = v;
        if (v) st_dev(&glow[b], 0u);   // clean for the next use
    }
    find_ranks<SEG_LBINS, SEL_WAVES>(C.h, r2, 0u, 0u, C.rowsum, C.res);
    const int b3 = C.res[0];
    if (b3 < 0) {   // the rank exceeds what the parts counted: cannot happen
        if (tid == 0) {
            st->status = SEG_FALLBACK;
            atomicAdd(&A.stats->internal_errors, 1ull);
        }
        return;
    }
    const uint32_t T = (pfx << SEG_LOWBITS) | (uint32_t)b3;
    const uint32_t rT = (uint32_t)C.res[1];   // entries equal to T that are taken, lowest index first
    __syncthreads();
    if (m <= PFX_CAP) {
        for (uint32_t p = tid; p < m; p += SEL_THREADS) {
            const uint2 *srcp = (const uint2 *)&plist[p];
            const uint2 e = ld_dev(&srcp[0]);
            const uint32_t seg = ld_dev(&srcp[1]).x;
            const uint32_t low = e.y & (SEG_LBINS - 1u);
            if (seg >= td.nseg) continue;      // (a corrupted list entry)
            if (low > (uint32_t)b3) atomicAdd(&C.sG[seg], 1u);
            else if (low == (uint32_t)b3) atomicAdd(&C.sQ[seg], 1u);
        }
        __syncthreads();
    } else {
        // too many entries share the prefix for the list (massive ties): count every part
        // against T here -- slow, reached by degenerate data only
        for (uint32_t s = 0; s < td.nseg; ++s) {
            const PartSource q = part_source(A, td.seg_first + s);
            uint32_t g = 0, qq = 0;
            for (uint32_t e = tid; e < q.count; e += SEL_THREADS) {
                const uint2 ent = ld_dev(&q.list[e]);
                const uint32_t key = ent.y & 0x7FFFFFFFu;
                if ((key >> SEG_LOWBITS) == pfx) {
                    g += (key > T) ? 1u : 0u;
                    qq += (key == T) ? 1u : 0u;
                }
            }
            const uint32_t Gs = block_sum(g, C.wsum, SEL_WAVES);
            const uint32_t Qs = block_sum(qq, C.wsum, SEL_WAVES);
            if (tid == 0) { C.sG[s] = Gs; C.sQ[s] = Qs; }
        }
        __syncthreads();
    }
    // parts in order: ties are taken lowest index first, i.e. earlier parts first
    uint32_t carry_q = 0, carry_o = 0;
    for (uint32_t sb = 0; sb < td.nseg; sb += SEL_THREADS) {
        const uint32_t s = sb + tid;
        const bool in = s < td.nseg;
        const uint32_t G = in ? (ld_dev(&A.segG1[td.seg_first + s]) + C.sG[s]) : 0u;
        const uint32_t Q = in ? C.sQ[s] : 0u;
        uint32_t totq, toto;
        const uint32_t qb = carry_q + block_excl_scan<SEL_WAVES>(Q, C.wsum, totq);
        const uint32_t take = min(Q, (rT > qb) ? (rT - qb) : 0u);
        const uint32_t ob = carry_o + block_excl_scan<SEL_WAVES>(G + take, C.wsum, toto);
        if (in) A.segOut[td.seg_first + s] = make_uint2(ob, take);
        carry_q += totq;
        carry_o += toto;
    }
    if (tid == 0) {
        st->T = T;
        st->pfxcount = 0;
        A.tprev[j] = T;
        if (carry_o != pe.k) atomicAdd(&A.stats->internal_errors, 1ull);
    }
}

template <int OP>
__global__ __launch_bounds__(SEG_THREADS) void k_chain_emit(const SelectArgs A)
{
    __shared__ uint32_t wsum[SEG_THREADS / 64];
    const uint32_t part = blockIdx.x;
    const SegDesc sd = A.segtab[part];
    const PlanEntry pe = A.plan[sd.j];
    if (!pe.seg) return;
    const SegState *st = &A.segstate[sd.j];
    const uint32_t tid = threadIdx.x;
    if (st->status != SEG_ACTIVE) return;
    const uint32_t T = st->T;
    const uint2 so = A.segOut[part];
    const PartSource src = part_source(A, part);
    const uint32_t cs = src.count;
    constexpr uint32_t ITEMS = 4;
    uint32_t run_sel = so.x, run_eq = 0;
    const uint32_t rT = so.y;
    for (uint32_t cb = 0; cb < cs; cb += SEG_THREADS * ITEMS) {
        const uint32_t p0 = cb + tid * ITEMS;
        uint2 v[ITEMS];
        uint32_t g = 0, q = 0;
#pragma unroll
        for (uint32_t i = 0; i < ITEMS; ++i) v[i] = (p0 + i < cs) ? src.list[p0 + i] : make_uint2(0, 0);
#pragma unroll
        for (uint32_t i = 0; i < ITEMS; ++i) {
            const uint32_t key = v[i].y & 0x7FFFFFFFu;
            if (p0 + i < cs) {
                g += (key > T);
                q += (key == T);
            }
        }
        uint32_t total;
        const uint32_t before = block_excl_scan<SEG_THREADS / 64>(g | (q << 16), wsum, total);
        const uint32_t g_before = before & 0xFFFFu, q_before = before >> 16;
        const uint32_t G = total & 0xFFFFu, Q = total >> 16;
        const uint32_t rem = (rT > run_eq) ? (rT - run_eq) : 0u;
        uint32_t pos = run_sel + g_before + min(q_before, rem);
        uint32_t eq_seen = q_before;
        if (g | q) {
#pragma unroll
            for (uint32_t i = 0; i < ITEMS; ++i) {
                if (p0 + i >= cs) break;
                const uint32_t key = v[i].y & 0x7FFFFFFFu;
                bool sel = key > T;
                if (key == T) {
                    sel = eq_seen < rem;
                    ++eq_seen;
                }
                if (sel) {
                    if (pos < pe.k) {
                        A.out_idx[pe.outoff + pos] = v[i].x;
                        A.out_val[pe.outoff + pos] = __uint_as_float(v[i].y);
                        if (index_ok(A, v[i].x)) fix_sent<OP>(A.state, v[i].x, __uint_as_float(v[i].y), A.m);
                    }
                    ++pos;
                }
            }
        }
        run_sel += G + min(Q, rem);
        run_eq += Q;
    }
}

void launch_chain(int op, const SelectArgs &a, void *stream, void *ev0, void *ev1)
{
    hipStream_t st = (hipStream_t)stream;
    if (a.nparts == 0) return;
    launch_k(k_chain_prefix, dim3(a.nparts), dim3(SEL_THREADS), st, ev0, nullptr, a);
    if (op == SEL_WORKER)
        launch_k(k_chain_emit<SEL_WORKER>, dim3(a.nparts), dim3(SEG_THREADS), st, nullptr, ev1, a);
    else if (op == SEL_PULL)
        launch_k(k_chain_emit<SEL_PULL>, dim3(a.nparts), dim3(SEG_THREADS), st, nullptr, ev1, a);
    else
        launch_k(k_chain_emit<SEL_PULL_V>, dim3(a.nparts), dim3(SEG_THREADS), st, nullptr, ev1, a);
}

// ---------------------------------------------------------------------------
// dense requests
// ---------------------------------------------------------------------------
//
// Above density 1/32 candidates stop paying off, and the tensors themselves are read again.  The
// accumulate pass has counted bits [30:19] of every key of the big tensors and k_pick_dense has
// found the bucket that holds the k-th one; then, one workgroup per slab of SLAB_TILES tiles of a
// part (a small tensor is one slab, and that workgroup counts its leading bits too),
//   refine 1  counts bits [18:8] of the keys in that bucket; the slab arriving last for a tensor
//             ranks: 23 leading bits of the k-th key
//   refine 2  counts, per slab, the entries above that prefix and the low 8 bits of those that
//             share it; the slab arriving last ranks: the exact key, and from every slab's own
//             counts how many entries it sends and where they go (no list that ties could outgrow)
//   emit      ordered emission and state fix-up.
// Each pass is bound by memory (4 B/param, mostly from the last-level cache up to a few 1e7
// parameters) and by having enough of the chip at work: slabs of 16 tiles put 1.6 K workgroups on
// 25.6M parameters.  ResNet-50 shapes at density 0.1: one workgroup per part (256 tiles and more,
// element by element) took 1070 + 72 + 361 us for a worker step.

constexpr uint32_t SLAB_WAVES = SLAB_THREADS / 64;
constexpr uint32_t TPW = SLAB_TILES / SLAB_WAVES;        // consecutive tiles of one wavefront
constexpr uint32_t REF1_SHIFT = 8, REF1_BINS = 2048;     // refine 1: key bits [18:8]
constexpr uint32_t REF2_BINS = 256;                      // refine 2: key bits [7:0]

struct Slab {
    TensorDesc td;
    SegDesc part;
    uint32_t tile0, ntiles;
};

__device__ __forceinline__ bool find_slab(const SelectArgs &A, Slab &s)
{
    s.part = A.segtab[blockIdx.x / A.slabs];
    const uint32_t first = (blockIdx.x % A.slabs) * SLAB_TILES;
    if (first >= s.part.ntiles || !A.plan[s.part.j].seg) return false;
    s.td = A.tdesc[s.part.j];
    s.tile0 = s.part.tile0 + first;
    s.ntiles = min(SLAB_TILES, s.part.ntiles - first);
    return true;
}

// Slabs of one full part, and of the whole tensor (only its last part may be shorter).
__device__ __forceinline__ uint32_t slabs_per_part(const SelectArgs &A, const TensorDesc &td)
{
    return (A.segtab[td.seg_first].ntiles + SLAB_TILES - 1u) / SLAB_TILES;
}

__device__ __forceinline__ uint32_t slabs_of_tensor(const SelectArgs &A, const TensorDesc &td)
{
    return (td.nseg - 1u) * slabs_per_part(A, td) +
           (A.segtab[td.seg_first + td.nseg - 1u].ntiles + SLAB_TILES - 1u) / SLAB_TILES;
}

// A slab's record, in the ordered-list scratch of its first tile: [0] first output position,
// [1] ties it sends, [2 + b] entries of the slab at or above (23-bit prefix, low bits b).
__device__ __forceinline__ uint32_t *slab_record(const SelectArgs &A, uint32_t tile0, uint32_t j)
{
    return (uint32_t *)(A.ord + (size_t)(tile0 + j) * CAPT);
}
static_assert(REF2_BINS == SLAB_THREADS && 2 + REF2_BINS + 1 <= 2 * CAPT, "a slab record fits one tile's scratch");

// This wavefront's tiles of the slab, 16 values per lane and tile; bit 4 r + x of in[i] says that
// value x of row r belongs to the tensor.  All loads are in flight together.
template <int OP>
__device__ __forceinline__ void load_slab(const SelectArgs &A, const Slab &s, uint32_t (&bits)[TPW][4][4],
                                          uint32_t (&in)[TPW])
{
    const uint32_t lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const uint32_t lo = s.td.off, hi = s.td.off + s.td.n;
#pragma unroll
    for (uint32_t i = 0; i < TPW; ++i) {
        const uint32_t ti = wave * TPW + i;
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

template <int OP, int LEVEL>
__global__ __launch_bounds__(SLAB_THREADS) void k_dense_refine(const SelectArgs A)
{
    constexpr uint32_t BINS = (LEVEL == 1) ? REF1_BINS : REF2_BINS;
    constexpr uint32_t SHIFT = (LEVEL == 1) ? HSHIFT : REF1_SHIFT;       // the prefix known so far
    constexpr uint32_t LOW = (LEVEL == 1) ? REF1_SHIFT : 0u;
    __shared__ uint32_t h[LEVEL == 1 ? HBINS : BINS];
    __shared__ uint32_t wsum[SLAB_WAVES];
    __shared__ uint32_t rowsum[64];
    __shared__ int res[6];
    __shared__ uint32_t bc;
    Slab s;
    if (!find_slab(A, s)) return;
    const uint32_t j = s.part.j, tid = threadIdx.x;
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
    uint32_t bits[TPW][4][4], in[TPW];
    load_slab<OP>(A, s, bits, in);
    if (leading) {
        for (uint32_t b = tid; b < HBINS; b += SLAB_THREADS) h[b] = 0;
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < TPW; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    if ((in[i] >> (4 * r + x)) & 1u) atomicAdd(&h[(bits[i][r][x] & 0x7FFFFFFFu) >> HSHIFT], 1u);
        find_ranks<(int)HBINS, (int)SLAB_WAVES>(h, k, 0u, 0u, rowsum, res);
        pfx = (uint32_t)res[0];
        r2 = (uint32_t)res[1];
        __syncthreads();
    }
    for (uint32_t b = tid; b < BINS; b += SLAB_THREADS) h[b] = 0;
    __syncthreads();
    uint32_t above = 0;
#pragma unroll
    for (uint32_t i = 0; i < TPW; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            bool hit[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const bool ok = (in[i] >> (4 * r + x)) & 1u;
                const uint32_t top = (bits[i][r][x] & 0x7FFFFFFFu) >> SHIFT;
                hit[x] = ok && top == pfx;
                if (LEVEL == 2) above += (ok && top > pfx) ? 1u : 0u;
            }
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if (hit[x]) atomicAdd(&h[(bits[i][r][x] >> LOW) & (BINS - 1u)], 1u);
        }
    uint32_t *g = A.ghist + (size_t)j * HBINS;
    if (LEVEL == 2) {
        const uint32_t G = block_sum(above, wsum, SLAB_WAVES);       // (its barriers also complete h)
        uint32_t *rec = slab_record(A, s.tile0, j);
        const uint32_t mine = h[tid];                                // one bin per thread
        uint32_t tot;
        const uint32_t below = block_excl_scan<(int)SLAB_WAVES>(mine, wsum, tot);
        st_dev(&rec[2 + tid], G + tot - below);
        if (tid == 0) st_dev(&rec[2 + REF2_BINS], G);
    } else {
        __syncthreads();
    }
    for (uint32_t b = tid; b < BINS; b += SLAB_THREADS) {
        const uint32_t v = h[b];
        if (v) atomicAdd(&g[b], v);
    }
    const uint32_t nslabs = slabs_of_tensor(A, s.td);
    if (!arrive_last(&st->arrive[LEVEL], nslabs, &bc)) return;

    // ------------------------------------------------------------------ the tensor's last slab
    for (uint32_t b = tid; b < BINS; b += SLAB_THREADS) {
        const uint32_t v = ld_dev(&g[b]);
        h[b] = v;
        if (v) st_dev(&g[b], 0u);   // clean for the next use
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
    if (LEVEL == 1) {
        if (tid == 0) {
            st->pfx = (pfx << (HSHIFT - REF1_SHIFT)) | (uint32_t)bin;
            st->r2 = rank;
        }
        return;
    }
    // slabs in order: ties are taken lowest index first, i.e. earlier slabs first
    const uint32_t spp = slabs_per_part(A, s.td), ptile0 = A.segtab[s.td.seg_first].tile0,
                   ptiles = A.segtab[s.td.seg_first].ntiles;
    uint32_t carry_q = 0, carry_o = 0;
    for (uint32_t s0 = 0; s0 < nslabs; s0 += SLAB_THREADS) {
        const uint32_t si = s0 + tid;
        uint32_t *rec = slab_record(A, ptile0 + (si / spp) * ptiles + (si % spp) * SLAB_TILES, j);
        uint32_t G = 0, Q = 0;
        if (si < nslabs) {
            G = ld_dev(&rec[2 + bin + 1]);
            Q = ld_dev(&rec[2 + bin]) - G;
        }
        uint32_t totq, toto;
        const uint32_t qb = carry_q + block_excl_scan<(int)SLAB_WAVES>(Q, wsum, totq);
        const uint32_t take = min(Q, (rank > qb) ? (rank - qb) : 0u);
        const uint32_t ob = carry_o + block_excl_scan<(int)SLAB_WAVES>(G + take, wsum, toto);
        if (si < nslabs) {
            st_dev(&rec[0], ob);
            st_dev(&rec[1], take);
        }
        carry_q += totq;
        carry_o += toto;
    }
    if (tid == 0) {
        st->T = (pfx << REF1_SHIFT) | (uint32_t)bin;
        if (carry_o != k) atomicAdd(&A.stats->internal_errors, 1ull);
    }
}

// Winners are staged per tile in LDS and leave as coalesced runs; the state is written by whole
// 64-byte lines wherever a line has a winner (at these densities most lines that have one would
// otherwise be read, merged and written back by the memory side for every 4-byte store).
template <int OP>
__global__ __launch_bounds__(SLAB_THREADS) void k_dense_emit(const SelectArgs A)
{
    __shared__ uint2 stage_all[SLAB_WAVES][TILE];
    __shared__ uint32_t wtot[SLAB_WAVES];
    Slab s;
    if (!find_slab(A, s)) return;
    const SegState *st = &A.segstate[s.part.j];
    const uint32_t status = st->status;
    if (status != SEG_ACTIVE && status != SEG_ALL) return;
    const PlanEntry pe = A.plan[s.part.j];
    const uint32_t lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const bool all = (status == SEG_ALL);
    const uint32_t *rec = slab_record(A, s.tile0, s.part.j);
    // density 1: everything is a "tie" that is sent, at its own position
    const uint32_t T = all ? 0u : st->T;
    const uint32_t take = all ? 0u : rec[1];
    uint32_t bits[TPW][4][4], in[TPW];
    load_slab<OP>(A, s, bits, in);
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
    const uint32_t sum = wave_sum(mine);         // at most 4096 of either kind
    if (lane == 0) wtot[wave] = sum;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (uint32_t w = 0; w < SLAB_WAVES; ++w) before += (w < wave) ? wtot[w] : 0u;
    uint32_t eq = before >> 16;                  // ties seen before this row
    uint32_t pos = (before & 0xFFFFu) + min(eq, take) +
                   (all ? max(s.tile0 * TILE, s.td.off) - s.td.off : rec[0]);
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
                        f[x] = er < take;
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
    const dim3 grid(a.nparts * a.slabs), block(SLAB_THREADS);
    if (op == SEL_PULL_V) {
        launch_k(k_dense_refine<SEL_PULL_V, 1>, grid, block, st, ev0, nullptr, a);
        launch_k(k_dense_refine<SEL_PULL_V, 2>, grid, block, st, nullptr, nullptr, a);
        launch_k(k_dense_emit<SEL_PULL_V>, grid, block, st, nullptr, ev1, a);
    } else {      // worker and difference row rank the same buffer
        launch_k(k_dense_refine<SEL_PULL, 1>, grid, block, st, ev0, nullptr, a);
        launch_k(k_dense_refine<SEL_PULL, 2>, grid, block, st, nullptr, nullptr, a);
        if (op == SEL_WORKER) launch_k(k_dense_emit<SEL_WORKER>, grid, block, st, nullptr, ev1, a);
        else launch_k(k_dense_emit<SEL_PULL>, grid, block, st, nullptr, ev1, a);
    }
}

}  // namespace dgs
