// Pick (histogram -> candidate threshold) and the selection kernel of libdgs: per tensor the
// exact k-th largest magnitude with the lowest-index tie rule ("thr <- R% of |x|" in
// Algorithms 1-3), the ordered emission ("encode()"), the state fix-up (Eq. 12 / Eq. 6) and
// the next threshold hint -- all tensors in one launch.
#include "dgs_tensor.h"

namespace dgs {

// ---------------------------------------------------------------------------
// pick: key histogram (bits [30:19], nonzero keys only) -> candidate threshold
// ---------------------------------------------------------------------------

// sample != 0: the histogram is that of a sample of the tensor, zero keys included (its total is
// the number of sampled elements).  The ranks shrink with the sampled share; the candidate rank
// aims at 2 k instead of the plan's and gets two standard deviations of slack on top, since a
// threshold that lets too few through costs a second collection and one that lets a few more
// through costs nothing.  A tensor that was sampled completely keeps the plan's ranks.
__global__ __launch_bounds__(256) void k_pick(const TensorDesc *tdesc, const PlanEntry *plan,
                                              uint32_t *ghist, uint32_t *tau, uint32_t *tprev,
                                              DevStats *stats, uint32_t sample)
{
    const uint32_t j = blockIdx.x;
    if (!tdesc[j].big) return;
    __shared__ uint32_t h[HBINS];
    __shared__ uint32_t rowsum[64];
    __shared__ int res[6];
    __shared__ uint32_t wsum[4];
    uint32_t *g = ghist + (size_t)j * HBINS;
    uint32_t mine = 0;
    for (uint32_t b = threadIdx.x; b < HBINS; b += 256) {
        const uint32_t v = g[b];
        h[b] = v;
        mine += v;
        g[b] = 0;   // leave the histogram clean for the next use
    }
    PlanEntry pe = plan[j];
    if (sample) {
        const uint32_t total = block_sum<4>(mine, wsum);
        // from here on the histogram is that of the nonzero keys, as in a full pass (bucket 0 held
        // the zeros; keys below 2^19, denormals of about 1e-39, go with them)
        if (threadIdx.x == 0) h[0] = 0;
        __syncthreads();
        const uint32_t n = tdesc[j].n;
        if (total < n) {
            const double share = (double)total / (double)n;
            const double want = share * (double)min(2u * pe.k, n);
            const uint32_t k2s = (uint32_t)ceil(want + 2.0 * sqrt(want)) + 1u;
            pe.k2 = max(1u, min(k2s, total));
            pe.k = max(1u, min((uint32_t)ceil(share * (double)pe.k), pe.k2));
        }
    }
    uint32_t t, tp;
    pick_from_hist<4>(h, pe, rowsum, res, t, tp);
    if (sample) {
        // A sample that holds fewer nonzeros than the scaled k says nothing about where the k-th
        // key lies, except that it cannot be far above the smallest nonzero seen: that bucket
        // anchors the window histograms then (a full pass knows the bucket itself).
        __shared__ uint32_t lowbin;
        if (threadIdx.x == 0) lowbin = 0xFFFFFFFFu;
        __syncthreads();
        uint32_t mine_low = 0xFFFFFFFFu;
        for (uint32_t b = 1 + threadIdx.x; b < HBINS; b += 256)
            if (h[b] != 0) { mine_low = b; break; }
        if (mine_low != 0xFFFFFFFFu) atomicMin(&lowbin, mine_low);
        __syncthreads();
        if (tp == 0 && lowbin != 0xFFFFFFFFu) tp = (lowbin << HSHIFT) + (1u << (HSHIFT - 1));
    }
    if (threadIdx.x == 0) {
        tau[j] = t;
        tprev[j] = tp;
    }
}

void launch_pick(const TensorDesc *tdesc, const PlanEntry *plan, uint32_t *ghist, uint32_t *tau,
                 uint32_t *tprev, DevStats *stats, uint32_t J, bool sample, void *stream)
{
    hipLaunchKernelGGL(k_pick, dim3(J), dim3(256), 0, (hipStream_t)stream, tdesc, plan, ghist, tau, tprev,
                       stats, sample ? 1u : 0u);
}

// Dense request: the histogram covers every nonzero element of the tensor, so the bucket that
// holds the k-th key is certain (the zeros, not counted by the pass, complete bucket 0).
__global__ __launch_bounds__(1024) void k_pick_dense(const TensorDesc *tdesc, const PlanEntry *plan, uint32_t *ghist,
                                                     uint32_t *dprev, SegState *segstate, DevStats *stats)
{
    const uint32_t j = blockIdx.x;
    const TensorDesc td = tdesc[j];
    if (!td.big) return;
    __shared__ uint32_t h[HBINS];
    __shared__ uint32_t rowsum[64];
    __shared__ int res[6];
    __shared__ uint32_t wsum[SEL_WAVES];
    uint32_t *g = ghist + (size_t)j * HBINS;
    uint32_t mine = 0;
    for (uint32_t b = threadIdx.x; b < HBINS; b += SEL_THREADS) {
        const uint32_t v = g[b];
        h[b] = v;
        mine += v;
        g[b] = 0;   // leave the histogram clean for the next use
    }
    const uint32_t nonzero = block_sum<SEL_WAVES>(mine, wsum);
    if (threadIdx.x == 0) h[0] += td.n - nonzero;
    const uint32_t k = plan[j].k;
    find_ranks<HBINS, SEL_WAVES>(h, k, 0u, 0u, rowsum, res);
    if (threadIdx.x == 0) {
        SegState *st = &segstate[j];
        st->status = (k == td.n) ? SEG_ALL : SEG_ACTIVE;
        st->pfx = (uint32_t)res[0];
        st->r2 = (uint32_t)res[1];
        const uint32_t now = (uint32_t)res[0] + 1u, was = (dprev != nullptr) ? dprev[j] : 0u;
        st->T = (was == (now | DPREV_STABLE)) ? 1u : 0u;
        if (dprev != nullptr) dprev[j] = now | ((was & ~DPREV_STABLE) == now ? DPREV_STABLE : 0u);
        atomicAdd(&stats->segmented_tensors, 1ull);
    }
}

void launch_pick_dense(const TensorDesc *tdesc, const PlanEntry *plan, uint32_t *ghist, uint32_t *dprev, SegState *segstate,
                       DevStats *stats, uint32_t J, void *stream)
{
    hipLaunchKernelGGL(k_pick_dense, dim3(J), dim3(SEL_THREADS), 0, (hipStream_t)stream, tdesc, plan, ghist, dprev,
                       segstate, stats);
}

// ---------------------------------------------------------------------------
// the selection kernel
// ---------------------------------------------------------------------------
//
// Grid, where the chain has launches of its own or there is none: block b < G is the JOIN of join group b (1024 threads; a
// group is a tensor, or up to GROUP_TILES tiles of one).  With the re-collecting roles enabled, nb = ceil(P / bgroup)
// RE-HISTOGRAM blocks follow (P: the number of parts), then as many RE-COLLECTION blocks; block
// b of a role looks after parts b, b + nb, b + 2 nb, ... in turn, so the parts of one tensor
// lie in different blocks.  These blocks act on tensors of several parts whose prediction
// failed, and pass over everything else.  Where the chain is part of the launch, one block per run of parts of the
// tensors that take it comes before all of these (its window histogram; the last of a tensor goes on as that tensor's JOIN,
// whose own block leaves at once), and two blocks per slab (ranking, then emission) come behind.
//
//   JOIN      compacts the candidates the streaming pass left in the part's tiles into one
//             ordered list.  The workgroup that arrives last for a tensor (the only one, for a
//             tensor of one part) gathers the parts' lists and SELECTS: exact k-th key, ordered
//             emission, state fix-up, next hint.  A tensor planned for the chain only
//             gets its key window resolved here.  Lists that are complete but beyond one
//             workgroup's reach are trimmed on the way (threshold from their own histogram).
//             If the prediction failed otherwise (fewer candidates than k, an overflowed tile)
//             the tensor is left pending: a tensor of one part is collected again on the spot,
//             for the others the verdict releases the waiting roles.
//   RE-HISTOGRAM  every part counts the keys of its own elements; the last one derives a fresh
//             threshold and publishes it.
//   RE-COLLECTION every part compacts its elements at or above that threshold straight from
//             the buffers into its list; the last one selects as above.  What still fails then
//             (one value filling the tensor, say) is selected from the buffers by that one
//             workgroup -- slow, never wrong.
//
// Waiting is only ever for blocks with a lower index, and every wait is bounded (A.spin_limit polls); why that
// makes progress is stated at the chain (dgs_chain.h).

// HERE: the chain's workgroups are in this launch, for the tensors that take it: before the others one per run of parts
// (the window histograms), behind them two per slab.  (They have no use for most of the LDS, but with 128 registers
// there is one workgroup on a compute unit anyway.)
// (The tables that a workgroup starts with come as arguments of their own, which are in registers then.)
template <int OP, bool HERE>
__global__ __launch_bounds__(SEL_THREADS) void k_select(const SegDesc *grptab, const TensorDesc *tdesc, const PlanEntry *plan,
                                                        uint32_t *tau, uint32_t *tprev, uint32_t ngroups, uint32_t nwin,
                                                        const SelectArgs rest)
{
    SelectArgs A = rest;
    A.grptab = grptab;
    A.tdesc = tdesc;
    A.plan = plan;
    A.tau = tau;
    A.tprev = tprev;
    A.ngroups = ngroups;
    A.nwin = nwin;
    __shared__ PartShared P;
    __shared__ uint2 llist[SEL_LDS_LIST];
    const uint32_t tid = threadIdx.x;
    const bool window = HERE && blockIdx.x < A.nwin;
    const uint32_t block = HERE ? blockIdx.x - A.nwin : blockIdx.x;      // (of the roles behind those)
    if (!window && block >= A.ngroups) {
        // RE-HISTOGRAM / RE-COLLECTION: this workgroup looks after up to B_GROUP parts, nb apart,
        // so that the parts of one failed tensor are spread over as many workgroups as there are
        const uint32_t nb = (A.nparts + A.bgroup - 1) / A.bgroup;
        const uint32_t b = block - A.ngroups, standby = A.repair && A.multi ? 2u * nb : 0u;
        if (HERE && b >= standby) {
            const uint32_t s = b - standby;
            finish_slab<OP, SEL_THREADS, true>(A, s >= A.nslab, A.slabtab[s < A.nslab ? s : s - A.nslab], *(FinishShared *)llist);
            return;
        }
        standby_block<OP, HERE ? FORM_CHAIN : FORM_SELECT>(A, b, nb, P, llist);
        return;
    }
    const SegDesc sd = window ? A.wintab[blockIdx.x] : A.grptab[block];      // this workgroup's join group, or run of parts
    const uint32_t j = sd.j;
    const TensorDesc td = A.tdesc[j];
    const PlanEntry pe = A.plan[j];
    const bool multi = td.ngrp > 1;               // the groups' lists go to the last group to arrive
    const bool has_parts = td.nseg > 1;           // a failed prediction is collected again part by part
    SegState *st = &A.segstate[j];
    uint2 *plist = A.ord + (size_t)(sd.tile0 + j) * CAPT;       // this group's list

    {
        // ------------------------------------------------------------------ JOIN
        if (HERE && !window && pe.seg) return;
        if (!td.big || A.dense) {
            if (sd.sidx != 0) return;
            if (tid == 0) st->status = SEG_DONE;
            if (A.dense) dense_select<OP, false>(A, td, pe, j, td.big ? A.tau[j] : TAU_NEVER, P, llist);
            else small_select<OP, false>(A, td, pe, j, P.S);
            return;
        }
        const uint32_t tau_cur = A.tau[j];
        const uint32_t tprev_cur = A.tprev[j];
        uint32_t cs = 0, kmin = 0xFFFFFFFFu;
        bool ovf = false;
        // window of the single-workgroup selection: starts at the collection threshold or, when
        // that lies far below (a relaxed hint), 1024 buckets under the previous k-th key
        const uint32_t win_join = win_base_of<OP>(tau_cur, tprev_cur);
        uint32_t *verdict = (has_parts && A.repair) ? &st->verdict : nullptr;
        uint32_t status;
        if (pe.seg) {
            // a tensor that takes the chain: its parts have counted their candidates already, and
            // one workgroup reads the result
            if (HERE) {
                if (!window_run(A, sd, td, tau_cur, tprev_cur, P)) return;
            } else {
                if (sd.sidx != 0) return;
                uint32_t o = 0, mine = 0;
                for (uint32_t p = tid; p < td.nseg; p += SEL_THREADS) {
                    const uint32_t v = A.segcnt[td.seg_first + p];
                    mine += v & 0x7FFFFFFFu;
                    o |= v >> 31;
                }
                cs = block_sum<SEL_WAVES>(mine, P.S.wsum);
                ovf = __syncthreads_or((int)o) != 0;
            }
            status = tensor_select<OP, HERE ? FORM_CHAIN : FORM_SELECT>(A, td, pe, j, 0, false, true, cs, ovf, kmin, tau_cur, tprev_cur, win_join,
                                       false, verdict, P, llist);
        } else if (multi) {
            cs = join_part(A, td, sd, P, ovf, [&](uint32_t pos, uint2 e) { st_dev(&plist[pos], e); });
            if (tid == 0) st_dev(&A.grpcnt[block], cs | (ovf ? 0x80000000u : 0u));
            if (!arrive_last(&st->arrive[0], td.ngrp, &P.bc)) return;
            status = tensor_select<OP, HERE ? FORM_CHAIN : FORM_SELECT>(A, td, pe, j, 0, true, false, cs, ovf, kmin, tau_cur, tprev_cur, win_join, true,
                                       verdict, P, llist);
        } else {
            for (uint32_t b = tid; b < WIN_BINS; b += SEL_THREADS) P.S.h[b] = 0;
            if (tid == 0) P.S.kmin = 0xFFFFFFFFu;
            __syncthreads();
            uint2 *glist = plist;
            cs = join_part(A, td, sd, P, ovf, [&](uint32_t pos, uint2 e) {
                put_entry(llist, glist, pos, e);
                kmin = min(kmin, e.y & 0x7FFFFFFFu);
                window_count<OP>(P.S.h, win_join, e.y & 0x7FFFFFFFu);
            });
            kmin = wave_min_to_last(kmin);
            if (lane_id() == 63) atomicMin(&P.S.kmin, kmin);
            wait_mem();
            __syncthreads();
            kmin = P.S.kmin;
            status = tensor_select<OP, HERE ? FORM_CHAIN : FORM_SELECT>(A, td, pe, j, 0, false, false, cs, ovf, kmin, tau_cur, tprev_cur, win_join, true,
                                       verdict, P, llist);
        }
        if (has_parts) return;        // the re-collecting workgroups have the verdict
        if (status != SEG_PENDING) return;
        recollect_here<OP, HERE ? FORM_CHAIN : FORM_SELECT>(A, td, pe, j, P, llist);
        return;
    }

}

// Pull on the printed state: sent_k += G, a thread per pair, behind the selection kernel.  A tensor's selection
// runs on one compute unit, and what that can have in flight bounds a scattered read and write of its row:
// 7.6 us for 2360 pairs, which the whole chip does in the 5 us of this launch (32-worker server on ResNet-50
// shapes 72.7 -> 68.8 us an event).  The row follows the message whatever becomes of the model meanwhile.  Only in
// a context that has counted an internal error may the message hold pairs that no selection has written:
// there, what the row does not show is not added.
__global__ __launch_bounds__(256) void k_add_sent(float *sent, const float *model, uint32_t n, const uint32_t *idx,
                                                  const float *val, uint32_t K, const DevStats *stats)
{
    const uint32_t e = blockIdx.x * 256 + threadIdx.x;
    if (e >= K) return;
    const uint32_t ix = idx[e];
    const float v = val[e];
    if (ix >= n) return;
    const float old = sent[ix];
    if (stats->internal_errors != 0 && __float_as_uint(model[ix] - old) != __float_as_uint(v)) return;
    store_scattered(&sent[ix], old + v);
}

void launch_add_sent(const SelectArgs &a, uint32_t K, void *stream, void *ev1)
{
    launch_k(k_add_sent, dim3((K + 255u) / 256u), dim3(256), (hipStream_t)stream, nullptr, ev1, a.state, a.model, a.n,
             (const uint32_t *)a.out_idx, (const float *)a.out_val, K, (const DevStats *)a.stats);
}

template <int OP>
static void launch_select_t(const SelectArgs &a, hipStream_t st, void *ev0, void *ev1)
{
    const uint32_t nb = (a.nparts + a.bgroup - 1) / a.bgroup;
    const uint32_t blocks = a.ngroups + (a.repair && a.multi ? 2u * nb : 0u);
    if (a.nwin) launch_k(k_select<OP, true>, dim3(a.nwin + blocks + 2u * a.nslab), dim3(SEL_THREADS), st, ev0, ev1, a.grptab, a.tdesc,
                         a.plan, a.tau, a.tprev, a.ngroups, a.nwin, a);
    else launch_k(k_select<OP, false>, dim3(blocks), dim3(SEL_THREADS), st, ev0, ev1, a.grptab, a.tdesc, a.plan, a.tau, a.tprev,
                  a.ngroups, a.nwin, a);
}

void launch_select(int op, const SelectArgs &a, void *stream, void *ev0, void *ev1)
{
    hipStream_t st = (hipStream_t)stream;
    if (a.ngroups == 0) return;
    if (op == SEL_WORKER) launch_select_t<SEL_WORKER>(a, st, ev0, ev1);
    else if (op == SEL_PULL) launch_select_t<SEL_PULL>(a, st, ev0, ev1);
    else launch_select_t<SEL_PULL_V>(a, st, ev0, ev1);
}

}  // namespace dgs
