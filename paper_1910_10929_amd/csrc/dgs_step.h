// A whole call in one launch, for layouts small enough that every unit of the work below has a compute unit to itself or
// nearly so: what a worker step or a pull costs there is launches and the latency of one workgroup after another, not bytes.
// Streaming pass and selection / one launch, us: a round (with push and apply) on nine tensors of 270 K elements in all 37.5 / 34.7, on
// one of 2^20 at 1 % 54.7 / 47.2 (more in dgs_device.h, where the line lies).  What bounds it now is a chain: the start of the
// workgroups (a die starts one of 16 wavefronts every 0.15 us), loads, the flags, the lists' way into one compute unit (29 bytes
// a ns), and the barriers of the ranking there, of which a tensor has only one workgroup.
//
//   COLLECT  one workgroup per unit of a tensor (4, 8 or 16 tiles' worth of its own elements: a unit never crosses a tensor's
//            border): accumulates, stores the state, compacts what reaches the predicted threshold into the unit's list, and
//            says so in a flag.  A small tensor (up to SMALL_N elements) is accumulated and selected in registers by its one
//            workgroup.
//   RANK     one workgroup per other tensor: awaits its units' flags, takes the lists into registers and ranks, and emits if the
//            tensor has few winners.
//   the standby roles of k_select, for tensors whose prediction failed
//   EMIT     where some tensor has many winners; for it and the other large ones, if they have too many entries to be held: a
//            wavefront per unit has its list in registers by the time the ranking publishes the k-th key, and writes the
//            unit's stretch of the message; positions by look-back over the workgroups before it.
//
// As everywhere, a workgroup waits only for workgroups with lower indices.  The state that COLLECT stores is written through
// (a copy of it left dirty in one die's L2 would end up over what the emission stores from another), and whoever reads
// it again in the same launch, after a failed prediction, reads past the L2 (quad_bits, row_value with WRITTEN).
#pragma once
#include "dgs_tensor.h"

namespace dgs {

// COLLECT of unit `unit` (u).
template <int OP>
__device__ __forceinline__ void step_collect(const SelectArgs &A, const StepUnit &u, uint32_t unit, PartShared &P)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uniform(tid >> 6), rows = u.rows;
    const uint32_t end = u.e0 + u.count, w0 = u.e0 + wave * rows * 256u;
    const uint32_t tau = A.tau[u.j];
    float a[4][4];
    const bool full = w0 + rows * 256u <= end;       // (wave-uniform)
    if (full) {
        f32x4 g[4], s[4];
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            if (r >= rows) continue;
            const uint32_t e = w0 + r * 256u + lane * 4u;
            if (OP == SEL_WORKER) g[r] = *(const f32x4_any *)(A.grad + e);
            if (OP == SEL_PULL_V) g[r] = *(const f32x4_any *)(A.model + e);
            s[r] = *(const f32x4_any *)(A.state + e);
        }
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r)
#pragma unroll
            for (int x = 0; x < 4; ++x)
                a[r][x] = (r >= rows) ? 0.0f
                          : (OP == SEL_WORKER) ? __builtin_fmaf(A.lr, g[r][x], s[r][x])
                          : (OP == SEL_PULL_V) ? g[r][x] - s[r][x] : s[r][x];
    } else {
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const uint32_t e = w0 + r * 256u + lane * 4u + x;
                a[r][x] = 0.0f;
                if (r >= rows || e >= end) continue;
                const float s = A.state[e];
                a[r][x] = (OP == SEL_WORKER) ? __builtin_fmaf(A.lr, A.grad[e], s)
                          : (OP == SEL_PULL_V) ? A.model[e] - s : s;
            }
    }
    // what reaches the threshold (at least 1: what lies beyond the unit, read as 0, does not)
    uint64_t mk[4][4];
    uint32_t mine = 0;
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r)
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            mk[r][x] = ballot64((__float_as_uint(a[r][x]) & 0x7FFFFFFFu) >= tau);
            mine += (uint32_t)__popcll(mk[r][x]);
        }
    if (lane == 0) P.wtot[wave] = mine;
    __syncthreads();
    uint32_t total, run = sum_waves<SEL_WAVES>(P.wtot, total);
    const bool fits = total <= u.cap;
    if (fits && mine != 0) {
        uint32_t *val = (uint32_t *)A.ord + step_val(u), *idx = (uint32_t *)A.ord + step_idx(u);
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            if ((mk[r][0] | mk[r][1] | mk[r][2] | mk[r][3]) == 0) continue;
            uint32_t p = run + mbcnt64(mk[r][0]) + mbcnt64(mk[r][1]) + mbcnt64(mk[r][2]) + mbcnt64(mk[r][3]);
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if ((mk[r][x] >> lane) & 1ull) {
                    st_dev(&val[p], __float_as_uint(a[r][x]));
                    st_dev(&idx[p], w0 + r * 256u + lane * 4u + x);
                    ++p;
                }
            run += (uint32_t)(__popcll(mk[r][0]) + __popcll(mk[r][1]) + __popcll(mk[r][2]) + __popcll(mk[r][3]));
        }
    }
    if (OP == SEL_WORKER) {                          // (behind the barrier above, which would wait for the stores)
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            if (r >= rows) continue;
            if (full) {
                f32x4 o;
#pragma unroll
                for (int x = 0; x < 4; ++x) o[x] = a[r][x];
                store_through16(A.state + uniform(w0), (r * 256u + lane * 4u) * 4u, o);
            } else {
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const uint32_t e = w0 + r * 256u + lane * 4u + x;
                    if (e < end) st_dev((uint32_t *)A.state + e, __float_as_uint(a[r][x]));
                }
            }
        }
    }
    if (tid == 0) slab_publish<false>(step_word(A, u.ord0), 0u, 0u, 0u);      // (the emission has published nothing yet)
    wait_mem();
    __syncthreads();
    const uint32_t flag = STEP_READY | (fits ? total : STEP_OVER);
    if (tid == 0) st_dev(&A.stepflag[unit], flag);
    if (tid == 64 && step_emits(A, u.n)) st_dev(&A.stepflag[A.nstep + unit], flag);
}

// The selection where the lists fit the registers: every thread takes the same share of its unit's list, ITEMS entries at
// most, so that the order of threads is the order of indices.  Keys are counted in the hinted window only; its bucket of the
// k-th key mostly holds a handful of entries, which every wavefront ranks bit by bit.  EMITS: the values alone are read, and
// the k-th key is published; otherwise the winners are emitted.  Returns false, with nothing done but the window counted, if the
// window has no answer.  (All lists into LDS by position first, then the selection that joins end with: a round on one tensor of
// 2^20 47.9 us, 47.2 so.)
template <int OP, bool EMITS>
__device__ __forceinline__ bool step_select(const SelectArgs &A, const TensorDesc &td, const PlanEntry &pe, const SegDesc &rd, uint32_t c,
                                            uint32_t share, uint32_t log_lanes, uint32_t tau_cur, uint32_t tprev_cur, uint32_t hint2_cur,
                                            uint32_t *verdict, PartShared &P)
{
    constexpr uint32_t ITEMS = EMITS ? STEP_ITEMS_KEYS : STEP_ITEMS, SHIFT = win_shift(OP);
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = uniform(tid >> 6), j = rd.j;
    const uint32_t win = win_base_of<OP>(tau_cur, tprev_cur);
    uint32_t val[ITEMS], idx[EMITS ? 1 : ITEMS], km = 0xFFFFFFFFu;
    const uint32_t mine = ((wave << 6) >> log_lanes) < rd.ntiles ? share : 0u;      // (of this wavefront's threads)
    auto each = [&](auto f) {      // f(i) for this thread's entries
#pragma unroll
        for (uint32_t i = 0; i < ITEMS; i += 4) {
            if (i >= mine) break;
            f(i);
            f(i + 1u);
            f(i + 2u);
            f(i + 3u);
        }
    };
    {
        const uint32_t u = tid >> log_lanes, q0 = (tid & ((1u << log_lanes) - 1u)) * share;
        const uint32_t n = (u < rd.ntiles) ? P.pbase[u] : 0u;
        // (the lists of a tensor are equally far apart, and equally long but for the last)
        const StepUnit first = A.steptab[rd.tile0], last = A.steptab[rd.tile0 + rd.ntiles - 1u];
        const uint32_t at = step_val(first) + 2u * u * first.rows * 4u * CAPT + q0;
        const uint32_t at_idx = at + (u + 1u < rd.ntiles ? first.cap : last.cap);
#pragma unroll
        for (uint32_t i = 0; i < ITEMS; i += 4) {
            uint4 v = make_uint4(0u, 0u, 0u, 0u), x = v;
            if (i >= mine) break;                    // (uniform, as in all loops over the entries)
            if (q0 + i < n) {                        // (a list's last load may read up to three words behind it: there is room)
                v = ld_dev16((const uint32_t *)A.ord, at + i);
                if (!EMITS) x = ld_dev16((const uint32_t *)A.ord, at_idx + i);
            }
            val[i] = v.x; val[i + 1] = v.y; val[i + 2] = v.z; val[i + 3] = v.w;
            if (!EMITS) { idx[i] = x.x; idx[i + 1] = x.y; idx[i + 2] = x.z; idx[i + 3] = x.w; }
        }
        each([&](uint32_t i) {
            if (q0 + i >= n) val[i] = 0u;            // (no candidate has key 0)
            const uint32_t key = val[i] & 0x7FFFFFFFu;
            if (key == 0) return;
            window_count<OP>(P.S.h, win, key);
            km = min(km, key);
        });
    }
    if (mine != 0) {
        km = wave_min_to_last(km);
        if (lane == 63) atomicMin(&P.S.kmin, km);
    }
    __syncthreads();
    const uint32_t kmin = P.S.kmin;
    uint32_t R = 0, Eq = 0, qlow = 0, third = 0;
    bool measurable = false;
    if (wave < 3u) {                                 // (those that search)
        R = hint_rank<OP>(td, pe, !A.exact_mode, c, hint2_cur, A.m, A.young, &Eq);
        measurable = R != 0 && c >= R;
        qlow = max(c / 4u, min(c, 16u));
        third = measurable ? ((Eq <= c) ? Eq : 0u) : ((R != 0) ? (c - qlow + 1u) : 0u);
    }
    find_ranks<WIN_BINS, SEL_WAVES, true>(P.S.h, pe.k, measurable ? R : pe.k, third, P.S.rowsum, P.S.res);
    const int lo = win > (kmin >> SHIFT) ? 1 : 0;    // (bucket 0 holds what lies below the window, too)
    const int bk = P.S.res[0], bR = P.S.res[2], bE = P.S.res[4];
    const uint32_t r2 = (uint32_t)P.S.res[1], rR = (uint32_t)P.S.res[3];
    if (bk < lo || bk >= (int)WIN_BINS - 1 || bR < lo || bR >= (int)WIN_BINS - 1) return false;
    if (verdict && tid == 0) st_dev(verdict, 0x100u | (uint32_t)SEG_DONE);
    if (!EMITS && step_emits(A, td.n) && tid == 0) st_dev(&A.segstate[j].key, make_uint2(STEP_DONE, KEY_READY));      // (nobody else emits)
    uint32_t tau_next = 0, expect = 0, q_e = 0;
    if (tid == 0) window_hint<OP>(P.S.h, win, lo, bR, rR, bE, measurable, R, c, qlow, kmin, &tau_next, &expect, &q_e);
    const uint32_t sharing = P.S.h[bk], pfx = win + (uint32_t)bk;
    uint32_t T, rT;
    if (sharing <= FEW) {
        each([&](uint32_t i) {
            const uint32_t key = val[i] & 0x7FFFFFFFu;
            if (key != 0 && (key >> SHIFT) == pfx) P.S.few_key[atomicAdd(&P.S.few, 1u) & (FEW - 1u)] = key;
        });
        __syncthreads();
        uint32_t low;
        rank_few(P.S, sharing, r2, SHIFT, low, rT);
        T = (pfx << SHIFT) | low;
    } else {
        __syncthreads();
        for (uint32_t b = tid; b < (1u << SHIFT); b += SEL_THREADS) P.S.h[b] = 0;
        __syncthreads();
        each([&](uint32_t i) {
            const uint32_t key = val[i] & 0x7FFFFFFFu;
            if (key != 0 && (key >> SHIFT) == pfx) atomicAdd(&P.S.h[key & ((1u << SHIFT) - 1u)], 1u);
        });
        find_ranks<(1 << SHIFT), SEL_WAVES>(P.S.h, r2, 0u, 0u, P.S.rowsum, P.S.res);
        T = (pfx << SHIFT) | (uint32_t)P.S.res[0];
        rT = (uint32_t)P.S.res[1];
    }
    if (EMITS) {
        if (tid == 0) st_dev(&A.segstate[j].key, make_uint2(rT, KEY_READY | T));
    } else {
        uint32_t g = 0, q = 0;
        each([&](uint32_t i) {
            const uint32_t key = val[i] & 0x7FFFFFFFu;
            g += key > T ? 1u : 0u;
            q += key == T ? 1u : 0u;
        });
        uint32_t total;
        const uint32_t before = block_excl_scan<SEL_WAVES>(g | (q << 16), P.S.wsum, total);
        uint32_t above = before & 0xFFFFu, eq = before >> 16;
        if ((g | q) != 0) {
            float was[OP == SEL_PULL_V ? ITEMS : 1];
            if (OP == SEL_PULL_V)
                each([&](uint32_t i) { was[i] = ((val[i] & 0x7FFFFFFFu) >= T && idx[i] < A.n) ? A.state[idx[i]] : 0.0f; });
            each([&](uint32_t i) {
                const uint32_t key = val[i] & 0x7FFFFFFFu, at = above + min(eq, rT);
                const bool send = key > T || (key == T && eq < rT);      // (ties: lowest index first, rT of them are taken)
                above += key > T ? 1u : 0u;
                eq += key == T ? 1u : 0u;
                if (!send || at >= pe.k || !index_ok(A, idx[i])) return;
                const float v = __uint_as_float(val[i]);
                A.out_idx[pe.outoff + at] = idx[i];
                A.out_val[pe.outoff + at] = v;
                if (OP == SEL_WORKER) store_scattered(&A.state[idx[i]], A.m * v);
                else if (OP == SEL_PULL) store_scattered(&A.state[idx[i]], 0.0f);
                else store_scattered(&A.state[idx[i]], was[i] + v);
            });
        }
        if (tid == 0 && (total & 0xFFFFu) + min(total >> 16, rT) != pe.k) atomicAdd(&A.stats->internal_errors, 1ull);
    }
    if (tid == 0) {
        A.segstate[j].status = EMITS ? (uint32_t)SEG_ACTIVE : (uint32_t)SEG_DONE;
        atomicAdd(&A.stats->candidates, (unsigned long long)c);
    }
    list_hints(A, j, tau_next, expect, q_e, T, tau_cur, kmin);
    return true;
}

// What RANK does with lists that step_select has no answer for: too many entries for the registers, too few for the message, or a
// k-th key that has moved on.  They go into one list, LDS first, from which it is selected as from any other: as it is up to SEL_LIST_HARD
// entries, cut down beyond, and completed with zeros where every nonzero is in it.  Where many workgroups wait for the k-th key
// and the list is long, that alone is found.  Returns the tensor's status: SEG_DONE, SEG_ACTIVE (those workgroups go on), or
// SEG_PENDING (collect again).  us a worker step without momentum whose scale grows by 1.1 each time, in several launches / lists
// beyond the LDS list cut down where they lie / so: one tensor of 1M elements at 0.1 % 37.3 / 85.3 / 29.5, of 2M 63.5 / 150.7 / 52.6,
// of 4M at 0.05 % 84.7 / 201.6 / 71.6.
template <int OP>
__device__ __forceinline__ uint32_t step_lists(const SelectArgs &A, const TensorDesc &td, const PlanEntry &pe, const SegDesc &rd, uint32_t c,
                                               bool ovf, uint32_t tau_cur, uint32_t tprev_cur, uint32_t hint2_cur, uint32_t *verdict,
                                               PartShared &P, uint2 *llist)
{
    const uint32_t tid = threadIdx.x, j = rd.j;
    const bool emits = step_emits(A, td.n);
    const bool zerofill = !ovf && c < pe.k && tau_cur <= 1u;      // (every nonzero is in the lists)
    uint32_t status = SEG_PENDING;
    bool known = false;      // the verdict is out (once: the last of those who wait for it clears it)
    if (emits && !ovf && c >= pe.k && (c > SEL_LDS_LIST || pe.k > STEP_EMIT_K)) {
        known = true;
        status = SEG_ACTIVE;
        if (verdict && tid == 0) st_dev(verdict, 0x100u | (uint32_t)SEG_DONE);
        // A worker's key is found in the list, as if this workgroup emitted: its next threshold follows the drift then.  (step_rank's does
        // not: one tensor of 8M elements at 0.1 % without momentum, 50 calls on, 4.8 entries for each that is sent and a step of 72 us, 3.8
        // and 46 so.)  A pull's has none, and step_rank is quicker: an event on one tensor of 1M at 1 % 29.4 us, 32.3 from the list.
        if (OP == SEL_WORKER) {
            uint2 *glist = step_tail(A, td);
            const uint32_t win = win_base_of<OP>(tau_cur, tprev_cur);
            uint32_t km = 0xFFFFFFFFu;
            step_gather<true>(A, rd.tile0, rd.ntiles, P.pbase, [&](uint32_t p, uint32_t, uint32_t v) {
                put_entry(llist, glist, p, make_uint2(0u, v));
                km = min(km, v & 0x7FFFFFFFu);
                window_count<OP>(P.S.h, win, v & 0x7FFFFFFFu);
            });
            km = wave_min_to_last(km);
            if (lane_id() == 63) atomicMin(&P.S.kmin, km);
            wait_mem();
            __syncthreads();
            list_select<OP, true>(A, td, pe, j, c, P.S.kmin, tau_cur, hint2_cur, win, true, false, P, llist, glist);
            if (tid == 0) {
                atomicAdd(&A.stats->candidates, (unsigned long long)c);
                if (c > SEL_LIST_HARD) atomicAdd(&A.stats->repaired_tensors, 1ull);
            }
        } else {
            step_rank<OP>(A, td, pe, j, rd.tile0, rd.ntiles, c, tau_cur, hint2_cur, P);
        }
    } else if (!ovf && (c >= pe.k || zerofill)) {
        uint2 *glist = step_tail(A, td);
        uint32_t win = win_base_of<OP>(tau_cur, tprev_cur), km = 0xFFFFFFFFu, tau = tau_cur;
        const bool whole = c <= SEL_LIST_HARD;
        if (whole) {
            known = true;
            if (verdict && tid == 0) st_dev(verdict, 0x100u | (uint32_t)SEG_DONE);
        }
        step_gather<false>(A, rd.tile0, rd.ntiles, P.pbase, [&](uint32_t p, uint32_t ix, uint32_t v) {
            put_entry(llist, glist, p, make_uint2(ix, v));
            km = min(km, v & 0x7FFFFFFFu);
            window_count<OP>(P.S.h, win, v & 0x7FFFFFFFu);      // (the hinted window, on the way)
        });
        km = wave_min_to_last(km);
        if (lane_id() == 63) atomicMin(&P.S.kmin, km);
        wait_mem();
        __syncthreads();
        uint32_t kmin = P.S.kmin;
        if (zerofill) {
            zero_fill_emit<OP, written<OP, FORM_STEP>()>(SrcSplit{llist, glist}, c, td, pe, A, P.S.wsum);
            if (tid == 0) {
                A.tau[j] = 1u;
                A.hint2[j] = 0u;
                A.tprev[j] = 0u;
                atomicAdd(&A.stats->candidates, (unsigned long long)c);
            }
            status = SEG_DONE;
        } else {
            if (!whole) {
                c = trim_list(A, SrcSplit{llist, glist}, c, SEL_LIST_HARD, pe, verdict, P, llist, glist, tau);
                kmin = tau;      // (a lower bound; the window is counted from the list)
                win = 0xFFFFFFFFu;
                if (c != 0) {
                    known = true;
                    if (tid == 0) atomicAdd(&A.stats->repaired_tensors, 1ull);
                }
            }
            if (c != 0) {
                list_select<OP>(A, td, pe, j, c, kmin, tau, hint2_cur, win, whole, !whole, P, llist, glist);
                if (tid == 0) atomicAdd(&A.stats->candidates, (unsigned long long)c);
                status = SEG_DONE;
            }
        }
    }
    if (tid == 0) A.segstate[j].status = status;
    if (emits && status != SEG_ACTIVE && tid == 0) st_dev(&A.segstate[j].key, make_uint2(STEP_DONE, KEY_READY));
    if (verdict && !known) {
        wait_mem();
        __syncthreads();
        if (tid == 0) st_dev(verdict, 0x100u | status);
    }
    return status;
}

// RANK of the tensor whose units rd describes.
template <int OP>
__device__ __forceinline__ void step_rank_block(const SelectArgs &A, const SegDesc &rd, PartShared &P, uint2 *llist)
{
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid >> 6, j = rd.j, units = rd.ntiles;
    const TensorDesc td = A.tdesc[j];
    PlanEntry pe = A.plan[j];
    pe.seg = 0;                                      // (no tensor takes the chain here)
    const uint32_t tau_cur = A.tau[j], tprev_cur = A.tprev[j], hint2_cur = A.hint2[j];
    const bool has_parts = td.nseg > 1, emits = step_emits(A, td.n) && pe.k > STEP_EMIT_K;
    uint32_t *verdict = (has_parts && A.repair) ? &A.segstate[j].verdict : nullptr;
    for (uint32_t b = tid; b < WIN_BINS; b += SEL_THREADS) P.S.h[b] = 0;
    if (tid == 0) {
        P.S.few = P.all = 0;
        P.least = 0xFFFFFFFFu;
        P.S.kmin = 0xFFFFFFFFu;
    }
    __syncthreads();
    uint32_t f = 0;
    if (tid < units) {
        uint32_t *flag = &A.stepflag[rd.tile0 + tid];
        for (uint32_t spin = 0; spin < A.spin_limit; ++spin) {
            f = ld_dev(flag);
            if (f != 0) break;
            __builtin_amdgcn_s_sleep(1);
        }
    }
    const uint32_t n = (tid < units) ? (f & ~(STEP_READY | STEP_OVER)) : 0u;
    if (tid <= units) P.pbase[tid] = n;              // (counts, for now)
    if (64u * wave < units) {
        const uint32_t sum = wave_sum(n), low = wave_min_to_last(~n);
        if (lane == 63) {
            atomicAdd(&P.all, sum);
            atomicMin(&P.least, low);
        }
    }
    const bool bad = __syncthreads_or((tid < units && f == 0) || (f & STEP_OVER)) != 0;
    if (bad && __syncthreads_or(tid < units && f == 0)) {      // gave up waiting
        if (tid == 0) atomicAdd(&A.stats->internal_errors, 1ull);
        return;
    }
    uint32_t c = P.all;
    const uint32_t most = ~P.least;
    // The threads of a unit and the entries of each: four, in as few wavefronts as that takes (those without entries
    // have nothing to issue), or more where the units have no more threads.
    auto log_up = [](uint32_t x) { return x > 1u ? 32u - (uint32_t)__builtin_clz(x - 1u) : 0u; };
    static_assert(SEL_THREADS == 1u << 10, "threads of the units");
    const uint32_t log_lanes = min(log_up((most + 3u) / 4u), 10u - log_up(units));
    const uint32_t share = (((most + (1u << log_lanes) - 1u) >> log_lanes) + 3u) & ~3u;
    bool done = false;
    if (!bad && c >= pe.k && share <= (emits ? STEP_ITEMS_KEYS : STEP_ITEMS)) {
        done = emits ? step_select<OP, true>(A, td, pe, rd, c, share, log_lanes, tau_cur, tprev_cur, hint2_cur, verdict, P)
                     : step_select<OP, false>(A, td, pe, rd, c, share, log_lanes, tau_cur, tprev_cur, hint2_cur, verdict, P);
    }
    if (__builtin_expect(!done, 0)) {
        // too few entries, or too many, or a k-th key that has moved on: as for any other tensor's lists
        __syncthreads();
        for (uint32_t b = tid; b < WIN_BINS; b += SEL_THREADS) P.S.h[b] = 0;
        if (tid == 0) P.S.kmin = 0xFFFFFFFFu;
        const uint32_t ex = block_excl_scan<SEL_WAVES>(n, P.S.wsum, c);
        if (tid <= units) P.pbase[tid] = ex;
        __syncthreads();
        const uint32_t status = step_lists<OP>(A, td, pe, rd, c, bad, tau_cur, tprev_cur, hint2_cur, verdict, P, llist);
        if (!has_parts && status == SEG_PENDING) recollect_here<OP, FORM_STEP>(A, td, pe, j, P, llist);
    }
    if (tid < units) st_dev(&A.stepflag[rd.tile0 + tid], 0u);       // for the next launch
}

// EMIT: up to SEL_WAVES consecutive units of a tensor (eb.tile0: the first, eb.ntiles: how many, eb.sidx: which run of them),
// a wavefront each, a lane four entries.  One that gives up a wait, and every one of the tensor behind it, emits nothing and leaves the
// state as it is.
template <int OP>
__device__ __forceinline__ void step_emit(const SelectArgs &A, const SegDesc &eb, PartShared &P)
{
    const PlanEntry pe = A.plan[eb.j];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uniform(tid >> 6);
    const bool have = wave < eb.ntiles;
    const uint32_t unit = eb.tile0 + (have ? wave : 0u);
    const StepUnit u = A.steptab[unit], u0 = A.steptab[eb.tile0];
    SegState *st = &A.segstate[eb.j];
    const uint32_t per = u0.rows * 4u * TILE, units = (u0.n + per - 1u) / per, runs = (units + SEL_WAVES - 1u) / SEL_WAVES;
    const uint32_t stride = u0.rows * 4u * CAPT * SEL_WAVES;       // (of the lists of two runs)
    uint2 *word = step_word(A, u0.ord0);
    uint32_t f = 0;
    if (have) {
        uint32_t *flag = &A.stepflag[A.nstep + unit];
        for (uint32_t spin = 0; spin < A.spin_limit; ++spin) {
            f = uniform(ld_dev(flag));
            if (f != 0) break;
            __builtin_amdgcn_s_sleep(1);
        }
        if (lane == 0) st_dev(flag, 0u);             // (read by nobody else)
    }
    // (where the ranking has given up on the lists already, others may be writing them again)
    const uint2 peek = ld_dev(&st->key);
    const uint32_t n = (uniform(peek.y) != 0 && uniform(peek.x) == STEP_DONE) ? 0u : f & ~(STEP_READY | STEP_OVER);
    constexpr uint32_t HELD = 2;                     // entries of a lane in registers: HELD times four, 256 HELD of the unit
    uint32_t val[HELD][4], idx[HELD][4];
    float was[HELD][4];
    auto fetch = [&](uint32_t q, uint32_t (&v)[4], uint32_t (&x)[4], float (&old)[4]) {      // entries q .. q + 3
        uint4 a = make_uint4(0u, 0u, 0u, 0u), b = a;
        if (q < n) {                                 // (a list's last load may read up to three words behind it: there is room)
            a = ld_dev16((const uint32_t *)A.ord, step_val(u) + q);
            b = ld_dev16((const uint32_t *)A.ord, step_idx(u) + q);
        }
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        x[0] = b.x; x[1] = b.y; x[2] = b.z; x[3] = b.w;
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) old[i] = (OP == SEL_PULL_V && q + i < n && x[i] < A.n) ? A.state[x[i]] : 0.0f;
    };
#pragma unroll
    for (uint32_t h = 0; h < HELD; ++h) fetch(256u * h + 4u * lane, val[h], idx[h], was[h]);
    const bool late = __syncthreads_or(have && f == 0) != 0;
    const uint2 key = wait_pair(&st->key, late ? 1u : A.spin_limit, P.pair);
    if (key.y == 0 || late) {                        // gave up waiting
        if (tid == 0) {
            slab_publish<false>(word, SLAB_FAIL, 0u, 0u);
            atomicAdd(&A.stats->internal_errors, 1ull);
        }
        return;
    }
    if (key.x != STEP_DONE) {
        const uint32_t T = uniform(key.y & ~KEY_READY), rT = uniform(key.x);
        uint32_t mine = 0;                           // entries above T (low half) and equal to it: 64 a lane at most of a unit's 4096
        auto count = [&](uint32_t q, const uint32_t (&v)[4]) {
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {
                const uint32_t k = v[i] & 0x7FFFFFFFu;
                if (q + i < n) mine += (k > T ? 1u : 0u) + (k == T ? 0x10000u : 0u);
            }
        };
#pragma unroll
        for (uint32_t h = 0; h < HELD; ++h) count(256u * h + 4u * lane, val[h]);
#pragma unroll 1
        for (uint32_t q0 = 256u * HELD; q0 < n; q0 += 256u) {
            uint32_t v[4], x[4];
            float old[4];
            fetch(q0 + 4u * lane, v, x, old);
            count(q0 + 4u * lane, v);
        }
        const uint32_t sum = wave_sum(mine);
        // (a run's counts together: 16 units of up to 4096 entries, of which up to 65536 may be equal)
        uint32_t gall, qall;
        if (lane == 0) {
            P.wtot[wave] = sum & 0xFFFFu;
            P.wmax[wave] = sum >> 16;
        }
        __syncthreads();
        const uint32_t g0 = sum_waves<SEL_WAVES>(P.wtot, gall), q0 = sum_waves<SEL_WAVES>(P.wmax, qall);
        if (wave == 0) {
            const bool head = eb.sidx == 0;
            if (lane == 0) slab_publish<false>(word, head ? SLAB_SUM : SLAB_OWN, gall, qall);
            uint32_t gb, qb;
            const uint32_t ord00 = u0.ord0 - eb.sidx * stride;      // the tensor's first list
            const bool known = slab_look_back<false>(A, eb.sidx, 0u, [&](uint32_t i) { return step_word(A, ord00 + i * stride); }, gb, qb);
            if (lane == 0) {
                if (!head) slab_publish<false>(word, known ? SLAB_SUM : SLAB_FAIL, gb + gall, qb + qall);
                P.pair[0] = gb;
                P.pair[1] = qb;
                P.bc = known ? pe.k : 0u;
                if (known && eb.sidx + 1u == runs && (gb + gall + rT != pe.k || qb + qall < rT))
                    atomicAdd(&A.stats->internal_errors, 1ull);
            }
        }
        __syncthreads();
        uint32_t eq = P.pair[1] + q0, pos = P.pair[0] + g0 + min(eq, rT);
        const uint32_t limit = P.bc;
        auto emit = [&](uint32_t q, const uint32_t (&v)[4], const uint32_t (&x)[4], const float (&old)[4]) {      // (all lanes call)
            uint64_t m[4];
            bool in[4];
            uint32_t e = eq;
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {
                in[i] = q + i < n;
                m[i] = ballot64(in[i] && (v[i] & 0x7FFFFFFFu) == T);
                e += mbcnt64(m[i]);
                eq += (uint32_t)__popcll(m[i]);
            }
            uint32_t at = pos;
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {       // (ties: lowest index first, rT of them are taken)
                const uint32_t k = v[i] & 0x7FFFFFFFu;
                const bool tie = in[i] && k == T;
                in[i] = in[i] && (k > T || (tie && e < rT));
                e += tie ? 1u : 0u;
                m[i] = ballot64(in[i]);
                at += mbcnt64(m[i]);
                pos += (uint32_t)__popcll(m[i]);
            }
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {
                if (!in[i]) continue;
                const float y = __uint_as_float(v[i]);
                if (at < limit) {
                    A.out_idx[pe.outoff + at] = x[i];
                    A.out_val[pe.outoff + at] = y;
                    if (index_ok(A, x[i])) {
                        if (OP == SEL_WORKER) store_scattered(&A.state[x[i]], A.m * y);
                        else if (OP == SEL_PULL) store_scattered(&A.state[x[i]], 0.0f);
                        else store_scattered(&A.state[x[i]], old[i] + y);
                    }
                }
                ++at;
            }
        };
#pragma unroll
        for (uint32_t h = 0; h < HELD; ++h)
            if (256u * h < n) emit(256u * h + 4u * lane, val[h], idx[h], was[h]);
#pragma unroll 1
        for (uint32_t q = 256u * HELD; q < n; q += 256u) {
            uint32_t v[4], x[4];
            float old[4];
            fetch(q + 4u * lane, v, x, old);
            emit(q + 4u * lane, v, x, old);
        }
    }
    // the last of the tensor's workgroups clears the key for the next launch
    if (tid == 0) {
        const uint32_t before = __hip_atomic_fetch_add(&st->chain_seen, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (before + 1u == runs) {
            st_dev(&st->key, make_uint2(0u, 0u));
            st_dev(&st->chain_seen, 0u);
        }
    }
}

// (What a workgroup begins with comes as arguments of its own, which are in registers then.)
template <int OP>
__global__ __launch_bounds__(SEL_THREADS) void k_step(const StepUnit *steptab, const SegDesc *ranktab, uint32_t *tau, const float *grad,
                                                      float *state, uint32_t *stepflag, uint32_t nstep, uint32_t nrank, float lr,
                                                      const SelectArgs rest)
{
    __shared__ PartShared P;
    __shared__ uint2 llist[SEL_LDS_LIST];
    SelectArgs A = rest;
    A.steptab = steptab;
    A.tau = tau;
    A.grad = grad;
    if (OP == SEL_PULL_V) A.model = grad;
    A.state = state;
    A.stepflag = stepflag;
    A.nstep = nstep;
    A.lr = lr;
    if (blockIdx.x < nstep) {
        const StepUnit u = steptab[blockIdx.x];
        if (u.n > SMALL_N) {
            step_collect<OP>(A, u, blockIdx.x, P);
        } else {
            if (threadIdx.x == 0) A.segstate[u.j].status = SEG_DONE;
            small_select<OP, true>(A, A.tdesc[u.j], A.plan[u.j], u.j, P.S);
        }
        return;
    }
    uint32_t b = blockIdx.x - nstep;
    if (b < nrank) {
        step_rank_block<OP>(A, ranktab[b], P, llist);
        return;
    }
    b -= nrank;
    const uint32_t nb = (A.nparts + A.bgroup - 1u) / A.bgroup, standby = (A.repair && A.multi) ? 2u * nb : 0u;
    if (b < standby) standby_block<OP, FORM_STEP>(A, b, nb, P, llist);
    else step_emit<OP>(A, A.emittab[b - standby], P);
}

}  // namespace dgs
