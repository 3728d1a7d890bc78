// Streaming pass of libdgs: one wavefront per 1024-element tile, 16-byte loads, fused
// accumulate + magnitude key + candidate collection or key histogram.  And the launch of a whole call (dgs_step.h).
#include "dgs_step.h"
#include "dgs_tile.h"

namespace dgs {

// What a wavefront needs first comes as arguments of its own, which are in registers when it starts; a struct has to be fetched
// before its fields can be used.  With that here, in k_select and in the small kernels: a round on nine small tensors 40.9 -> 39.8 us, on
// ResNet-50 shapes 127.5 -> 122.8, an event of a server with 32 sent rows 62.5 -> 61.2.
template <int OP, int MODE>
__global__ __launch_bounds__(STREAM_THREADS) void k_stream(const float *grad, float *state,
                                                           const uint32_t *__restrict__ toff,
                                                           const uint32_t *__restrict__ tau, uint32_t n, uint32_t J,
                                                           uint32_t quads_per_block, uint32_t nquads, float lr,
                                                           const StreamArgs rest)
{
    StreamArgs A = rest;
    A.grad = grad;
    A.state = state;
    A.n = n;
    A.J = J;
    A.quads_per_block = quads_per_block;
    A.nquads = nquads;
    A.lr = lr;
    constexpr bool HISTO = (MODE == MODE_HIST || MODE == MODE_SAMPLE);
    __shared__ uint32_t lhist[HISTO ? HBINS : 1];
    constexpr uint32_t ROOM = MODE == MODE_COLLECT ? STAGE : (MODE == MODE_HIST ? TKEYS_STAGE / 2 : 0);      // of a wavefront
    __shared__ uint2 stage_all[ROOM ? WAVES_PER_BLOCK * ROOM : 1];
    const uint32_t wave = uniform(threadIdx.x >> 6);
    uint2 *stage = stage_all + wave * ROOM;
    const uint32_t q0 = blockIdx.x * A.quads_per_block;
    const uint32_t q1 = min(q0 + A.quads_per_block, A.nquads);
    int cur = -1;
    if (HISTO) {
        for (uint32_t b = threadIdx.x; b < HBINS; b += STREAM_THREADS) lhist[b] = 0;
        __syncthreads();
    }
    for (uint32_t q = q0; q < q1; ++q) {
        // (a sampling pass takes its tiles from a list, four at a time: "quad" q = entries 4 q ..)
        const uint32_t t = (MODE == MODE_SAMPLE)
                               ? ((q * WAVES_PER_BLOCK + wave < A.nlist) ? A.tile_list[q * WAVES_PER_BLOCK + wave] : 0xFFFFFFFFu)
                               : q * WAVES_PER_BLOCK + wave;
        if (HISTO) {
            // the LDS histogram belongs to the big tensor the quad starts in
            const uint32_t qfirst = ((MODE == MODE_SAMPLE) ? A.tile_list[q * WAVES_PER_BLOCK] : q * WAVES_PER_BLOCK) * TILE;
            const uint32_t fx = span_desc(toff, A.J, qfirst, qfirst).x;
            const int qt = (fx >> 31) ? (int)(fx & 0x7FFFFFFFu) : -1;
            if (qt != cur) {
                flush_hist<MODE>(lhist, A.ghist, cur);
                cur = qt;
            }
        }
        if (t < A.ntiles) process_tile<OP, MODE>(A, toff, tau, t, lhist, cur, stage);
    }
    flush_hist<MODE>(lhist, A.ghist, cur);
}

template <int OP, int MODE>
static void launch_stream_t(const StreamArgs &a, uint32_t blocks, hipStream_t st, void *ev0, void *ev1)
{
    launch_k(k_stream<OP, MODE>, dim3(blocks), dim3(STREAM_THREADS), st, ev0, ev1, a.grad, a.state, a.toff, a.tau, a.n, a.J,
             a.quads_per_block, a.nquads, a.lr, a);
}

void launch_stream(int op, int mode, const StreamArgs &a, uint32_t blocks, void *stream, void *ev0, void *ev1)
{
    hipStream_t st = (hipStream_t)stream;
    if (blocks == 0) return;
    if (op == OP_FMA) {
        if (mode == MODE_PLAIN) launch_stream_t<OP_FMA, MODE_PLAIN>(a, blocks, st, ev0, ev1);
        else if (mode == MODE_COLLECT) launch_stream_t<OP_FMA, MODE_COLLECT>(a, blocks, st, ev0, ev1);
        else if (mode == MODE_SAMPLE) launch_stream_t<OP_FMA, MODE_SAMPLE>(a, blocks, st, ev0, ev1);
        else launch_stream_t<OP_FMA, MODE_HIST>(a, blocks, st, ev0, ev1);
    } else if (op == OP_SUB) {
        if (mode == MODE_COLLECT) launch_stream_t<OP_SUB, MODE_COLLECT>(a, blocks, st, ev0, ev1);
        else if (mode == MODE_HIST) launch_stream_t<OP_SUB, MODE_HIST>(a, blocks, st, ev0, ev1);
        else if (mode == MODE_SAMPLE) launch_stream_t<OP_SUB, MODE_SAMPLE>(a, blocks, st, ev0, ev1);
    } else {
        if (mode == MODE_COLLECT) launch_stream_t<OP_IDENT, MODE_COLLECT>(a, blocks, st, ev0, ev1);
        else if (mode == MODE_HIST) launch_stream_t<OP_IDENT, MODE_HIST>(a, blocks, st, ev0, ev1);
        else if (mode == MODE_SAMPLE) launch_stream_t<OP_IDENT, MODE_SAMPLE>(a, blocks, st, ev0, ev1);
    }
}

template <int OP>
static void launch_step_t(const SelectArgs &a, uint32_t blocks, hipStream_t st, void *ev0, void *ev1)
{
    launch_k(k_step<OP>, dim3(blocks), dim3(SEL_THREADS), st, ev0, ev1, a.steptab, a.ranktab, a.tau,
             OP == SEL_PULL_V ? a.model : a.grad, a.state, a.stepflag, a.nstep, a.nrank, a.lr, a);
}

void launch_step(int op, const SelectArgs &a, void *stream, void *ev0, void *ev1)
{
    hipStream_t st = (hipStream_t)stream;
    const uint32_t nb = (a.nparts + a.bgroup - 1) / a.bgroup;
    const uint32_t blocks = a.nstep + a.nrank + (a.repair && a.multi ? 2u * nb : 0u) + a.nemit;
    if (op == SEL_WORKER) launch_step_t<SEL_WORKER>(a, blocks, st, ev0, ev1);
    else if (op == SEL_PULL) launch_step_t<SEL_PULL>(a, blocks, st, ev0, ev1);
    else launch_step_t<SEL_PULL_V>(a, blocks, st, ev0, ev1);
}

}  // namespace dgs
