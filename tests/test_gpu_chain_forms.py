"""The two forms of the chain: as roles of the selection's launch (up to 512 slabs of 128 tiles, 1024 of a single tensor) and
as launches of its own.  The same tensors go through both -- behind them, for the second form, lie enough others of one slab
each -- with distinct values, ties, crowded tiles, predictions that fail (with and without the workgroups that
collect again) and fewer nonzeros than k, as worker step and as pull in both server forms.  Then plans on either side of
the lines between the forms and between one workgroup's selection and the chain; replays from a captured graph; two contexts on two
streams.  Bit for bit against the oracle, or against the single-workgroup selection where the oracle would take minutes."""
import gc

import numpy as np
import pytest

from paper_1910_10929_amd import dgs, synth
from harness import assert_pairs_match, assert_state_match, to_host_u32

pytestmark = pytest.mark.gpu

FRONT = [9001, 70_001, 131_072, 262_144 + 128 * 1024 + 1, 64]
OTHERS = 520                     # tensors of one slab


@pytest.fixture(autouse=True)
def no_collection_while_capturing():
    gc.collect()
    gc.disable()
    yield
    gc.enable()


def contents(kind, n, rng, count):
    """Values of the tensors that are compared, call after call."""
    for t in range(count):
        v = rng.standard_normal(n).astype(np.float32)
        if kind == "ties":
            v = (np.round(v * 4) / 4).astype(np.float32)
        elif kind == "crowded":
            for tile in (9, 20, 63, 64, 127, 128, 129, 200, 201, 202, 203, 400):      # up to 250 entries of a tile far above the rest
                v[tile * 1024 + rng.choice(1024, int(rng.integers(60, 250)), replace=False)] *= np.float32(40.0)
        elif kind == "side by side":        # 60 winners in each of four tiles, no tile beyond 64 candidates
            at = np.arange(n)
            tile, run = at // 1024, (at // 1024) % 16
            few = (at * 619 + tile) % 1024 < np.where((run >= 8) & (run < 12), 60, 20)
            v = np.where(few, np.sign(v) * np.where((run >= 8) & (run < 12), 20, 1) * (1 + np.abs(v) / 8), 0).astype(np.float32)
        elif kind == "jumps":
            v *= np.float32([1.0, 1.0, 1e-6, 1e3, 1.0, 1e-6][t % 6])
        elif kind == "zeros":
            v[rng.random(n) < 0.9995] = 0.0
        yield v


def run_calls(oracle, op, kind, form, repair, rho=0.01, calls=6):
    import torch
    sizes = FRONT + ([65_536] * OTHERS if form == "separate" else [])
    off, front = synth.offsets_from_sizes(sizes), synth.offsets_from_sizes(FRONT)
    n, nf = int(off[-1]), int(front[-1])
    rng = np.random.default_rng(91)
    dev = "cuda:0"
    ctx = dgs.Context(off, W=0 if op == "worker" else 1)
    ctx.set_option(dgs.OPT_SEGMENTED, dgs.SEG_ALWAYS)
    ctx.set_option(dgs.OPT_REPAIR_ROUND, repair)
    ctx.set_option(dgs.OPT_PROFILE, 1)
    K, Kf = ctx.nnz(rho), int(sum(np.ceil(rho * s) for s in FRONT))
    idx, val = torch.zeros(K, dtype=torch.int32, device=dev), torch.zeros(K, device=dev)
    row = torch.zeros((1, n), device=dev)
    given = torch.randn(n, device=dev, generator=torch.Generator(device=dev).manual_seed(6))
    if op != "worker":
        (ctx.server_attach if op == "diff" else ctx.server_attach_sent)(row)
    ref = np.zeros((1, nf), np.float32)
    for t, v in enumerate(contents(kind, nf, rng, calls)):
        given[:nf].copy_(torch.from_numpy(v))
        if op == "worker":
            wi, wv = oracle.worker_step(v, ref[0], front, np.float32(1.0), np.float32(0.0), rho)
            ctx.worker_step(given, row[0], 1.0, 0.0, rho, idx, val, residual_mode=True)
        elif op == "diff":
            ref[0] += v
            row[0] += given
            wi, wv = oracle.server_pull(ref, 0, front, rho)
            ctx.server_pull(0, rho, idx, val)
        else:
            wi, wv = oracle.server_pull_sent(v, ref, 0, front, rho)
            ctx.server_pull_sent(given, 0, rho, idx, val)
        torch.cuda.synchronize()
        assert_pairs_match(to_host_u32(idx)[:Kf], val.cpu().numpy()[:Kf], wi, wv, f"call {t}")
        assert_state_match(row[0, :nf].cpu().numpy(), ref[0], f"state {t}")
    launches = ctx.profile_read(dgs.PROF_WORKER_SEGMENTED if op == "worker" else dgs.PROF_PULL_SEGMENTED)[0]
    st = ctx.stats()
    ctx.close()
    assert st.internal_errors == 0 and st.segmented_tensors > 0
    assert launches == (calls if form == "separate" else 0)
    return st


@pytest.mark.parametrize("form", ["in-launch", "separate"])
@pytest.mark.parametrize("kind", ["gaussian", "ties", "crowded", "side by side", "zeros"])
@pytest.mark.parametrize("op", ["worker", "diff", "sent"])
def test_both_forms(oracle, op, kind, form):
    run_calls(oracle, op, kind, form, 1)


@pytest.mark.parametrize("form", ["in-launch", "separate"])
@pytest.mark.parametrize("repair", [1, 0], ids=["roles", "no-roles"])
@pytest.mark.parametrize("op", ["worker", "diff", "sent"])
def test_failed_predictions(oracle, op, repair, form):
    st = run_calls(oracle, op, "jumps", form, repair, rho=0.004, calls=8)
    assert (st.repaired_tensors if repair else st.fallback_tensors) >= 2


@pytest.mark.parametrize("form", ["in-launch", "separate"])
@pytest.mark.parametrize("op", ["worker", "diff", "sent"])
def test_missed_windows(oracle, op, form):
    """Values that double from call to call on a fresh row: the k-th key lies more than an octave above the hinted threshold, but
    no tile overflows.  In the selection's launch the candidates are counted again; without the re-collecting workgroups nothing
    but the slow selection from the buffers could resolve such a tensor otherwise, and that must stay unused there."""
    import torch
    off = synth.offsets_from_sizes(FRONT + ([65_536] * OTHERS if form == "separate" else []))
    front, rho, dev = synth.offsets_from_sizes(FRONT), 0.001, "cuda:0"
    n, nf, Kf = int(off[-1]), int(front[-1]), int(sum(np.ceil(rho * s) for s in FRONT))
    ctx = dgs.Context(off, W=0 if op == "worker" else 1)
    ctx.set_option(dgs.OPT_SEGMENTED, dgs.SEG_ALWAYS)
    ctx.set_option(dgs.OPT_REPAIR_ROUND, 0)
    K = ctx.nnz(rho)
    idx, val = torch.zeros(K, dtype=torch.int32, device=dev), torch.zeros(K, device=dev)
    row = torch.zeros((1, n), device=dev)
    others = torch.randn(n, device=dev, generator=torch.Generator(device=dev).manual_seed(8))
    if op != "worker":
        (ctx.server_attach if op == "diff" else ctx.server_attach_sent)(row)
    rng = np.random.default_rng(94)
    for t, scale in enumerate([1, 1, 2, 4, 8]):
        v = (rng.standard_normal(nf) * scale).astype(np.float32)
        given = others.clone()
        given[:nf].copy_(torch.from_numpy(v))
        ref = np.zeros((1, nf), np.float32)
        row.zero_()
        if op == "worker":
            wi, wv = oracle.worker_step(v, ref[0], front, np.float32(1.0), np.float32(0.0), rho)
            ctx.worker_step(given, row[0], 1.0, 0.0, rho, idx, val, residual_mode=True)
        elif op == "diff":
            ref[0] = v
            row[0] = given
            wi, wv = oracle.server_pull(ref, 0, front, rho)
            ctx.server_pull(0, rho, idx, val)
        else:
            wi, wv = oracle.server_pull_sent(v, ref, 0, front, rho)
            ctx.server_pull_sent(given, 0, rho, idx, val)
        torch.cuda.synchronize()
        assert_pairs_match(to_host_u32(idx)[:Kf], val.cpu().numpy()[:Kf], wi, wv, f"call {t}")
        assert_state_match(row[0, :nf].cpu().numpy(), ref[0], f"state {t}")
    st = ctx.stats()
    assert st.internal_errors == 0
    if form == "in-launch":
        assert st.repaired_tensors >= 2 and st.fallback_tensors == 0
    ctx.close()


SLABS256 = 256 * 128 * 1024      # elements of 256 full slabs


@pytest.mark.parametrize("op", ["worker", "sent"])
@pytest.mark.parametrize("sizes,in_launch", [([SLABS256, SLABS256], True), ([SLABS256, SLABS256 + 1], False),
                                             ([4 * SLABS256], True), ([4 * SLABS256 + 1], False)],
                         ids=["512", "513", "one-1024", "one-1025"])
def test_either_side_of_the_line_between_the_forms(op, sizes, in_launch):
    import torch
    off = synth.offsets_from_sizes(sizes)
    n, rho, dev = int(off[-1]), 1e-3, "cuda:0"
    outs = []
    for mode in (dgs.SEG_ALWAYS, dgs.SEG_NEVER):
        gen = torch.Generator(device=dev).manual_seed(7)
        ctx = dgs.Context(off, W=0 if op == "worker" else 1)
        ctx.set_option(dgs.OPT_SEGMENTED, mode)
        ctx.set_option(dgs.OPT_PROFILE, 1)
        K = ctx.nnz(rho)
        idx, val = torch.zeros(K, dtype=torch.int32, device=dev), torch.zeros(K, device=dev)
        row, given = torch.randn((1, n), device=dev, generator=gen), torch.randn(n, device=dev, generator=gen)
        if op == "sent":
            ctx.server_attach_sent(row)
        run = []
        for _ in range(3):
            if op == "worker":
                ctx.worker_step(given, row[0], 0.1, 0.5, rho, idx, val)
            else:
                ctx.server_pull_sent(given, 0, rho, idx, val)
            run += [idx.clone(), val.view(torch.int32).clone()]
        run.append(row.view(torch.int32).clone())
        launches = ctx.profile_read(dgs.PROF_WORKER_SEGMENTED if op == "worker" else dgs.PROF_PULL_SEGMENTED)[0]
        st = ctx.stats()
        assert st.internal_errors == 0 and (st.segmented_tensors > 0) == (mode == dgs.SEG_ALWAYS)
        assert launches == (0 if in_launch or mode == dgs.SEG_NEVER else 3)
        ctx.close()
        outs.append(run)
    for a, b in zip(*outs):
        assert torch.equal(a, b)


# tiles, k, does the tensor take the chain: lists planned for 2 k + 4 floor(sqrt k) + 16 entries, beyond 10,240 on
# 512 to 3583 tiles, beyond 20,480 otherwise
@pytest.mark.parametrize("tiles,k,chain", [(512, 4972, False), (512, 4973, True), (511, 4973, False), (511, 10032, False),
                                           (511, 10033, True), (3583, 4973, True), (3584, 4973, False),
                                           (3584, 10032, False), (3584, 10033, True)])
def test_either_side_of_the_line_to_the_chain(oracle, tiles, k, chain, launches):
    import torch
    n = tiles * 1024
    off, rho, dev = synth.offsets_from_sizes([n]), (k - 0.5) / n, "cuda:0"
    ctx = dgs.Context(off, W=1)
    assert ctx.nnz(rho) == k
    row, given = torch.zeros((1, n), device=dev), torch.zeros(n, device=dev)
    idx, val = torch.zeros(k, dtype=torch.int32, device=dev), torch.zeros(k, device=dev)
    ctx.server_attach_sent(row)
    ref = np.zeros((1, n), np.float32)
    rng = np.random.default_rng(92)
    for t in range(3):
        v = rng.standard_normal(n).astype(np.float32)
        given.copy_(torch.from_numpy(v))
        wi, wv = oracle.server_pull_sent(v, ref, 0, off, rho)
        ctx.server_pull_sent(given, 0, rho, idx, val)
        torch.cuda.synchronize()
        assert_pairs_match(to_host_u32(idx), val.cpu().numpy(), wi, wv, f"call {t}")
        assert_state_match(row[0].cpu().numpy(), ref[0], f"row {t}")
    st = ctx.stats()
    # (where later calls are one launch, the first has been on the chain, and all of them where the plan's lists are too long for that)
    on_chain = {3} if launches == "several_launches" else {1, 3}
    assert st.internal_errors == 0 and st.segmented_tensors in (on_chain if chain else {0})
    ctx.close()


def test_in_launch_chain_replayed_from_a_graph(oracle, launches):
    """Worker step and pull with the chain in the selection's launch, captured once; the scale of the gradients collapses and
    returns between replays, so that some replays collect tensors again.  And the same as one launch each."""
    import torch
    off = synth.offsets_from_sizes([900_001, 64, 70_001, 9408])
    n, rho, dev = int(off[-1]), 0.007, "cuda:0"      # (lists planned for 12.9 K entries: on the chain, and within the line of one launch)
    s = torch.cuda.Stream(device=dev)
    ctx = dgs.Context(off, W=1, device=dev, stream=s)
    K = ctx.nnz(rho)
    ref_state, ref_model, ref_rows = np.zeros(n, np.float32), np.zeros(n, np.float32), np.zeros((1, n), np.float32)
    rng = np.random.default_rng(93)
    with torch.cuda.stream(s):
        g, state, model = (torch.zeros(n, device=dev) for _ in range(3))
        rows = torch.zeros((1, n), device=dev)
        idx, pidx = (torch.zeros(K, dtype=torch.int32, device=dev) for _ in range(2))
        val, pval = (torch.zeros(K, device=dev) for _ in range(2))
        ctx.server_attach(rows)

        def enqueue():
            ctx.worker_step(g, state, 1.0, 0.0, rho, idx, val, residual_mode=True)
            ctx.server_push(model, 0, idx, val, K)
            ctx.server_pull(0, rho, pidx, pval)

        graph = None
        for t, scale in enumerate([1, 1, 1, 1e-6, 1, 1e3, 1e3, 1e-3, 1]):
            v = (rng.standard_normal(n) * scale).astype(np.float32)
            if scale == 1e-6:
                state.zero_()
                ref_state[:] = 0
            g.copy_(torch.from_numpy(v))
            if t < 2:
                enqueue()
            else:
                if graph is None:
                    s.synchronize()
                    eager = ctx.stats().segmented_tensors
                    graph = torch.cuda.CUDAGraph()
                    with torch.cuda.graph(graph, stream=s):
                        enqueue()
                graph.replay()
            wi, wv = oracle.worker_step(v, ref_state, off, np.float32(1.0), np.float32(0.0), rho)
            oracle.server_push(ref_model, ref_rows, wi, wv)
            pi, pv = oracle.server_pull(ref_rows, 0, off, rho)
            s.synchronize()
            assert_pairs_match(to_host_u32(idx), val.cpu().numpy(), wi, wv, f"worker {t}")
            assert_pairs_match(to_host_u32(pidx), pval.cpu().numpy(), pi, pv, f"pull {t}")
            assert_state_match(state.cpu().numpy(), ref_state, f"state {t}")
            assert_state_match(rows[0].cpu().numpy(), ref_rows[0], f"row {t}")
            (state.abs().sum() + model.sum()).item()          # eager work and a host wait in between
    st = ctx.stats()
    assert st.internal_errors == 0 and st.repaired_tensors >= 1
    # a step and a pull in each of seven replays (the chain counts a tensor that it resolves, also after it was collected again)
    assert st.segmented_tensors - eager == (14 if launches == "several_launches" else 0)
    ctx.close()


def test_two_contexts_on_two_streams():
    """Two contexts whose selections each fill the chip with the chain's workgroups, running side by side on two streams: each
    gives what it gives alone."""
    import torch
    dev, rho, steps = "cuda:0", 0.01, 40
    offs = [synth.offsets_from_sizes([1 << 20] * 40), synth.offsets_from_sizes([700_001, 1_300_003] * 16)]
    grads = [[torch.randn(int(off[-1]), device=dev, generator=torch.Generator(device=dev).manual_seed(10 * i + t)) for t in range(3)]
             for i, off in enumerate(offs)]

    def contexts():
        out = []
        for off in offs:
            s = torch.cuda.Stream(device=dev)
            ctx = dgs.Context(off, W=0, device=dev, stream=s)
            K = ctx.nnz(rho)
            out.append((ctx, s, torch.zeros(int(off[-1]), device=dev), torch.zeros((steps, K), dtype=torch.int32, device=dev),
                        torch.zeros((steps, K), device=dev)))
        torch.cuda.synchronize()
        return out

    def step(c, i, t):
        ctx, s, state, idx, val = c[i]
        with torch.cuda.stream(s):
            ctx.worker_step(grads[i][t % 3], state, 1.0, 0.0, rho, idx[t], val[t], residual_mode=True)

    alone, beside = contexts(), contexts()
    for i in range(2):
        for t in range(steps):
            step(alone, i, t)
        torch.cuda.synchronize()
    for t in range(steps):
        for i in range(2):
            step(beside, i, t)
    torch.cuda.synchronize()
    for a, b in zip(alone, beside):
        assert a[0].stats().segmented_tensors > 0
        for c in (a, b):
            assert c[0].stats().internal_errors == 0
        for x, y in zip(a[2:], b[2:]):
            assert torch.equal(x.view(torch.int32), y.view(torch.int32))
        a[0].close()
        b[0].close()


@pytest.mark.parametrize("tensors,chain", [(80, True), (81, False)])
def test_the_chain_gives_way_to_many_tensors(tensors, chain):
    """Tensors of 512 tiles (4 slabs) with lists planned for 10,242 entries: the chain while there are 32 of them to a slab, one
    workgroup per tensor from 321 slabs on."""
    import torch
    off, dev = synth.offsets_from_sizes([512 * 1024] * tensors), "cuda:0"
    n, rho = int(off[-1]), (4973 - 0.5) / (512 * 1024)
    outs = []
    for mode in (dgs.SEG_AUTO, dgs.SEG_NEVER):
        gen = torch.Generator(device=dev).manual_seed(12)
        ctx = dgs.Context(off, W=0)
        ctx.set_option(dgs.OPT_SEGMENTED, mode)
        K = ctx.nnz(rho)
        idx, val = torch.zeros(K, dtype=torch.int32, device=dev), torch.zeros(K, device=dev)
        state, grad = torch.zeros(n, device=dev), torch.randn(n, device=dev, generator=gen)
        run = []
        for _ in range(3):
            ctx.worker_step(grad, state, 1.0, 0.0, rho, idx, val, residual_mode=True)
            run += [idx.clone(), val.view(torch.int32).clone()]
        run.append(state.view(torch.int32).clone())
        st = ctx.stats()
        assert st.internal_errors == 0
        assert st.segmented_tensors == (3 * tensors if chain and mode == dgs.SEG_AUTO else 0)
        ctx.close()
        outs.append(run)
    for a, b in zip(*outs):
        assert torch.equal(a, b)
