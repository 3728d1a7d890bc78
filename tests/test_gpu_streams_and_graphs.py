"""Launch modes around the same calls.  (1) One whole step (dgs_worker_step + dgs_server_push +
dgs_server_pull) captured into a HIP graph on the context's stream and replayed: every replay
must give what the oracle gives for that step, with eager work and synchronisations between the
replays; the calls enqueue kernels only (no memset or copy nodes, no host wait) once the plan of a
density is cached.  (2) Worker and server as two contexts on two streams, overlapping."""
import gc

import numpy as np
import pytest

from paper_1910_10929_amd import dgs, synth
from harness import assert_pairs_match, assert_state_match, to_host_u32

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_collection_while_capturing():
    """A collection inside a capture may find an earlier test's graph or context, and destroying one
    is not permitted then: a graph's destructor ends the process."""
    gc.collect()
    gc.disable()
    yield
    gc.enable()


def test_step_replayed_from_a_graph(oracle):
    import torch
    sizes = [300_000, 64, 9408, 70_001, 5]
    off = synth.offsets_from_sizes(sizes)
    n = int(off[-1])
    rho = 0.004
    lr, m = np.float32(0.5), np.float32(0.9)
    scales = synth.tensor_scales(len(sizes), 80)
    rng = np.random.default_rng(81)
    dev = "cuda:0"
    s = torch.cuda.Stream(device=dev)
    ctx = dgs.Context(off, W=1, device=dev, stream=s)
    K = ctx.nnz(rho)
    with torch.cuda.stream(s):
        g_static = torch.zeros(n, device=dev)
        state = torch.zeros(n, device=dev)
        model = torch.zeros(n, device=dev)
        diff = torch.zeros((1, n), device=dev)
        idx = torch.zeros(K, dtype=torch.int32, device=dev)
        val = torch.zeros(K, device=dev)
        pidx = torch.zeros(K, dtype=torch.int32, device=dev)
        pval = torch.zeros(K, device=dev)
    ctx.server_attach(diff)
    s_ref = np.zeros(n, np.float32)
    model_ref = np.zeros(n, np.float32)
    diff_ref = np.zeros((1, n), np.float32)

    def enqueue():
        ctx.worker_step(g_static, state, float(lr), float(m), rho, idx, val)
        ctx.server_push(model, 0, idx, val, K)
        ctx.server_pull(0, rho, pidx, pval)

    def check(tag, g):
        wi, wv = oracle.worker_step(g, s_ref, off, lr, m, rho)
        oracle.server_push(model_ref, diff_ref, wi, wv)
        pi, pv = oracle.server_pull(diff_ref, 0, off, rho)
        s.synchronize()
        assert_pairs_match(to_host_u32(idx), val.cpu().numpy(), wi, wv, f"{tag}: worker message")
        assert_pairs_match(to_host_u32(pidx), pval.cpu().numpy(), pi, pv, f"{tag}: pull message")
        assert_state_match(state.cpu().numpy(), s_ref, f"{tag}: worker state")
        assert_state_match(diff[0].cpu().numpy(), diff_ref[0], f"{tag}: difference row")

    grads = [synth.gaussian_grads(off, scales, rng) for _ in range(8)]
    with torch.cuda.stream(s):
        for t in range(2):                       # eager: the non-predicted first call, then a predicted one
            g_static.copy_(torch.from_numpy(grads[t]))
            enqueue()
            check(f"eager {t}", grads[t])
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            enqueue()
        for t in range(2, 8):
            g_static.copy_(torch.from_numpy(grads[t]))
            graph.replay()
            check(f"replay {t}", grads[t])
            (state.abs().sum() + model.sum()).item()          # eager work and a host wait in between
    assert_state_match(model.cpu().numpy(), model_ref, "model")
    st = ctx.stats()
    assert st.internal_errors == 0 and st.exact_calls == 2
    ctx.close()


@pytest.mark.parametrize("rho_up", [0.006, 0.002])
def test_pull_on_the_printed_state_replayed_from_a_graph(oracle, rho_up):
    """dgs_server_push_model + dgs_server_pull_sent of a server with two workers, captured where the row is updated
    by a launch of its own behind the selection (more than 1400 pairs in a tensor): every replay against
    the oracle, messages as dense as the pull and sparser ones."""
    import torch
    off = synth.offsets_from_sizes([300_001, 64, 9408, 70_001, 5])
    n, rho, W = int(off[-1]), 0.006, 2
    dev = "cuda:0"
    rng = np.random.default_rng(85)
    scales = synth.tensor_scales(5, 84)
    kj, K_up = oracle.nnz(off, rho_up)
    model_ref = synth.gaussian(n, rng)
    rows_ref = np.tile(model_ref, (W, 1))
    s = torch.cuda.Stream(device=dev)
    ctx = dgs.Context(off, W=W, device=dev, stream=s)
    K = ctx.nnz(rho)
    with torch.cuda.stream(s):
        model, rows = torch.from_numpy(model_ref.copy()).to(dev), torch.from_numpy(rows_ref.copy()).to(dev)
        idx, val = torch.zeros(K_up, dtype=torch.int32, device=dev), torch.zeros(K_up, device=dev)
        pidx, pval = torch.zeros(K, dtype=torch.int32, device=dev), torch.zeros(K, device=dev)
        ctx.server_attach_sent(rows)

        def enqueue(w):
            ctx.server_push_model(model, idx, val, K_up)
            ctx.server_pull_sent(model, w, rho, pidx, pval)

        def event(w, go, tag):
            i, v = synth.sparse_payload(off, kj, scales, rng)
            idx.copy_(torch.from_numpy(i.view(np.int32)))
            val.copy_(torch.from_numpy(v))
            go()
            oracle.server_push_model(model_ref, i, v)
            wi, wv = oracle.server_pull_sent(model_ref, rows_ref, w, off, rho)
            s.synchronize()
            assert_pairs_match(to_host_u32(pidx), pval.cpu().numpy(), wi, wv, tag)
            assert_state_match(rows.cpu().numpy().ravel(), rows_ref.ravel(), f"{tag}: rows")
            (rows.sum() + model.sum()).item()                 # eager work and a host wait in between

        graphs = []
        for w in range(W):
            for t in range(2):
                event(w, lambda: enqueue(w), f"eager {w} {t}")
            graphs.append(torch.cuda.CUDAGraph())
            with torch.cuda.graph(graphs[w], stream=s):
                enqueue(w)
        for t in range(8):
            event(t % W, graphs[t % W].replay, f"replay {t}")
    assert_state_match(model.cpu().numpy(), model_ref, "model")
    assert ctx.stats().internal_errors == 0
    ctx.close()


def test_an_unplanned_density_is_refused_during_capture(oracle):
    """Planning a density copies its tables to the device, which a stream capture must not contain:
    a call with a density that has no cached plan returns DGS_ENOTSUP while the stream is being
    captured, and nothing of it is recorded.  The plan that WAS used during a capture survives any
    number of other densities afterwards: the replay keeps giving the oracle's result."""
    import torch
    sizes = [200_000, 64, 9408]
    off = synth.offsets_from_sizes(sizes)
    n = int(off[-1])
    rho = 0.004
    lr, m = np.float32(1.0), np.float32(0.0)
    dev = "cuda:0"
    s = torch.cuda.Stream(device=dev)
    ctx = dgs.Context(off, W=0, device=dev, stream=s)
    K = ctx.nnz(rho)
    rng = np.random.default_rng(82)
    grads = [synth.gaussian(n, rng) for _ in range(4)]
    with torch.cuda.stream(s):
        g_static = torch.zeros(n, device=dev)
        state = torch.zeros(n, device=dev)
        idx = torch.zeros(2 * K, dtype=torch.int32, device=dev)
        val = torch.zeros(2 * K, device=dev)
        s_ref = np.zeros(n, np.float32)
        for t in range(2):
            g_static.copy_(torch.from_numpy(grads[t]))
            ctx.worker_step(g_static, state, float(lr), float(m), rho, idx, val, residual_mode=True)
            oracle.worker_step(grads[t], s_ref, off, lr, m, rho)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            with pytest.raises(dgs.DgsError) as e:
                ctx.worker_step(g_static, state, float(lr), float(m), 0.0071, idx, val, residual_mode=True)
            assert e.value.code == dgs.DGS_ENOTSUP
            ctx.worker_step(g_static, state, float(lr), float(m), rho, idx, val, residual_mode=True)
        # nine other densities, eagerly: more than the cache holds
        scratch = torch.zeros(n, device=dev)
        for i in range(9):
            ctx.worker_step(g_static, scratch, float(lr), float(m), 0.001 + 0.0005 * i, idx, val, residual_mode=True)
        for t in range(2, 4):
            g_static.copy_(torch.from_numpy(grads[t]))
            graph.replay()
            wi, wv = oracle.worker_step(grads[t], s_ref, off, lr, m, rho)
            s.synchronize()
            assert_pairs_match(to_host_u32(idx)[:K], val.cpu().numpy()[:K], wi, wv, f"replay {t}")
            assert_state_match(state.cpu().numpy(), s_ref, f"replay {t}: state")
    assert ctx.stats().internal_errors == 0
    ctx.close()


def test_the_pull_that_waits_for_its_count_is_refused_during_capture():
    """dgs_server_pull_all hands its count to the host; under capture nothing runs, so the call is
    refused, records nothing and leaves the next eager call its count."""
    import torch
    n, dev = 70_001, "cuda:0"
    s = torch.cuda.Stream(device=dev)
    with torch.cuda.stream(s):
        ctx = dgs.Context(synth.layout_flat(n), W=1, device=dev, stream=s)
        row = torch.zeros((1, n), device=dev)
        ctx.server_attach(row)
        idx, val = torch.zeros(n, dtype=torch.int32, device=dev), torch.zeros(n, device=dev)
        row[0, ::1000] = 1.0
        assert ctx.server_pull_all(0, idx, val, n) == 71
        row[0, ::7] = 2.0
        counter = torch.zeros(1, device=dev)
        graph = torch.cuda.CUDAGraph()
        code = None
        with torch.cuda.graph(graph, stream=s):
            counter += 1.0
            try:
                ctx.server_pull_all(0, idx, val, n)
            except dgs.DgsError as err:
                code = err.code
        assert code == dgs.DGS_ENOTSUP
        for _ in range(3):
            graph.replay()
        s.synchronize()
        assert counter.item() == 3.0 and int((row != 0).sum()) == (n + 6) // 7
        assert ctx.server_pull_all(0, idx, val, n) == (n + 6) // 7
        s.synchronize()
        assert not row.any()
    ctx.close()


def test_worker_and_server_on_two_streams(oracle):
    """Two contexts on two streams of default priority: the worker's step t+1 is enqueued while
    the server still handles push / pull t; messages are double-buffered and ordered with
    events.  Everything is compared at the end, after a single wait."""
    import torch
    sizes = [300_000, 64, 9408, 70_001, 5]
    off = synth.offsets_from_sizes(sizes)
    n = int(off[-1])
    rho = 0.004
    lr, m = np.float32(0.5), np.float32(0.9)
    scales = synth.tensor_scales(len(sizes), 82)
    rng = np.random.default_rng(83)
    dev = "cuda:0"
    sa, sb = torch.cuda.Stream(device=dev), torch.cuda.Stream(device=dev)
    wctx = dgs.Context(off, W=0, device=dev, stream=sa)
    sctx = dgs.Context(off, W=1, device=dev, stream=sb)
    K = wctx.nnz(rho)
    steps = 8
    grads = [synth.gaussian_grads(off, scales, rng) for _ in range(steps)]
    g_dev = [torch.from_numpy(g).to(dev) for g in grads]
    state = torch.zeros(n, device=dev)
    model = torch.zeros(n, device=dev)
    diff = torch.zeros((1, n), device=dev)
    sctx.server_attach(diff)
    msg = [(torch.zeros(K, dtype=torch.int32, device=dev), torch.zeros(K, device=dev)) for _ in range(2)]
    pidx = torch.zeros(K, dtype=torch.int32, device=dev)
    pval = torch.zeros(K, device=dev)
    sent_log = [(torch.zeros(K, dtype=torch.int32, device=dev), torch.zeros(K, device=dev)) for _ in range(steps)]
    pull_log = [(torch.zeros(K, dtype=torch.int32, device=dev), torch.zeros(K, device=dev)) for _ in range(steps)]
    produced = [torch.cuda.Event() for _ in range(2)]
    consumed = [torch.cuda.Event() for _ in range(2)]
    torch.cuda.synchronize()
    for t in range(steps):
        b = t % 2
        if t >= 2:
            sa.wait_event(consumed[b])
        wctx.worker_step(g_dev[t], state, float(lr), float(m), rho, msg[b][0], msg[b][1])
        produced[b].record(sa)
        sb.wait_event(produced[b])
        with torch.cuda.stream(sb):
            sent_log[t][0].copy_(msg[b][0])
            sent_log[t][1].copy_(msg[b][1])
        sctx.server_push(model, 0, msg[b][0], msg[b][1], K)
        consumed[b].record(sb)
        sctx.server_pull(0, rho, pidx, pval)
        with torch.cuda.stream(sb):
            pull_log[t][0].copy_(pidx)
            pull_log[t][1].copy_(pval)
    torch.cuda.synchronize()
    s_ref = np.zeros(n, np.float32)
    model_ref = np.zeros(n, np.float32)
    diff_ref = np.zeros((1, n), np.float32)
    for t in range(steps):
        wi, wv = oracle.worker_step(grads[t], s_ref, off, lr, m, rho)
        oracle.server_push(model_ref, diff_ref, wi, wv)
        pi, pv = oracle.server_pull(diff_ref, 0, off, rho)
        assert_pairs_match(to_host_u32(sent_log[t][0]), sent_log[t][1].cpu().numpy(), wi, wv, f"step {t}: worker message")
        assert_pairs_match(to_host_u32(pull_log[t][0]), pull_log[t][1].cpu().numpy(), pi, pv, f"step {t}: pull message")
    assert_state_match(state.cpu().numpy(), s_ref, "worker state")
    assert_state_match(model.cpu().numpy(), model_ref, "model")
    assert_state_match(diff[0].cpu().numpy(), diff_ref[0], "difference row")
    assert wctx.stats().internal_errors == 0 and sctx.stats().internal_errors == 0
    wctx.close()
    sctx.close()
