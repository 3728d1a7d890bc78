"""Dense requests on layouts without a tensor of 65,536 elements, where one workgroup selects each tensor from LDS (up
to 32,768 elements) or from the buffers: sizes around one and several turns of the emission (1024 threads with 3 or 4
entries each) and around that limit; distinct values, ties, more zeros than the rest; as worker step and as pull
in both server forms.  Bit for bit against the oracle: each value is the result of one correctly rounded operation."""
import numpy as np
import pytest

from paper_1910_10929_amd import dgs, synth
from harness import Server, assert_pairs_match, assert_state_match, run_worker_parity, to_dev, to_host_u32

pytestmark = pytest.mark.gpu

SIZES = [3071, 3072, 3073, 4095, 4096, 4097, 5, 9216, 12289, 20000, 32767, 32768, 32769, 60001, 1]


def gradients(kind, n, seed, count=3):
    rng = np.random.default_rng(seed)
    for _ in range(count):
        g = rng.standard_normal(n).astype(np.float32)
        if kind == "levels":
            g = np.round(g).astype(np.float32)
        elif kind == "sparse":
            g[rng.random(n) < 0.8] = 0.0
        yield g


@pytest.mark.parametrize("kind", ["gauss", "levels", "sparse"])
@pytest.mark.parametrize("rho", [0.05, 0.5])
def test_worker(oracle, kind, rho):
    off = synth.offsets_from_sizes(SIZES)
    st = run_worker_parity(oracle, off, list(gradients(kind, int(off[-1]), 3)), np.float32(0.5), np.float32(0.9), rho)
    assert st.internal_errors == 0


@pytest.mark.parametrize("form", ["diff", "sent"])
@pytest.mark.parametrize("kind", ["gauss", "levels", "sparse"])
def test_pull(oracle, kind, form):
    import torch
    off = synth.offsets_from_sizes(SIZES)
    n, rho = int(off[-1]), 0.3
    ctx = dgs.Context(off, W=1)
    model = np.random.default_rng(4).standard_normal(n).astype(np.float32)
    rows = np.zeros((1, n), np.float32) if form == "diff" else model[None].copy()
    srv = Server(ctx, model, density_max=rho)
    dev_rows = srv.diff
    if form == "sent":
        dev_rows = to_dev(rows)
        ctx.server_attach_sent(dev_rows)
    for t, g in enumerate(gradients(kind, n, 5)):
        idx = np.flatnonzero(g).astype(np.uint32)
        di, dv = to_dev(idx), to_dev(g[idx])
        if form == "diff":
            ctx.server_push(srv.model, 0, di, dv, idx.size)
            oracle.server_push(model, rows, idx, g[idx])
            wi, wv = oracle.server_pull(rows, 0, off, rho)
            ctx.server_pull(0, rho, srv.idx, srv.val)
        else:
            ctx.server_push_model(srv.model, di, dv, idx.size)
            oracle.server_push_model(model, idx, g[idx])
            wi, wv = oracle.server_pull_sent(model, rows, 0, off, rho)
            ctx.server_pull_sent(srv.model, 0, rho, srv.idx, srv.val)
        torch.cuda.synchronize()
        assert_pairs_match(to_host_u32(srv.idx), srv.val.cpu().numpy(), wi, wv, f"pull {t}")
        assert_state_match(dev_rows.cpu().numpy(), rows, f"rows {t}")
    assert ctx.stats().internal_errors == 0
    ctx.close()
