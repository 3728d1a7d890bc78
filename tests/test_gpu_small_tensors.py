"""Small tensors (up to 8192 elements, 8 per thread): one element, counts around a thread's 8 and the
workgroup's 1024 threads, the largest, at unaligned offsets; k-th keys that stay near the previous one, that
jump out of its window and back, ties, fewer nonzeros than k; as worker step and as pull in both server forms.
Bit for bit against the oracle: each value is the result of one correctly rounded operation."""
import numpy as np
import pytest

from paper_1910_10929_amd import dgs, synth
from harness import Server, assert_pairs_match, assert_state_match, run_worker_parity, to_dev, to_host_u32

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("launches")]

SIZES = [1, 7, 8, 9, 1023, 1025, 4097, 8191, 8192, 20000, 3]
SCALES = [1.0, 1.0, 1.1, 30.0, 30.0, 0.02, 1.0, 0.0, 1.0]


def gradients(kind, n, seed):
    rng = np.random.default_rng(seed)
    for s in SCALES:
        g = rng.standard_normal(n).astype(np.float32)
        if kind == "levels":
            g = np.round(g).astype(np.float32)           # ties at every k-th key, zeros among them
        elif kind == "sparse":
            g[rng.random(n) < 0.97] = 0.0                # fewer nonzeros than k in some tensors
        yield (g * np.float32(s)).astype(np.float32)


@pytest.mark.parametrize("kind", ["gauss", "levels", "sparse"])
@pytest.mark.parametrize("rho", [0.002, 0.03])
def test_worker(oracle, kind, rho):
    off = synth.offsets_from_sizes(SIZES)
    for m in (0.9, 0.0):
        run_worker_parity(oracle, off, list(gradients(kind, int(off[-1]), 7)), np.float32(0.5), np.float32(m), rho,
                          misalign=1)


@pytest.mark.parametrize("kind", ["gauss", "levels", "sparse"])
@pytest.mark.parametrize("form", ["diff", "sent"])
def test_pull(oracle, kind, form):
    import torch
    off = synth.offsets_from_sizes(SIZES)
    n, rho, W = int(off[-1]), 0.02, 2
    ctx = dgs.Context(off, W=W)
    model = np.random.default_rng(3).standard_normal(n).astype(np.float32)
    rows = np.zeros((W, n), np.float32) if form == "diff" else np.repeat(model[None], W, 0)
    srv = Server(ctx, model, density_max=rho)
    dev_rows = srv.diff
    if form == "sent":
        dev_rows = to_dev(rows)
        ctx.server_attach_sent(dev_rows)
    for t, g in enumerate(gradients(kind, n, 11)):
        idx = np.flatnonzero(g).astype(np.uint32)
        val = g[idx]
        w = t % W
        di, dv = to_dev(idx), to_dev(val)
        if form == "diff":
            ctx.server_push(srv.model, w, di, dv, idx.size)
            oracle.server_push(model, rows, idx, val)
            wi, wv = oracle.server_pull(rows, w, off, rho)
            ctx.server_pull(w, rho, srv.idx, srv.val)
        else:
            ctx.server_push_model(srv.model, di, dv, idx.size)
            oracle.server_push_model(model, idx, val)
            wi, wv = oracle.server_pull_sent(model, rows, w, off, rho)
            ctx.server_pull_sent(srv.model, w, rho, srv.idx, srv.val)
        torch.cuda.synchronize()
        assert_pairs_match(to_host_u32(srv.idx), srv.val.cpu().numpy(), wi, wv, f"pull {t}")
        assert_state_match(dev_rows.cpu().numpy(), rows, f"rows {t}")
    assert ctx.stats().internal_errors == 0
    ctx.close()
