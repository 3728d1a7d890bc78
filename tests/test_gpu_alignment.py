"""Buffers at every 4-byte alignment take the 16-byte loads and stores of the full tiles: worker
state and gradient at offsets 1 to 3, server rows that start at odd addresses (odd n, three
workers), on the predicted, sampled, two-pass and dense paths.  Bit for bit against the oracle."""
import numpy as np
import pytest

from paper_1910_10929_amd import dgs, synth
from harness import assert_pairs_match, assert_state_match, run_worker_parity, to_host_u32

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("launches")]
SIZES = [70_001, 3, 8193, 1023, 20_000, 6]       # odd total; tiles shared by two and more tensors


@pytest.mark.parametrize("rho,force", [(0.004, False), (0.004, 1), (0.004, 2), (0.2, False)])
@pytest.mark.parametrize("misalign", [1, 2, 3])
def test_worker_at_any_alignment(oracle, misalign, rho, force):
    off = synth.offsets_from_sizes(SIZES)
    rng = np.random.default_rng(71)
    grads = [synth.gaussian(int(off[-1]), rng) for _ in range(3)]
    run_worker_parity(oracle, off, grads, np.float32(0.5), np.float32(0.9), rho, misalign=misalign, force_exact=force)


@pytest.mark.parametrize("rho", [0.004, 0.2])
def test_server_rows_at_odd_addresses(oracle, rho):
    import torch
    off = synth.offsets_from_sizes(SIZES)
    n, W = int(off[-1]), 3
    rng = np.random.default_rng(72)
    ctx, ctx_sent = dgs.Context(off, W=W), dgs.Context(off, W=W)
    model = torch.zeros(n, dtype=torch.float32, device="cuda:0")
    diff, sent = torch.zeros((W, n), device="cuda:0"), torch.zeros((W, n), device="cuda:0")
    ctx.server_attach(diff)
    ctx_sent.server_attach_sent(sent)
    idx = torch.zeros(ctx.nnz(rho), dtype=torch.int32, device="cuda:0")
    val = torch.zeros(ctx.nnz(rho), dtype=torch.float32, device="cuda:0")
    s_ref, model_ref = np.zeros(n, np.float32), np.zeros(n, np.float32)
    diff_ref, sent_ref = np.zeros((W, n), np.float32), np.zeros((W, n), np.float32)
    for e in range(6):
        wi, wv = oracle.worker_step(synth.gaussian(n, rng), s_ref, off, np.float32(1.0), np.float32(0.9), rho)
        oracle.server_push(model_ref, diff_ref, wi, wv)
        ctx.server_push(model, e % W, torch.from_numpy(wi.view(np.int32)).cuda(), torch.from_numpy(wv).cuda(), wi.size)
        for form, rows, ref in (("diff", diff, diff_ref), ("sent", sent, sent_ref)):
            if form == "diff":
                qi, qv = oracle.server_pull(diff_ref, e % W, off, rho)
                K = ctx.server_pull(e % W, rho, idx, val)
            else:
                qi, qv = oracle.server_pull_sent(model_ref, sent_ref, e % W, off, rho)
                K = ctx_sent.server_pull_sent(model, e % W, rho, idx, val)
            torch.cuda.synchronize()
            assert_pairs_match(to_host_u32(idx[:K]), val[:K].cpu().numpy(), qi, qv, f"{form} event {e}")
            assert_state_match(rows.cpu().numpy().ravel(), ref.ravel(), f"{form} rows {e}")
    for c in (ctx, ctx_sent):
        assert c.stats().internal_errors == 0
        c.close()
