"""The pull without secondary compression at the edges of its kernels: a last tile with one
element, rows at odd addresses, tiles whose nonzeros just fit their slots (256) or outgrow them,
more than one chunk of the position scan (4096 tiles), a capacity that is one short.  Values are
copies or single fp32 operations: compared bit for bit with numpy."""
import numpy as np
import pytest

from paper_1910_10929_amd import dgs, synth

pytestmark = pytest.mark.gpu


def _row(n, rng):
    row = np.where(rng.random(n) < 0.02, rng.standard_normal(n), 0.0).astype(np.float32)
    for t, count in ((0, 256), (1, 257), (2, 1024), (5, 255)):      # crowded tiles
        if (t + 1) * 1024 <= n:
            row[t * 1024:(t + 1) * 1024] = 0.0
            row[t * 1024 + rng.choice(1024, count, replace=False)] = rng.standard_normal(count).astype(np.float32)
    row[::97] = np.float32(-0.0)                                    # zeros of either sign are not sent
    return row


@pytest.mark.parametrize("form", ["diff", "sent"])
@pytest.mark.parametrize("n", [1, 1025, 7 * 1024 + 3, 4096 * 1024 + 1027])
def test_every_nonzero_in_order(n, form):
    import torch
    rng = np.random.default_rng(n)
    diffs = [_row(n, rng), _row(n, rng)]
    model = rng.standard_normal(n).astype(np.float32)
    rows = np.stack(diffs if form == "diff" else [np.where(d != 0, model - d, model).astype(np.float32) for d in diffs])
    ctx = dgs.Context(synth.layout_flat(n), W=2)
    rows_g, model_g = torch.from_numpy(rows).cuda(), torch.from_numpy(model).cuda()
    (ctx.server_attach if form == "diff" else ctx.server_attach_sent)(rows_g)
    idx = torch.full((n + 1,), -1, dtype=torch.int32, device="cuda:0")
    val = torch.zeros(n + 1, dtype=torch.float32, device="cuda:0")
    for w in (1, 0, 1):
        value = rows[w] if form == "diff" else model - rows[w]
        want = np.nonzero(value.view(np.uint32) & 0x7FFFFFFF)[0]
        pull = ((lambda cap: ctx.server_pull_all(w, idx, val, cap)) if form == "diff"
                else (lambda cap: ctx.server_pull_all_sent(model_g, w, idx, val, cap)))
        if want.size:
            idx.fill_(-1)
            with pytest.raises(dgs.DgsError):
                pull(want.size - 1)
            torch.cuda.synchronize()
            assert (idx == -1).all() and np.array_equal(rows_g.cpu().numpy().view(np.uint32), rows.view(np.uint32))
        assert pull(want.size) == want.size
        torch.cuda.synchronize()
        assert np.array_equal(idx[:want.size].cpu().numpy(), want.astype(np.int32))
        assert np.array_equal(val[:want.size].cpu().numpy().view(np.uint32), value[want].view(np.uint32))
        rows[w][want] = 0.0 if form == "diff" else rows[w][want] + value[want]
        assert np.array_equal(rows_g.cpu().numpy().view(np.uint32), rows.view(np.uint32))
    ctx.close()
