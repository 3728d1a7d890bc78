"""Which rank a pull aims its next threshold at.  The row is drawn anew before every pull, so a pull
finds about as many candidates as the one before it has aimed at: 2 k, or 2.5 k for layouts of many
tensors once a row has been pulled ten times.  (The message is exact either way; the lists' length is
what it costs.)"""
import numpy as np
import pytest

from paper_1910_10929_amd import dgs, synth

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("launches")]


@pytest.mark.parametrize("sizes,rho,young,old", [
    ([600_000], 0.01, 2.0, 2.0),                          # one tensor
    ([150_000] * 7, 0.01, 2.0, 2.0),                      # seven
    ([150_000] * 8 + [100] * 5, 0.01, 2.0, 2.5),          # eight (and small ones, which have no lists)
    ([800_000] * 8, 0.01, 2.0, 2.0),                      # 2.5 k beyond the LDS list of one workgroup
    ([1_500_000] * 8, 0.01, 2.0, 2.5),                    # on the chain
])
def test_candidates_per_pull(oracle, sizes, rho, young, old):
    import torch
    off = synth.offsets_from_sizes(sizes)
    n = int(off[-1])
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(11)
    ctx = dgs.Context(off, W=1)
    row = torch.zeros((1, n), device="cuda:0")
    ctx.server_attach(row)
    K = ctx.nnz(rho)
    listed = sum(int(np.ceil(rho * s)) for s in sizes if s > 8192)
    idx, val = torch.zeros(K, dtype=torch.int32, device="cuda:0"), torch.zeros(K, device="cuda:0")
    seen = []
    for t in range(16):
        row[0] = torch.randn(n, device="cuda:0", generator=gen)
        before = ctx.stats().candidates
        ref = row.cpu().numpy() if t in (9, 11) and n < 2_000_000 else None
        ctx.server_pull(0, rho, idx, val)
        seen.append((ctx.stats().candidates - before) / listed)
        if ref is not None:
            wi, wv = oracle.server_pull(ref, 0, off, rho)
            assert np.array_equal(idx.cpu().numpy().view(np.uint32), wi) and np.array_equal(val.cpu().numpy(), wv)
    assert ctx.stats().internal_errors == 0 and ctx.stats().repaired_tensors == 0
    ctx.close()
    # expected: the rank, 4 sqrt(k) + 16 of slack included, to within five standard deviations of a count
    # of that size and the width of the threshold's bucket (the pull that first aims higher extrapolates
    # from a list that ends below its rank: not checked)
    for factor, part in ((young, seen[1:11]), (old, seen[12:])):
        ks = [int(np.ceil(rho * s)) for s in sizes if s > 8192]
        want = sum(factor * k + 4 * np.sqrt(k) + 16 for k in ks) / listed
        slack = 5 * np.sqrt(want / listed) + 0.03
        assert all(abs(c - want) < slack for c in part), (want, slack, seen)
