"""The chain for long candidate lists at the edges of its work split: tensors of one slab (128
tiles) and one element more, a last slab of one tile, tensors that share tiles, tiles with more
than 64 candidates, tie classes that cross slabs; and the form with half-sized workgroups, which
takes over at 2048 slabs.  Bit for bit against the oracle, or against the single-workgroup
selection where the oracle would take minutes."""
import numpy as np
import pytest

from paper_1910_10929_amd import dgs, synth
from harness import run_worker_parity

pytestmark = pytest.mark.gpu
SIZES = [65_536, 3, 131_072, 131_073, 64 * 1024 + 1, 262_144 + 128 * 1024 + 1, 70_001]


@pytest.mark.parametrize("kind", ["gaussian", "ties", "crowded"])
@pytest.mark.parametrize("rho", [0.0005, 0.03])
def test_chain_slab_edges(oracle, rho, kind):
    off = synth.offsets_from_sizes(SIZES)
    n = int(off[-1])
    rng = np.random.default_rng(81)
    grads = [synth.gaussian(n, rng) for _ in range(4)]
    for g in grads:
        if kind == "ties":
            g[:] = np.round(g * 4) / 4
        elif kind == "crowded":
            for t in (0, 63, 64, 127, 128, 129, 200):       # up to 150 of a tile's elements far above the rest
                g[t * 1024 + rng.choice(1024, 150, replace=False)] *= np.float32(40.0)
    st = run_worker_parity(oracle, off, grads, np.float32(0.5), np.float32(0.9), rho, seg_mode=dgs.SEG_ALWAYS)
    assert st.segmented_tensors > 0 and st.internal_errors == 0


@pytest.mark.parametrize("op", ["worker", "diff", "sent"])
def test_half_sized_workgroups_agree_with_the_single_workgroup_selection(op):
    import torch
    n, rho = 2050 * 128 * 1024 + 77, 2e-5
    off = np.array([0, 200_000_003, n], dtype=np.uint64)
    outs = []
    for mode in (dgs.SEG_ALWAYS, dgs.SEG_NEVER):
        gen = torch.Generator(device="cuda:0")
        gen.manual_seed(5)
        ctx = dgs.Context(off, W=0 if op == "worker" else 1)
        ctx.set_option(dgs.OPT_SEGMENTED, mode)
        K = ctx.nnz(rho)
        idx, val = torch.zeros(K, dtype=torch.int32, device="cuda:0"), torch.zeros(K, device="cuda:0")
        row = torch.randn((1, n), device="cuda:0", generator=gen)
        model = torch.randn(n, device="cuda:0", generator=gen)
        if op == "diff":
            ctx.server_attach(row)
        elif op == "sent":
            ctx.server_attach_sent(row)
        run = []
        for _ in range(2):
            if op == "worker":
                ctx.worker_step(model, row[0], 0.1, 0.5, rho, idx, val)
            elif op == "diff":
                ctx.server_pull(0, rho, idx, val)
            else:
                ctx.server_pull_sent(model, 0, rho, idx, val)
            run += [idx.clone(), val.view(torch.int32).clone()]
        run.append(row.view(torch.int32).clone())
        st = ctx.stats()
        assert st.internal_errors == 0 and (st.segmented_tensors > 0) == (mode == dgs.SEG_ALWAYS)
        ctx.close()
        outs.append(run)
    for a, b in zip(*outs):
        assert torch.equal(a, b)
