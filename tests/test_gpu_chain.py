"""The chain for long candidate lists at the edges of its work split: tensors that fill exactly one
slab (128 tiles) and one element more, a last slab of one tile, tensors that share tiles, tiles with
more than 64 candidates, tie classes that cross slabs, messages completed with zeros; and the form
with half-sized workgroups, which takes over at 2048 slabs.  Bit for bit against the oracle, or against the single-workgroup
selection where the oracle would take minutes."""
import numpy as np
import pytest

from paper_1910_10929_amd import dgs, synth
from harness import assert_pairs_match, assert_state_match, run_worker_parity, to_host_u32

pytestmark = pytest.mark.gpu
SIZES = [65_536, 3, 131_072, 131_073, 64 * 1024 + 1, 262_144 + 128 * 1024 + 1, 70_001]


# tensors that start at a tile: slabs are full, or hold one element more (the 1023 fill the tile up)
ALIGNED = [128 * 1024, 128 * 1024 + 1, 1023, 256 * 1024, 65_536, 129 * 1024]


@pytest.mark.parametrize("kind", ["gaussian", "ties", "crowded"])
@pytest.mark.parametrize("rho", [0.0005, 0.03])
def test_chain_slab_edges(oracle, rho, kind):
    _edges(oracle, SIZES, rho, kind)


@pytest.mark.parametrize("kind", ["gaussian", "ties"])
def test_chain_full_slabs(oracle, kind):
    _edges(oracle, ALIGNED, 0.01, kind)


def _edges(oracle, sizes, rho, kind):
    off = synth.offsets_from_sizes(sizes)
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


def _sparse_rows(n, off, rho, rng):
    """Rows with fewer nonzeros than k in every tensor: none, a few at the start, k / 4 anywhere, k - 1
    packed around the place where the leading run of zeros ends, and all of them behind it."""
    for kind in ("empty", "start", "anywhere", "run-end", "tail"):
        row = np.zeros(n, np.float32)
        for j in range(len(off) - 1):
            lo, nj = int(off[j]), int(off[j + 1] - off[j])
            k = int(np.ceil(rho * nj))
            if kind == "start":
                at = np.arange(min(k // 2, 5))
            elif kind == "anywhere":
                at = rng.choice(nj, k // 4, replace=False)
            elif kind == "run-end":
                at = np.clip(np.arange(k - 1) + k // 2, 0, nj - 1)
            elif kind == "tail":
                at = nj - 1 - np.arange(k // 3)
            else:
                at = np.zeros(0, np.int64)
            row[lo + at] = rng.standard_normal(at.size).astype(np.float32)
        row[::97] += np.float32(-0.0)
        yield kind, row


@pytest.mark.parametrize("form", ["worker", "diff", "sent"])
def test_messages_completed_with_zeros(oracle, form):
    """Fewer nonzeros than k on the chain: several slabs and more than 1024 tiles, tensors that share
    tiles, twice per row content (estimated threshold, then the hint)."""
    import torch
    off = synth.offsets_from_sizes([70_001, 3, 1100 * 1024 + 17, 131_072, 65_536])
    n, rho = int(off[-1]), 0.03
    rng = np.random.default_rng(84)
    ctx = dgs.Context(off, W=0 if form == "worker" else 1)
    ctx.set_option(dgs.OPT_SEGMENTED, dgs.SEG_ALWAYS)
    K = ctx.nnz(rho)
    idx, val = torch.zeros(K, dtype=torch.int32, device="cuda:0"), torch.zeros(K, device="cuda:0")
    row, zero = torch.zeros((1, n), device="cuda:0"), torch.zeros(n, device="cuda:0")
    if form != "worker":
        (ctx.server_attach if form == "diff" else ctx.server_attach_sent)(row)
    for kind, content in _sparse_rows(n, off, rho, rng):
        for again in range(2):
            ref = content.reshape(1, n).copy()
            row.copy_(torch.from_numpy(ref))
            if form == "worker":
                wi, wv = oracle.worker_step(np.zeros(n, np.float32), ref[0], off, np.float32(1.0), np.float32(0.5), rho)
                ctx.worker_step(zero, row[0], 1.0, 0.5, rho, idx, val)
            elif form == "diff":
                wi, wv = oracle.server_pull(ref, 0, off, rho)
                ctx.server_pull(0, rho, idx, val)
            else:
                wi, wv = oracle.server_pull_sent(np.zeros(n, np.float32), ref, 0, off, rho)
                ctx.server_pull_sent(zero, 0, rho, idx, val)
            torch.cuda.synchronize()
            assert_pairs_match(to_host_u32(idx), val.cpu().numpy(), wi, wv, f"{kind} {again}")
            assert_state_match(row.cpu().numpy()[0], ref[0], f"{kind} {again}")
    st = ctx.stats()
    assert st.internal_errors == 0 and st.segmented_tensors > 0 and st.fallback_tensors == 0
    ctx.close()
