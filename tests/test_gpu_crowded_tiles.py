"""Joins of tiles that hold more candidates than their first line (8): few of them in a round of 1024
tiles (up to 32, one wavefront each) and many (16 lanes each, 256 at a time), with counts around a line,
a step of the copy (16) and the slots of a tile (256), behind a tensor whose last tile is shared.
Bit for bit against the oracle: each value is the result of one correctly rounded operation."""
import numpy as np
import pytest

from paper_1910_10929_amd import dgs, synth
from harness import Worker, assert_pairs_match, assert_state_match

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("launches")]

COUNTS = [9, 24, 25, 40, 8, 41, 10]


@pytest.mark.parametrize("crowded", [1, 32, 33, 64, 255, 256, 257, 300])
def test_crowded_tiles(oracle, crowded):
    rng = np.random.default_rng(crowded)
    tiles = 1100                                     # a full round and a part of one
    off = synth.offsets_from_sizes([9001, tiles * 1024])
    n, base = int(off[-1]), 9216                     # (tile 8 belongs to both tensors)
    where = [np.arange(8950, 9020)]                  # nonzeros of both in the shared tile
    for i, t in enumerate(rng.permutation(1000)[:crowded]):
        c = 256 if i == 0 else COUNTS[i % len(COUNTS)]
        where.append(base + t * 1024 + rng.permutation(1024)[:c])
    for t in range(1000, 1098):
        where.append(base + t * 1024 + rng.permutation(1024)[:t % 12])
    where = np.unique(np.concatenate(where))
    own = int((where >= 9001).sum())
    rho = (own // 2 + 0.5) / (tiles * 1024)
    ctx = dgs.Context(off, W=0)
    w = Worker(ctx, density_max=rho)
    s_ref = np.zeros(n, np.float32)
    for step in range(4):
        g = np.zeros(n, np.float32)
        g[where] = 1.0 + rng.random(where.size).astype(np.float32)
        wi, wv = oracle.worker_step(g, s_ref, off, np.float32(1.0), np.float32(0.0), rho)
        gi, gv = w.step(g, 1.0, 0.0, rho)
        assert_pairs_match(gi, gv, wi, wv, f"step {step}")
        assert_state_match(w.state_host(), s_ref, f"state {step}")
    st = ctx.stats()
    assert st.internal_errors == 0 and st.fallback_tensors == 0
    ctx.close()
