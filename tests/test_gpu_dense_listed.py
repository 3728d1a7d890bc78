"""Dense requests whose k-th keys stay where they were: from the third call on the accumulate pass writes down the keys that share
the k-th one's leading bits, tile by tile, and the refinements read those.  Lists of no entry, of what a wavefront stages (64),
of all there is room for (496) and of one more each; tiles shared by two tensors; tensors whose keys move away, so that the list is of
the wrong bits, and back.  Bit for bit against the oracle: each value is the result of one correctly rounded operation."""
import numpy as np
import pytest

from paper_1910_10929_amd import dgs, synth
from harness import Worker, assert_pairs_match, assert_state_match

pytestmark = pytest.mark.gpu

SIZES = [700, 70_001, 9_000, 8_193, 2_000, 600_123]


def gradient(off, rho, inside, rng):
    """Every tensor's k-th key in [1, 1.0625), with `inside` keys there in one whole tile of it and 60 in the others."""
    a = rng.uniform(0.01, 0.1, off[-1]).astype(np.float32)
    for lo, hi in zip(off[:-1].astype(int), off[1:].astype(int)):
        n, k = hi - lo, int(np.ceil(rho * (hi - lo)))
        if n <= 8192:
            continue
        first = -(-lo // 1024) * 1024                   # its first whole tile
        rest = np.setdiff1d(np.arange(lo, hi), np.arange(first, first + 1024))
        rest = rng.permutation(rest)
        a[rest[:k - 40]] = 4.0
        a[rest[k - 40:k + 20]] = 1.0 + 0.06 * rng.random(60).astype(np.float32)
        a[first + rng.permutation(1024)[:inside]] = 1.0 + 0.06 * rng.random(inside).astype(np.float32)
    return a * rng.choice([-1.0, 1.0], a.size).astype(np.float32)


@pytest.mark.parametrize("misalign", [0, 3])
@pytest.mark.parametrize("inside", [0, 64, 65, 496, 497, 1024])
def test_listed_keys(oracle, inside, misalign):
    rng = np.random.default_rng(40 + inside)
    off = synth.offsets_from_sizes(SIZES)
    ctx = dgs.Context(off, W=0)
    w = Worker(ctx, density_max=1.0, misalign=misalign)
    for call, scale in enumerate([1, 1, 1, 1, 1.5, 1.5, 1.5, 1.5, 1]):
        grad = gradient(off, 0.1, inside, rng)
        s_ref = np.zeros(int(off[-1]), np.float32)
        w.state.zero_()
        wi, wv = oracle.worker_step(grad, s_ref, off, np.float32(scale), np.float32(0.5), 0.1)
        gi, gv = w.step(grad, scale, 0.5, 0.1)
        assert_pairs_match(gi, gv, wi, wv, f"call {call}")
        assert_state_match(w.state_host(), s_ref, f"call {call}")
    assert ctx.stats().internal_errors == 0
    ctx.close()
