"""The region-ordered insert's dedupe of bins larger than its LDS table takes at once, against
the oracle: blocks that thousands of requests share, on few instances (the repeated pairs
stream through LDS), on thousands (too many distinct pairs: the fallback table), and on a
number where bins lie on both sides; the lowest request of a pair gives its session."""
import numpy as np
import pytest

from tests.parity import Pair
from tests.test_gpu_insert_paths import _prompts, insert_both

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(dev):
    yield


@pytest.mark.parametrize("I,R,shared", [(3, 6000, 50), (40, 6000, 50), (700, 6000, 50), (1024, 7000, 50),
                                        (2500, 9000, 40), (6000, 9000, 40), (40, 70_000, 4)])
def test_shared_blocks(I, R, shared):
    rng = np.random.default_rng(I + R)
    pair = Pair(shared * min(I, R) + 8 * R, I)
    toks, off = _prompts(rng, R, shared, 3)
    d_boff, nb, d_keys, okeys, blk_off = pair.hash_both(toks, off)
    assert nb > 1 << 18
    for epoch in (1, 2):
        rc = insert_both(pair, True, d_keys, d_boff, nb, okeys, blk_off, rng.integers(0, I, R), rng.permutation(R), epoch)
        assert rc == 0
        pair.compare_index(f"I={I} R={R} epoch {epoch}")
