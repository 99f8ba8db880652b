"""Refreshes by store and by atomic against the oracle, on batches of every insert path:
epochs that rise, stay, fall and rise again, in an index that keeps its highest epoch and in
one whose bytes were written before it was kept (its word in the header zero); inserts that
change nothing (too large, a bad target) with a higher epoch in between; after an eviction in
place and after a rebuild."""
import numpy as np
import pytest

from tests.parity import Pair, to_dev
from tests.test_gpu_insert_paths import _sized, insert_both

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(dev):
    yield


@pytest.mark.parametrize("kept", [True, False])
@pytest.mark.parametrize("R,nb,probed", [(3000, 270_000, True), (600, 20_000, True), (600, 20_000, False), (9, 900, True)])
def test_epochs_only_rise(R, nb, probed, kept):
    rng = np.random.default_rng(R)
    I = 40
    pair = Pair(3 * nb, I)
    toks, off = _sized(rng, R, nb, 6)
    d_boff, n, d_keys, okeys, blk_off = pair.hash_both(toks, off)
    sess = rng.permutation(R)
    inst = rng.integers(0, I, R)
    for k, epoch in enumerate((5, 9, 3, 9, 4, 10, 2)):
        if not kept:
            pair.gix.mem[12:16] = 0  # as in an index of older bytes
        if k % 2:
            inst = np.where(rng.random(R) < 0.3, rng.integers(0, I, R), inst)
        if k == 3:  # changes nothing, whatever its epoch
            bad = inst.copy()
            bad[R // 2] = I
            insert_both(pair, probed, d_keys, d_boff, n, okeys, blk_off, bad, sess, 50)
        if k in (4, 5):
            pair.gix.evict(1, 30 if k == 4 else 2)
            assert pair.oix.evict(1, 30 if k == 4 else 2) == 0
        insert_both(pair, probed, d_keys, d_boff, n, okeys, blk_off, inst, sess, epoch)
        pair.compare_index(f"insert {k} at epoch {epoch}")
