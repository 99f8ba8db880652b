"""Refreshes by store and by atomic against the oracle, on batches of every insert path:
epochs that rise, stay, fall and rise again, in an index that keeps its highest epoch and in
one whose bytes were written before it was kept (its word in the header zero); inserts that
change nothing (too large, a bad target) with a higher epoch in between; after an eviction in
place and after a rebuild; bytes that another process wrote to in between."""
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


def test_epochs_raised_by_another_process():
    """An index's bytes that went through a process that raises epochs and leaves the header's
    highest one as it was: restored here, its entries keep the newer epochs."""
    rng = np.random.default_rng(8)
    R, nb = 3000, 270_000
    pair = Pair(2 * nb, 40)
    toks, off = _sized(rng, R, nb, 6)
    d_boff, n, d_keys, okeys, blk_off = pair.hash_both(toks, off)
    inst, sess = rng.integers(0, 40, R), rng.permutation(R)
    for epoch in (1, 20, 10):
        if epoch == 20:
            before = pair.gix.mem[12:16].clone()
        insert_both(pair, True, d_keys, d_boff, n, okeys, blk_off, inst, sess, epoch)
        if epoch == 20:
            snap = pair.gix.snapshot()
            snap[12:16] = before
            snap[24:32] ^= 0x55  # the process that keeps it
            pair.gix.restore(snap)
        pair.compare_index(f"epoch {epoch}")
