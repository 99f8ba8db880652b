"""The insert's paths against the oracle at the sizes where they part: refreshes of entries
many requests share."""
import numpy as np
import pytest

from paper_2607_08565_amd import workload as W
from tests.parity import Pair, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(dev):
    yield


def _prompts(rng, R, shared, own, block=16):
    """R prompts: a common prefix of `shared` blocks, then up to `own` private blocks."""
    base = rng.integers(0, W.VOCAB, block * shared, dtype=np.int32)
    ps = [np.concatenate([base, rng.integers(0, W.VOCAB, int(rng.integers(0, block * own + 1)), dtype=np.int32)])
          for _ in range(R)]
    off = np.zeros(R + 1, np.int64)
    off[1:] = np.cumsum([len(p) for p in ps])
    return np.concatenate(ps), off


def insert_both(pair, probed, d_keys, d_boff, nb, okeys, blk_off, inst, sess, epoch):
    inst, sess = np.asarray(inst, np.int32), np.asarray(sess, np.uint32)
    if not probed:
        return pair.insert_both(d_keys, d_boff, nb, okeys, blk_off, inst, sess, epoch)
    state = pair.gix.probe(d_keys, d_boff, nb)
    pair.gix.insert_probed(state, len(blk_off) - 1, nb, to_dev(inst), to_dev(sess), epoch)
    return pair.oix.insert(okeys, blk_off, inst, sess, epoch)


@pytest.mark.parametrize("I,n_inst_used", [(24, 24), (300, 12), (300, 5)])
def test_refresh_of_entries_shared_by_many_requests(I, n_inst_used):
    """Each instance's entries of a shared prefix are refreshed by ~100 requests at once, with a
    newer, the same and an older epoch: bitmap members (more holders than the threshold), plain
    keys of several holders, and a mix with new blocks; an entry's epoch only rises."""
    rng = np.random.default_rng(I + n_inst_used)
    R = 100 * n_inst_used
    pair = Pair(400_000, I)
    toks, off = _prompts(rng, R, 24, 3)
    d_boff, nb, d_keys, okeys, blk_off = pair.hash_both(toks, off)
    for k, epoch in enumerate((5, 9, 9, 3, 11)):
        inst = rng.integers(0, n_inst_used, R)
        assert insert_both(pair, True, d_keys, d_boff, nb, okeys, blk_off, inst, rng.permutation(R), epoch) == 0
        say(f"  I={I} used={n_inst_used} insert {k}: epoch {epoch}, {nb} blocks")
        pair.compare_index(f"insert {k} at epoch {epoch}")
