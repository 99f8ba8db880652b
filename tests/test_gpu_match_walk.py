"""The self-contained match against the oracle at each number of wavefronts per request (1, 2, 4
and 8) and at the edges of their rounds: prompts of 0, 1 and a round's blocks and one less
or more, shared prefixes held by few instances (lists), by more than a list keeps and by most
(bitmaps), prompts that miss early, late and not at all."""
import numpy as np
import pytest

from paper_2607_08565_amd import workload as W
from tests.parity import Pair, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(dev):
    yield


@pytest.mark.parametrize("R,lens,I", [(1, [511], 8), (1, [513], 300), (3, [512, 0, 1025], 24), (40, [63, 64, 65, 700], 5),
                                      (1100, [255, 256, 257, 300, 0], 40), (2100, [127, 128, 129, 140], 9),
                                      (8200, [64, 65, 66, 90, 1], 12), (6, [520, 1, 2, 64], 5000)])
def test_match_rounds(R, lens, I):
    rng = np.random.default_rng(R + I)
    B = 2  # short blocks keep the prompts small
    n = np.array([lens[r % len(lens)] for r in range(R)], np.int64)
    pre = [rng.integers(0, W.VOCAB, B * 600, dtype=np.int32) for _ in range(3)]
    ps = []
    for r in range(R):
        p = rng.integers(0, W.VOCAB, B * int(n[r]), dtype=np.int32)
        k = min(len(p), B * int(rng.choice([0, 30, 100, 600])))
        p[:k] = pre[int(rng.integers(0, 3))][:k]
        ps.append(p)
    off = np.zeros(R + 1, np.int64)
    off[1:] = np.cumsum([len(p) for p in ps])
    toks = np.concatenate(ps) if len(ps) else np.zeros(0, np.int32)
    pair = Pair(4 * int(n.sum()) + 100, I, block=B)
    d_boff, nb, d_keys, okeys, blk_off = pair.hash_both(toks, off)
    # whole prompts on few, then on many instances; then half of the oldest entries leave
    for k, holders in enumerate((min(I, 3), I)):
        inst = rng.integers(0, holders, R)
        assert pair.insert_both(d_keys, d_boff, nb, okeys, blk_off, inst, np.arange(R), k) == 0
        g, o = pair.gix.match(d_keys, d_boff, nb).cpu().numpy(), pair.oix.match(okeys, blk_off)
        assert np.array_equal(g, o), np.argwhere(g != o)[:4]
    pair.gix.evict(1, 2)
    assert pair.oix.evict(1, 2) == 0
    g, o = pair.gix.match(d_keys, d_boff, nb).cpu().numpy(), pair.oix.match(okeys, blk_off)
    assert np.array_equal(g, o), np.argwhere(g != o)[:4]
    say(f"  R={R} I={I} blocks={nb}: hits {int((o > 0).sum())}")
