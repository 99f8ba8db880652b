"""The self-contained match against the oracle at each number of wavefronts per request (1, 2, 4
and 8) and at the edges of their rounds: prompts of 0, 1 and a round's blocks and one less
or more, shared prefixes held by few instances (lists), by more than a list keeps and by most
(bitmaps), prompts that miss early, late and not at all, and prompts whose blocks around the
edges of the wavefronts' stretches are the only ones that nobody holds."""
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


@pytest.mark.parametrize("R,nb", [(1, 700), (40, 300), (3000, 130)])
def test_gaps_at_the_edges_of_stretches(R, nb):
    """Block j of a prompt is held by nobody, those before and after it by one, a few or most
    instances (a bitmap): hits end at j, whatever lies behind it."""
    rng = np.random.default_rng(R)
    for I, holders in ((6, 1), (6, 4), (300, 200)):
        gaps = [g for g in (0, 1, 62, 63, 64, 126, 127, 128, 191, 255, 447, 511, 512, nb - 1) if g < nb]
        n = R * nb
        pair = Pair(min(R, 40) * nb * (holders + 4) + 2 * n, I, block=2)
        toks = rng.integers(0, W.VOCAB, 2 * n, dtype=np.int32)
        off = np.arange(R + 1, dtype=np.int64) * 2 * nb
        d_boff, n, d_keys, okeys, blk_off = pair.hash_both(toks, off)
        for g0 in range(0, len(gaps), max(1, R)):  # every gap, some of them once per request
            at = np.array([gaps[(g0 + r) % len(gaps)] for r in range(R)])
            pair = Pair(min(R, 40) * nb * (holders + 4) + 2 * n, I, block=2)
            keep = np.ones(n, bool)
            keep[blk_off[:-1] + at] = False
            for r0 in range(0, R, 40):  # many holders for the first 40 prompts, one for the rest
                rows = np.arange(r0, min(R, r0 + 40))
                k = np.concatenate([okeys[blk_off[r]:blk_off[r + 1]][keep[blk_off[r]:blk_off[r + 1]]] for r in rows])
                ko = np.arange(len(rows) + 1, dtype=np.int64) * (nb - 1)
                for i in rng.permutation(I)[:holders if r0 == 0 else 1]:
                    assert pair.insert_both(to_dev(k), to_dev(ko), len(k), k, ko, np.full(len(rows), i), rows, 1) == 0
            gm, om = pair.gix.match(d_keys, d_boff, n).cpu().numpy(), pair.oix.match(okeys, blk_off)
            assert np.array_equal(gm, om), np.argwhere(gm != om)[:4]
            assert np.array_equal(om.max(1), at)


@pytest.mark.parametrize("I", [100, 5000])
@pytest.mark.parametrize("R,nb", [(1, 600), (5, 130), (1, 64), (3000, 66)])
def test_prompts_whose_first_blocks_were_evicted(R, nb, I):
    """Prompts of which most instances held every block but the last of a wavefront's stretch,
    after an eviction of everybody's first block: its key's bitmap is there and empty."""
    rng = np.random.default_rng(R + I)
    pair = Pair(60 * nb + 5000, I)
    keys = np.sort(rng.integers(1 << 40, 2**63, nb, dtype=np.int64).astype(np.uint64))  # the lowest key goes first
    held = np.delete(keys, 63)
    ko = np.array([0, len(held)], np.int64)
    who = rng.permutation(I)[:50]
    for i in who:
        assert pair.insert_both(to_dev(held), to_dev(ko), len(held), held, ko, [i], [7], 1) == 0
    blk_off = np.arange(R + 1, dtype=np.int64) * nb
    okeys = np.tile(keys, R)
    d_keys, d_off = to_dev(okeys), to_dev(blk_off)
    for num in (0, 20, 30):  # entries to evict: none, some of the first block's, the rest of them
        n, _ = pair.gix.stats()
        pair.gix.evict(num, n)
        assert pair.oix.evict(num, n) == 0
        gm, om = pair.gix.match(d_keys, d_off, R * nb).cpu().numpy(), pair.oix.match(okeys, blk_off)
        assert np.array_equal(gm, om), np.argwhere(gm != om)[:4]
    pair.compare_index("evicted")
    assert not om.any()
