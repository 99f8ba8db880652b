"""GPU eviction's selection at its route edges against the CPU oracle, bit for bit on the
dumped entry set: one or few epochs of 65,535 to 100,001 entries, so that the entries left on
the digits lie at, below and above the 2^16 that one workgroup settles; tables below and above
the 2^15 buckets from which a sample narrows the entries copied out; a table whose sampled
buckets hold one epoch and the others another, so that the sample's range misses the cut; an
empty table, which is not read; a rebuild of keys held by few and by most instances; keys
on several instances (the last digits decide); evicted in place (small fractions of a roomy
table) and by a rebuild (large ones); bucket counts that are no multiple of a tile."""
import numpy as np
import pytest
import torch

from tests.parity import Pair, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(dev):
    yield


def _fill(pair, rng, n, epoch, n_inst, shared, keys=None):
    """n new keys in one epoch: `shared` of them on every one of four instances."""
    if keys is None:
        keys = rng.integers(1, 2**63, n, dtype=np.int64).astype(np.uint64)
    per = n // 4
    ks = []
    for r in range(4):
        own = keys[r * per:(r + 1) * per] if r < 3 else keys[3 * per:]
        ks.append(np.concatenate([keys[:shared], own[shared if r == 0 else 0:]]))
    okeys = np.concatenate(ks).astype(np.uint64)
    blk_off = np.zeros(5, np.int64)
    blk_off[1:] = np.cumsum([len(k) for k in ks])
    inst = rng.permutation(n_inst)[:4].astype(np.int32)
    sess = rng.integers(0, 1 << 24, 4).astype(np.uint32)
    d_keys = torch.from_numpy(okeys.view(np.int64)).cuda().view(torch.uint64)
    assert pair.insert_both(d_keys, to_dev(blk_off), len(okeys), okeys, blk_off, inst, sess, epoch) == 0
    return len(okeys)


@pytest.mark.parametrize("sizes,cap,fracs", [
    ((65535,), 90_000, [(1, 1000), (1, 2)]),               # one epoch, no sample, straight to one workgroup
    ((65536, 30), 400_000, [(1, 100), (65536, 65566)]),    # a whole epoch and no more
    ((65537, 40_000), 400_000, [(1, 50), (1, 3)]),         # one over
    ((100_001,), 100_200, [(1, 7)]),                       # no sample: a pass with the host first
    ((100_001, 70_000), 300_000, [(1, 90), (9, 10)]),      # and one that does
    ((30_000, 900, 50_000), 200_003, [(1, 60), (1, 50), (4, 5), (1, 1)]),
])
def test_selection_edges(sizes, cap, fracs):
    rng = np.random.default_rng(sum(sizes))
    pair = Pair(cap, 64)
    shared = 100
    for e, n in enumerate(sizes):
        got = _fill(pair, rng, n - 3 * min(shared, n // 8), e + 1, 64, min(shared, n // 8))
        assert got == n
    for num, den in fracs:
        n0, _ = pair.gix.stats()
        pair.gix.evict(num, den)
        assert pair.oix.evict(num, den) == 0
        pair.compare_index(f"{sizes} evict {num}/{den}")
        n1, _ = pair.gix.stats()
        assert n0 - n1 == -(-n0 * num // den)


def test_sample_that_misses():
    rng = np.random.default_rng(5)
    pair = Pair(300_000, 64, n_slots=1 << 19)  # 2^16 buckets, every 16th of them sampled
    keys = rng.integers(1, 2**63, 400_000, dtype=np.int64).astype(np.uint64)
    with np.errstate(over="ignore"):
        mix = (keys ^ (keys >> np.uint64(32))) * np.uint64(0xD6E8FEB86659FD93)
        mix = mix ^ (mix >> np.uint64(32))
    home = (mix >> np.uint64(48)).astype(np.int64)  # the high half of mix * 2^16
    old, new = keys[(home % 16 > 0) & (home % 16 < 12)][:60_000], keys[home % 16 == 0][:20_000]
    for epoch, ks in ((1, old), (2, new)):
        _fill(pair, rng, len(ks), epoch, 64, 0, ks)
    for num, den in ((1, 100), (1, 4), (1, 2)):
        pair.gix.evict(num, den)
        assert pair.oix.evict(num, den) == 0
        pair.compare_index(f"evict {num}/{den}")


@pytest.mark.parametrize("slots", [1 << 16, 1 << 19])
def test_empty_index(slots):
    """Nothing of the table is read into the workspace: past the counters it stays as it is."""
    rng = np.random.default_rng(3)
    pair = Pair(slots // 2, 64, n_slots=slots)
    ws = pair.gix._workspace(pair.gix.evict_ws_bytes())
    for _ in range(2):  # never filled; emptied
        ws.fill_(0xA5)
        for num, den in ((1, 20), (1, 1)):
            pair.gix.evict(num, den)
        assert bool((ws[256 + 8 * 4096:] == 0xA5).all())
        pair.compare_index("empty")
        _fill(pair, rng, 5000, 7, 64, 10)
        pair.gix.evict(1, 1)
        assert pair.oix.evict(1, 1) == 0


@pytest.mark.parametrize("n_keys,holders", [(700, 200), (3000, 40), (40, 3)])
def test_rebuild_of_widely_held_keys(n_keys, holders):
    """Members are entered again by the passes after the tiles', in several workgroups' lists."""
    rng = np.random.default_rng(n_keys)
    pair = Pair(n_keys * holders + 4000, 256)
    keys = rng.integers(1, 2**63, n_keys, dtype=np.int64).astype(np.uint64)
    off = np.array([0, n_keys], np.int64)
    for k, i in enumerate(rng.permutation(256)[:holders]):
        assert pair.insert_both(to_dev(keys), to_dev(off), n_keys, keys, off, [i], [k], 1 + k % 5) == 0
    _fill(pair, rng, 2000, 3, 256, 20)
    for num, den in ((1, 3), (1, 2)):
        pair.gix.evict(num, den)
        assert pair.oix.evict(num, den) == 0
        pair.compare_index(f"{n_keys} keys on {holders}: evict {num}/{den}")
