"""Block keys against the oracle for blocks of 32 to 256 tokens (read as sub-blocks of 16) at
the edges of their tiles and at each number of wavefronts per request, and of prompts around
the lengths from which they are tiled, through the hash call and the fused hash + partition; a
bad token range keeps the caller's earlier keys."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_08565_amd import workload as W
from tests.parity import Pair, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(dev):
    yield


@pytest.mark.parametrize("B", [16, 32, 48, 64, 128, 256])
@pytest.mark.parametrize("blocks", [[0, 1, 63, 64, 65, 3], [0, 1, 63, 64, 65, 127, 128, 129],
                                    [127, 128, 129, 200], [255, 256, 257, 513, 600]])
def test_keys_at_tile_edges(B, blocks):
    from paper_2607_08565_amd import smetric as S
    rng = np.random.default_rng(B + len(blocks))
    lens = np.array([B * n + int(rng.integers(0, B)) for n in blocks for _ in range(2)], np.int64)
    off = np.zeros(len(lens) + 1, np.int64)
    off[1:] = np.cumsum(lens)
    toks = rng.integers(-2**31, 2**31, int(off[-1]), dtype=np.int64).astype(np.int32)
    pair = Pair(50_000, 4, block=B)
    d_boff, nb, d_keys, okeys, blk_off = pair.hash_both(toks, off)  # compares every key
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    keys, state = pair.gix.hash_partition(to_dev(toks), to_dev(off), d_boff, nb, block_size=B, status=status)
    assert int(status.item()) == 0 and np.array_equal(keys[:nb].cpu().numpy(), okeys)
    R = len(lens)
    for epoch in (1, 2):
        pair.gix.probe_lookup(state, keys, d_boff, nb)
        assert np.array_equal(pair.gix.match_probed(state, keys, d_boff, nb).cpu().numpy(), pair.oix.match(okeys, blk_off))
        inst = rng.integers(0, 4, R).astype(np.int32)
        pair.gix.insert_probed(state, R, nb, to_dev(inst), to_dev(np.arange(R, dtype=np.uint32)), epoch)
        assert pair.oix.insert(okeys, blk_off, inst, np.arange(R), epoch) == 0
        pair.compare_index(f"B={B} epoch {epoch}")
    say(f"  B={B}: {nb} blocks")


@pytest.mark.parametrize("B", [32, 64, 256])
@pytest.mark.parametrize("R,mean", [(255, 32), (255, 64), (255, 65), (256, 32), (256, 33), (1, 64), (1, 65), (3000, 1)])
def test_keys_where_short_prompts_end(B, R, mean):
    """Batches whose blocks per prompt are just at and above the tiled kernel's line."""
    from paper_2607_08565_amd import smetric as S
    rng = np.random.default_rng(B + R)
    n = rng.integers(0, 2 * mean + 1, R)
    while n.sum() != R * mean:  # exactly R * mean blocks
        n[rng.integers(0, R)] += 1 if n.sum() < R * mean else 0
        n[rng.integers(0, R)] -= 1 if n.sum() > R * mean else 0
        n = np.maximum(n, 0)
    off = np.zeros(R + 1, np.int64)
    off[1:] = np.cumsum(B * n + rng.integers(0, B, R))
    toks = rng.integers(-2**31, 2**31, int(off[-1]), dtype=np.int64).astype(np.int32)
    pair = Pair(100, 4, block=B)
    d_boff, nb, d_keys, okeys, blk_off = pair.hash_both(toks, off)
    assert nb == R * mean
    keys, state = pair.gix.hash_partition(to_dev(toks), to_dev(off), d_boff, nb, block_size=B)
    assert np.array_equal(keys[:nb].cpu().numpy(), okeys)
    pair.gix.probe_lookup(state, keys, d_boff, nb)
    assert not pair.gix.match_probed(state, keys, d_boff, nb).any()


@pytest.mark.parametrize("B", [32, 256])
def test_bad_token_range_of_long_prompts(B):
    """As below with prompts long enough to be tiled."""
    test_bad_token_range_keeps_earlier_keys(B, 10)


@pytest.mark.parametrize("B", [32, 48, 256])
def test_bad_token_range_keeps_earlier_keys(B, k=1):
    """A request whose token range does not give its block range: status is set, its keys stay
    what the buffer held, and the probe state is valid with those (blocks of 16 invalidate it)."""
    from paper_2607_08565_amd import smetric as S
    rng = np.random.default_rng(B)
    T = B * k
    toks = rng.integers(0, W.VOCAB, T * 40, dtype=np.int32)
    good = np.array([0, T * 10, T * 27, T * 40], np.int64)
    bad = np.array([0, T * 10, T * 25, T * 40], np.int64)  # request 1 has 15 k blocks of tokens for 17 k
    blk_off = np.array([0, 10, 27, 40], np.int64) * k
    pair = Pair(10_000, 4, block=B)
    d_boff = to_dev(blk_off)
    _, okeys = oracle.hash_blocks(toks, good, B, W.DEFAULT_SEED)
    keys = to_dev(okeys.copy())
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    tokd = to_dev(np.concatenate([toks[: T * 25], toks[T * 27:], toks[: T * 2]]))
    keys, state = pair.gix.hash_partition(tokd, to_dev(bad), d_boff, 40 * k, block_size=B, keys=keys, status=status)
    assert int(status.item()) == S.EINVAL
    got = keys.cpu().numpy()
    assert np.array_equal(got[10 * k:27 * k], okeys[10 * k:27 * k]) and np.array_equal(got[:10 * k], okeys[:10 * k])
    pair.gix.probe_lookup(state, keys, d_boff, 40 * k)
    inst = np.array([0, 1, 2], np.int32)
    pair.gix.insert_probed(state, 3, 40 * k, to_dev(inst), to_dev(np.arange(3, dtype=np.uint32)), 1)
    assert pair.oix.insert(got, blk_off, inst, np.arange(3), 1) == 0
    pair.compare_index(f"B={B}")
