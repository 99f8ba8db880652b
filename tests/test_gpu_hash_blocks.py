"""Block keys against the oracle for blocks of 32 to 256 tokens (read as sub-blocks of 16) at
the edges of their tiles and at each number of wavefronts per request, through the hash call
and the fused hash + partition; a bad token range keeps the caller's earlier keys."""
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
@pytest.mark.parametrize("blocks", [[0, 1, 63, 64, 65, 3], [127, 128, 129, 200], [255, 256, 257, 513, 600]])
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


@pytest.mark.parametrize("B", [32, 48, 256])
def test_bad_token_range_keeps_earlier_keys(B):
    """A request whose token range does not give its block range: status is set, its keys stay
    what the buffer held, and the probe state is valid with those (blocks of 16 invalidate it)."""
    from paper_2607_08565_amd import smetric as S
    rng = np.random.default_rng(B)
    toks = rng.integers(0, W.VOCAB, B * 40, dtype=np.int32)
    good = np.array([0, B * 10, B * 27, B * 40], np.int64)
    bad = np.array([0, B * 10, B * 25, B * 40], np.int64)  # request 1 has 15 blocks of tokens for 17
    blk_off = np.array([0, 10, 27, 40], np.int64)
    pair = Pair(10_000, 4, block=B)
    d_boff = to_dev(blk_off)
    _, okeys = oracle.hash_blocks(toks, good, B, W.DEFAULT_SEED)
    keys = to_dev(okeys.copy())
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    tokd = to_dev(np.concatenate([toks[: B * 25], toks[B * 27:], toks[: B * 2]]))
    keys, state = pair.gix.hash_partition(tokd, to_dev(bad), d_boff, 40, block_size=B, keys=keys, status=status)
    assert int(status.item()) == S.EINVAL
    got = keys.cpu().numpy()
    assert np.array_equal(got[10:27], okeys[10:27]) and np.array_equal(got[:10], okeys[:10])
    pair.gix.probe_lookup(state, keys, d_boff, 40)
    inst = np.array([0, 1, 2], np.int32)
    pair.gix.insert_probed(state, 3, 40, to_dev(inst), to_dev(np.arange(3, dtype=np.uint32)), 1)
    assert pair.oix.insert(got, blk_off, inst, np.arange(3), 1) == 0
    pair.compare_index(f"B={B}")
