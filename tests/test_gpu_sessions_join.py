"""Session reconstruction's join and chains at their route edges against the CPU oracle: one
request and a few (the offers' bitmap at its smallest), request counts on both sides of the
2^17 and mean lengths of the 64 blocks where the bitmap turns lookups away, prefix lengths around the 64 lanes and the
512 lengths tested together, several candidates for one length, one chain through every
request of a batch of several workgroups, the same turns against arrival order (no parents),
many chains across them, and session written over another array of the call."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_08565_amd import smetric as S
from tests.parity import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(dev):
    yield


def _check(keys, blk_off, user, turn):
    nb = int(blk_off[-1])
    d_keys = to_dev(keys.view(np.int64) if nb else np.zeros(1, np.int64)).view(torch.uint64)
    gp, gs = S.sessions(d_keys, to_dev(blk_off), nb, to_dev(user.astype(np.uint32)), to_dev(turn.astype(np.int32)))
    op, os_ = oracle.sessions(keys, blk_off, user.astype(np.uint32), turn.astype(np.int32))
    assert np.array_equal(gp.cpu().numpy(), op) and np.array_equal(gs.cpu().numpy(), os_)
    return op


@pytest.mark.parametrize("R,longest", [(1, 3), (2, 70), (33, 1100), (700, 513), (131_072, 3), (131_073, 3),
                                       (1, 400), (2, 400), (300, 140), (131_072, 140), (131_073, 140)])
def test_streams(R, longest):
    rng = np.random.default_rng(R)
    n_stream = max(1, R // 6)
    stream = rng.integers(0, n_stream, R)
    nb = rng.integers(0, longest + 1, R)
    turn = np.where(rng.random(R) < 0.1, 0, nb * 5 // (longest + 1))
    if R > 2:
        edge = np.array([e for e in (0, 1, 63, 64, 65, 511, 512, 513) if e <= longest])
        nb = np.where(rng.random(R) < 0.3, rng.choice(edge, R), nb)
    blk_off = np.zeros(R + 1, np.int64)
    blk_off[1:] = np.cumsum(nb)
    at = np.arange(int(blk_off[-1])) - np.repeat(blk_off[:-1], nb)
    pool = rng.integers(1, 2**63, (n_stream, longest + 1), dtype=np.int64).astype(np.uint64)
    op = _check(pool[np.repeat(stream, nb), at], blk_off, stream % 97, turn)
    assert R < 700 or (op >= 0).any()


@pytest.mark.parametrize("order", ["arrival", "reversed"])
def test_one_chain(order):
    R = 20_000
    turn = np.arange(R) if order == "arrival" else np.arange(R)[::-1].copy()
    op = _check(np.zeros(0, np.uint64), np.zeros(R + 1, np.int64), np.zeros(R, np.int64), turn)
    assert (op >= 0).sum() == (R - 1 if order == "arrival" else 0)


def test_chains_interleaved():
    """Forty users' chains, whose requests arrive in random order: a request's parent is the
    latest earlier one of the turn before, if any, so chains of all lengths run across the
    workgroups."""
    rng = np.random.default_rng(11)
    R = 40_000
    turn = np.minimum(np.arange(R) // 80 + rng.integers(-3, 4, R), 400).clip(0)
    op = _check(np.zeros(0, np.uint64), np.zeros(R + 1, np.int64), rng.integers(0, 40, R), turn)
    assert (op >= 0).sum() > R // 2


@pytest.mark.parametrize("over", ["turn", "user", "parent", "keys", "blk_off"])
@pytest.mark.parametrize("R", [33, 700, 20_000])
def test_session_written_over_another_array(R, over):
    """The session array may be one of the call's other arrays: it is written after the last
    read of them."""
    rng = np.random.default_rng(R)
    stream, nb = rng.integers(0, R // 6, R), rng.integers(60, 101, R)
    blk_off = np.zeros(R + 1, np.int64)
    blk_off[1:] = np.cumsum(nb)
    at = np.arange(int(blk_off[-1])) - np.repeat(blk_off[:-1], nb)
    keys = rng.integers(1, 2**63, (R // 6, 100), dtype=np.int64).astype(np.uint64)[np.repeat(stream, nb), at]
    user, turn = (stream % 97).astype(np.uint32), ((nb - 60) // 8).astype(np.int32)
    op, os_ = oracle.sessions(keys, blk_off, user, turn)
    assert (op >= 0).any()
    d_keys, d_user, d_turn, d_off = to_dev(keys.view(np.int64)), to_dev(user.view(np.int32)), to_dev(turn), to_dev(blk_off)
    parent = torch.empty(R, dtype=torch.int32, device="cuda")
    session = {"turn": d_turn, "user": d_user, "parent": parent, "keys": d_keys.view(torch.int32)[:R],
               "blk_off": d_off.view(torch.int32)[:R]}[over]
    gp, gs = S.sessions(d_keys.view(torch.uint64), d_off, len(at), d_user.view(torch.uint32), d_turn,
                        parent=parent, session=session)
    assert np.array_equal(gs.cpu().numpy(), os_)
    assert over == "parent" or np.array_equal(gp.cpu().numpy(), op)
