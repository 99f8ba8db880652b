"""The online route against the oracle at the sizes where its kernel changes form: instance
counts around each form's slots, batches around windows of 64 requests and the 64 windows
looked ahead at, with runs of follow-ups of every length between requests that need a
scan, prevs shared within a run, out-of-domain requests, and loads on both sides of 2^50, and
each form with every load past it."""
import numpy as np
import pytest

import oracle
from paper_2607_08565_amd import workload as W
from tests.parity import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(dev):
    yield


def _batch(rng, R, I, scan_pct, prevs, big):
    """Follow-ups with their session on one of `prevs` instances (few: shared within a run),
    scan_pct % first turns or evicted sessions, 1 % out of domain."""
    L = rng.integers(64, 60000, R).astype(np.int32)
    m = np.zeros((R, I), np.int32)
    home = rng.integers(0, max(1, min(prevs, I)), R)
    m[np.arange(R), home] = L // 16 * rng.integers(5, 10, R) // 10
    for _ in range(2):
        j = rng.integers(0, I, R)
        m[np.arange(R), j] = np.maximum(m[np.arange(R), j], rng.integers(0, 4, R))
    m = np.minimum(m, (L // 16)[:, None]).astype(np.int32)
    kind = rng.random(R) * 100
    turn = (kind >= scan_pct / 2).astype(np.int32)
    hist = np.where((kind >= scan_pct / 2) & (kind < scan_pct), 1 << 20, L // 4).astype(np.int32)
    bad = rng.random(R) < 0.01
    L = np.where(bad, -1, L).astype(np.int32)
    m[bad] = 0
    q = rng.poisson(3, I).astype(np.int64) * W.Q_UNIT_NS
    if big:  # some loads at the double-precision scan's limit
        q[rng.integers(0, I, max(1, I // 4))] += (1 << 49) - int(2e9)
    return m, L, hist, turn, q


@pytest.mark.parametrize("I", [1, 2, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096])
def test_windows_of_runs_and_scans(I):
    from paper_2607_08565_amd import smetric as S
    sizes = [1, 63, 64, 65, 200] + ([4095, 4097] if I <= 64 else [4161] if I == 1024 else [700])
    for k, R in enumerate(sizes):
        rng = np.random.default_rng(9000 + 37 * I + R)
        scan_pct = (0, 3, 100, 30, 10, 1, 50)[(k + I) % 7]
        prevs = (1, 5, I, 40)[(k + I) % 4]
        batch = _batch(rng, R, I, scan_pct, prevs, big=(k + I) % 3 == 0)
        for over in ({}, dict(slack_num=3, slack_den=0), dict(slack_num=5, slack_den=7, slo_b=200_000_000)):
            p = dict(W.DEFAULT_PARAMS, **over)
            gt, gb, gq = S.route_seq(*[to_dev(x) for x in batch], p, 11)
            ot, ob, oq = oracle.route_seq(*batch, p, 11)
            gt, gb, gq = gt.cpu().numpy(), gb.cpu().numpy(), gq.cpu().numpy()
            bad = np.nonzero((gt != ot) | (gb != ob))[0]
            assert len(bad) == 0, (I, R, scan_pct, over, bad[:4], gt[bad[:4]], ot[bad[:4]], gb[bad[:4]], ob[bad[:4]])
            assert np.array_equal(gq, oq), (I, R, over)
        say(f"  I={I} R={R} scans {scan_pct}% prevs {prevs}: branches {np.bincount(ob, minlength=5)[:5].tolist()}")


@pytest.mark.parametrize("I", [7, 64, 100, 200, 500, 512, 1000, 2000, 2048, 4000])
def test_every_load_wide(I):
    """Scans in 128 bits at each form's slots, the last ones past the last instance."""
    from paper_2607_08565_amd import smetric as S
    rng = np.random.default_rng(I)
    m, L, hist, turn, _ = _batch(rng, 300, I, 60, I, False)
    q = (1 << 51) + rng.integers(0, 4, I) * W.Q_UNIT_NS
    got = S.route_seq(*[to_dev(x) for x in (m, L, hist, turn, q)], W.DEFAULT_PARAMS, 5)
    for g, o in zip(got, oracle.route_seq(m, L, hist, turn, q, W.DEFAULT_PARAMS, 5)):
        assert np.array_equal(g.cpu().numpy(), o)
