"""The batch rules whose scores are formed in doubles where those are exact, against the CPU
oracle's wide integers at the edges of that: queues, loads and products one below, at and one
above the bounds (2^49 and 2^52 for queues, 2^46 for a load that is summed, 2^53 for a
product), where neighbouring integers must still be told apart, with exact ties, one wide
value among small ones, and sizes around the 64-lane wave."""
import numpy as np
import pytest

import oracle
from paper_2607_08565_amd import workload as W
from tests.parity import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(dev):
    yield


def _same(got, want, what):
    for g, w in zip(got, want):
        assert np.array_equal(g.cpu().numpy(), w), what


def _rows(rng, R, I):
    L = rng.integers(0, 4000, R).astype(np.int32)
    m = np.minimum(rng.integers(0, 251, (R, I)), (L // 16)[:, None]).astype(np.int32)
    return m, L, rng.integers(0, 4000, R).astype(np.int32), rng.integers(0, 3, R).astype(np.int32)


def _near(rng, edge, I, wide):
    """Values within two of `edge` (a tie every few), or one of them among small ones."""
    v = rng.integers(0, 100, I) if wide == "one" else edge + rng.integers(-2, 3 if wide == "at" else 0, I)
    if wide == "one":
        v[rng.integers(0, I)] = edge + rng.integers(0, 2)
    return v.astype(np.int64)


@pytest.mark.parametrize("wide", ["below", "at", "one"])
@pytest.mark.parametrize("I", [1, 63, 65, 300])
def test_edges(I, wide):
    from paper_2607_08565_amd import smetric as S
    rng = np.random.default_rng(I)
    R = 200
    m, L, hist, turn = _rows(rng, R, I)
    d = [to_dev(x) for x in (m, L, hist, turn)]
    for p in (W.DEFAULT_PARAMS, dict(W.DEFAULT_PARAMS, c_att=0, c_lin=1)):
        for edge, n_hi in ((1 << 49, 1), (1 << 49, 8), (1 << 40, 1 << 12), (1 << 22, (1 << 31) - 1)):
            q = _near(rng, edge, I, wide)
            slack = (q + rng.integers(-3, 4, I)) // 2
            slack[::3] = oracle.NO_DECODE
            run = rng.integers(max(0, n_hi - 2), n_hi + 1, I).astype(np.int32)
            _same(S.route_coloc(*d, to_dev(q), to_dev(slack), to_dev(run), p, 3),
                  oracle.route_coloc(m, L, hist, turn, q, slack, run, p, 3), f"coloc {edge} {n_hi}")
        for edge in (1 << 46, 1 << 61):
            load = _near(rng, edge, I, wide)
            q = rng.integers(0, 1 << 40, I)
            for margin in ((0, 1), (1, 10**9), (1, 0)):
                _same(S.route_loadaware(*d, to_dev(q), to_dev(load), margin, p, 3),
                      oracle.route_loadaware(m, L, hist, turn, q, load, margin, p, 3), f"load-aware {edge} {margin}")
    for edge, l_hi in ((1 << 52, 2), (1 << 50, 8), (1 << 30, (1 << 23) + 1), (1 << 23, (1 << 31) - 1)):
        q = _near(rng, edge, I, wide)
        load = rng.integers(max(0, l_hi - 2), l_hi + 1, I).astype(np.int32)
        _same(S.route_score(2, d[0], d[1], to_dev(q), to_dev(load), 16, (0, 1), 3),
              oracle.route_score(2, m, L, q, load, 16, (0, 1), 3), f"product {edge} {l_hi}")
    for den in (10, 1 << 17, (1 << 31) - 1):
        for l_hi in (0, 1 << 10, 1 << 24, (1 << 31) - 1):
            load = rng.integers(max(0, l_hi - 2), l_hi + 1, I).astype(np.int32)
            for kind in (3, 4):
                lam = (den // 3, den)
                _same(S.route_score(kind, d[0], d[1], to_dev(q), to_dev(load), 16, lam, 3),
                      oracle.route_score(kind, m, L, q, load, 16, lam, 3), f"kind {kind} {lam} {l_hi}")
