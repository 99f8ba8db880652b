"""The probed path and the insert's paths against the oracle at the sizes where they part:
refreshes of entries many requests share, batches around the limits of the one-workgroup
insert and of the direct form, and few long requests."""
import numpy as np
import pytest
import torch

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


def _sized(rng, R, nb, shared, block=16):
    """R prompts of nb blocks in all (some empty), those long enough starting with one of
    three prefixes of `shared` blocks; a few prompts are copies of an earlier one."""
    cut = np.sort(rng.integers(0, nb + 1, R - 1)) if R > 1 else np.zeros(0, np.int64)
    n = np.diff(np.concatenate([[0], cut, [nb]]))
    pre = [rng.integers(0, W.VOCAB, block * shared, dtype=np.int32) for _ in range(3)]
    ps = []
    for r in range(R):
        p = rng.integers(0, W.VOCAB, block * int(n[r]), dtype=np.int32)
        k = min(len(p), block * shared)
        p[:k] = pre[int(rng.integers(0, 3))][:k]
        if r and rng.random() < 0.1 and len(ps[r - 1]) >= len(p):
            p = ps[r - 1][: len(p)].copy()
        ps.append(np.concatenate([p, rng.integers(0, W.VOCAB, int(rng.integers(0, block)), dtype=np.int32)]))
    off = np.zeros(R + 1, np.int64)
    off[1:] = np.cumsum([len(p) for p in ps])
    return np.concatenate(ps), off


@pytest.mark.parametrize("probed", [False, True])
@pytest.mark.parametrize("R,nb", [(1, 0), (1, 1), (1, 1023), (3, 1024), (64, 1025), (1023, 4095), (1024, 4096),
                                  (1025, 4096), (40, 4097), (1, 4096), (70, 2047), (70, 2048), (70, 2049), (1024, 2048),
                                  (1025, 2048), (4, 2049), (5, 2559), (5, 2560), (8, 4095), (8, 4096), (1, 4097)])
def test_insert_around_the_small_batch_limits(R, nb, probed):
    """Batches of exactly R requests and nb blocks on few and on many instances (keys turning
    into bitmap records while pairs of theirs wait), entered three times on new targets with
    rising and falling epochs; then a batch that does not fit and one with a bad target,
    which change nothing."""
    rng = np.random.default_rng(1000 * R + nb)
    for I in (2, 40):
        pair = Pair(max(64, 3 * nb), I)
        toks, off = _sized(rng, R, nb, 12)
        d_boff, n, d_keys, okeys, blk_off = pair.hash_both(toks, off)
        assert n == nb
        say(f"  I={I} R={R} blocks={nb} probed={probed}")
        for epoch in (4, 6, 5):
            args = (rng.integers(0, I, R), rng.permutation(R), epoch)
            rc = insert_both(pair, probed, d_keys, d_boff, nb, okeys, blk_off, *args)
            assert rc == 0
            pair.compare_index(f"I={I} epoch {epoch}")
        bad = rng.integers(0, I, R)
        bad[-1] = I
        insert_both(pair, probed, d_keys, d_boff, nb, okeys, blk_off, bad, np.arange(R), 9)
        pair.compare_index(f"I={I} bad target")
        tight = Pair(max(1, nb // 2), I)
        insert_both(tight, probed, d_keys, d_boff, nb, okeys, blk_off, rng.integers(0, I, R), np.arange(R), 1)
        tight.compare_index(f"I={I} capacity {max(1, nb // 2)}")


@pytest.mark.parametrize("B,R,nb", [(16, 300, (1 << 18) - 1), (16, 300, 1 << 18), (16, 300, (1 << 18) + 1),
                                    (32, 9, 5000), (16, 20000, 5000), (16, 16384, 4097), (64, 70, 0)])
def test_probed_path_around_the_direct_form(B, R, nb):
    """The fused hash + partition, the lookup, the match and the insert on both sides of the
    direct form's limits -- blocks, requests with a flag of their own -- on an index that holds
    the first half of every prompt, then all of them: rows, index and the lookup's counts (the
    blocks before each request's first of no holder; direct: the rest as searched)."""
    from paper_2607_08565_amd import smetric as S
    rng = np.random.default_rng(nb + R)
    I = 24
    pair = Pair(3 * nb + 100, I, block=B)
    toks, off = _sized(rng, R, nb, 30, B)
    d_boff, n, d_keys, okeys, blk_off = pair.hash_both(toks, off)
    assert n == nb
    # enter the first half of every prompt, on several instances
    half = (np.diff(blk_off) + 1) // 2
    sel = np.repeat(blk_off[:-1] - np.concatenate([[0], np.cumsum(half)[:-1]]), half) + np.arange(half.sum())
    hoff = np.concatenate([[0], np.cumsum(half)]).astype(np.int64)
    hk = okeys[sel.astype(np.int64)]
    assert pair.insert_both(to_dev(hk if len(hk) else np.ones(1, np.uint64)), to_dev(hoff), len(hk), hk, hoff,
                            rng.integers(0, I, R), np.arange(R), 1) == 0
    for epoch in (2, 3):
        say(f"  B={B} R={R} blocks={nb} epoch {epoch}")
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        keys, state = pair.gix.hash_partition(to_dev(toks if len(toks) else np.zeros(1, np.int32)), to_dev(off), d_boff, nb,
                                              block_size=B, status=status)
        assert int(status.item()) == 0 and np.array_equal(keys[:nb].cpu().numpy(), okeys)
        for _ in range(2):  # a lookup may run again on its state
            pair.gix.probe_lookup(state, keys, d_boff, nb)
        om = pair.oix.match(okeys, blk_off)
        assert np.array_equal(pair.gix.match_probed(state, keys, d_boff, nb).cpu().numpy(), om)
        probed, searched = S.Index.probe_stats(state, nb)
        n_r = np.diff(blk_off)  # blocks before each request's first of no holder
        first = n_r.copy()
        miss = np.nonzero(~np.isin(okeys, pair.oix.dump()[0]))[0]
        of, at = np.unique(np.repeat(np.arange(R), n_r)[miss], return_index=True)
        first[of] = miss[at] - blk_off[of]
        assert probed == first.sum()
        if nb <= 1 << 18:
            assert searched == nb - probed
        else:
            assert np.count_nonzero(n_r) <= searched <= 4 * 20 * R
        inst, sess = rng.integers(0, I, R).astype(np.int32), rng.permutation(R).astype(np.uint32)
        pair.gix.insert_probed(state, R, nb, to_dev(inst), to_dev(sess), epoch)
        assert pair.oix.insert(okeys, blk_off, inst, sess, epoch) == 0
        pair.compare_index(f"epoch {epoch}")


@pytest.mark.parametrize("R,nb", [(1, 1 << 16), (2, 1 << 16), (1, 1 << 18), (2, 1 << 18)])
def test_few_long_requests(R, nb):
    """One or two requests with all of the batch's blocks, part of them held: rows, index, and a
    lookup whose time is that of the blocks, not of the longest request (one workgroup for
    it took 50 to 140 times as long as the same blocks in 1,024 requests)."""
    rng = np.random.default_rng(nb + R)
    pair = Pair(3 * nb, 8)
    toks, off = _sized(rng, R, nb, 30)
    d_boff, n, d_keys, okeys, blk_off = pair.hash_both(toks, off)
    hoff = np.stack([blk_off[:-1], (blk_off[:-1] + blk_off[1:]) // 2], 1)
    hk = np.concatenate([okeys[a:b] for a, b in hoff])
    ho = np.concatenate([[0], np.cumsum(hoff[:, 1] - hoff[:, 0])]).astype(np.int64)
    assert pair.insert_both(to_dev(hk), to_dev(ho), len(hk), hk, ho, np.arange(R), np.arange(R), 1) == 0
    for epoch in (2, 3):
        say(f"  R={R} blocks={nb} epoch {epoch}")
        state = pair.gix.probe(d_keys, d_boff, nb)
        om = pair.oix.match(okeys, blk_off)
        assert np.array_equal(pair.gix.match_probed(state, d_keys, d_boff, nb).cpu().numpy(), om)
        assert np.array_equal(pair.gix.match(d_keys, d_boff, nb).cpu().numpy(), om)
        inst, sess = rng.integers(0, 8, R).astype(np.int32), np.arange(R, dtype=np.uint32)
        pair.gix.insert_probed(state, R, nb, to_dev(inst), to_dev(sess), epoch)
        assert pair.oix.insert(okeys, blk_off, inst, sess, epoch) == 0
        pair.compare_index(f"epoch {epoch}")

    def lookup_us(d_off):
        st = pair.gix.probe(d_keys, d_off, nb)
        t = []
        for _ in range(9):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            pair.gix.probe_lookup(st, d_keys, d_off, nb)
            e[1].record()
            torch.cuda.synchronize()
            t.append(e[0].elapsed_time(e[1]) * 1e3)
        return sorted(t)[4]

    few, many = lookup_us(d_boff), lookup_us(to_dev(np.arange(1025, dtype=np.int64) * (nb // 1024)))
    say(f"  lookup: {few:.0f} us, as 1,024 requests {many:.0f} us")
    assert few < 5 * many


@pytest.mark.parametrize("probed", [False, True])
@pytest.mark.parametrize("R,shared,own,n_inst", [(16384, 16, 0, 1), (4000, 60, 5, 3), (2000, 128, 0, 40)])
def test_pairs_entered_by_many_requests(R, shared, own, n_inst, probed):
    """A new prefix that thousands of requests enter on one or a few instances, with and without
    blocks of their own: each pair takes the lowest request's session.  Pairs met that often
    cost no more than as many distinct ones (one atomic each on the same words: 3 times)."""
    rng = np.random.default_rng(R + n_inst)
    nb = R * (shared + own)
    keys = rng.integers(1, 2**63, (R, shared + own), dtype=np.int64).astype(np.uint64)
    keys[:, :shared] = keys[0, :shared]
    keys = keys.reshape(-1)
    blk_off = np.arange(R + 1, dtype=np.int64) * (shared + own)
    pair = Pair(nb + 1000, 40)
    inst, sess = rng.integers(0, n_inst, R).astype(np.int32), rng.permutation(R).astype(np.uint32)
    d_keys, d_off, d_inst, d_sess = to_dev(keys), to_dev(blk_off), to_dev(inst), to_dev(sess)
    assert insert_both(pair, probed, d_keys, d_off, nb, keys, blk_off, inst, sess, 3) == 0
    pair.compare_index(f"R={R} shared={shared} own={own} instances={n_inst} probed={probed}")
    if own or n_inst > 1:
        return
    empty = pair.S.Index(nb + 1000, 40)
    snap = empty.snapshot()

    def insert_us(k):
        t = []
        for _ in range(9):
            empty.restore(snap)
            state = empty.probe(k, d_off, nb) if probed else None
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            if probed:
                empty.insert_probed(state, R, nb, d_inst, d_sess, 1)
            else:
                empty.insert(k, d_off, nb, d_inst, d_sess, 1)
            e[1].record()
            torch.cuda.synchronize()
            t.append(e[0].elapsed_time(e[1]) * 1e3)
        return sorted(t)[4]

    same, distinct = insert_us(d_keys), insert_us(to_dev(rng.integers(1, 2**63, nb, dtype=np.int64).astype(np.uint64)))
    say(f"  insert probed={probed}: {same:.0f} us, distinct pairs {distinct:.0f} us")
    assert same < 1.5 * distinct
