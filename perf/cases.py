"""The workloads this framework is timed on: what a router built on it does, through its
public calls, from one agent's session to the throughput configuration.

A case is a dict of plain values with a `kind`:
  replay     a closed-loop replay of agent sessions from an empty index: every turn's prompts
             are hashed, matched, routed and entered on their targets; optionally a share of
             the oldest entries is evicted after each turn.  `path` "plain" makes the
             self-contained calls (hash_blocks, match, insert), "probed" the batched ones
             (hash_partition, probe_lookup, match_probed, insert_probed); `rule` "batch" is
             the snapshot rule, "online" the one-request-at-a-time rule.
  saved      batches routed from a saved index: the snapshot is restored, then every batch
             takes the batched path (the throughput benchmark's step).
  policies   every batch rule on one batch's matched rows -- SMetric's, the colocation rule,
             the load-aware filter, the five comparison scorers -- and the load imbalance of
             SMetric's placement.
  online     requests routed one at a time; `coloc` adds the colocation rule.
  sessions   an anonymised trace: its prompts hashed, its sessions reconstructed.
  evict      a saved index restored, 5 % of it evicted (in place), a third of the rest
             evicted (a rebuild), a batch matched after each.

Every output is a whole number (keys, hit lengths, targets, branch codes, loads), so results
are compared exactly.  The index's bytes are not returned: concurrent claims settle the slots
in an order that differs from run to run; what it holds shows in the rows matched after it.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_08565_amd import smetric as S
from paper_2607_08565_amd.workload import DEFAULT_PARAMS, NO_DECODE, Q_UNIT_NS, VOCAB

DEV = "cuda"


def listed():
    return [
        # one agent in front of a small deployment: eight turns, one request per call
        dict(name="session_alone", kind="replay", sessions=1, turns=8, instances=8, first=1024, grow_lo=128,
             grow_hi=1024, cap=65536, prefixes=1, prefix=512, block=16, path="plain", rule="batch", evict=0),
        # the tiny trace: 64 sessions x 4 turns on 8 instances, a shared 512-token prefix
        dict(name="tiny_fleet", kind="replay", sessions=64, turns=4, instances=8, first=1024, grow_lo=128,
             grow_hi=1024, cap=65536, prefixes=4, prefix=512, block=16, path="probed", rule="batch", evict=0),
        # engines with 64-token pages, routed through the self-contained calls
        dict(name="direct_page64", kind="replay", sessions=500, turns=6, instances=200, first=4001, grow_lo=256,
             grow_hi=4096, cap=65536, prefixes=8, prefix=2048, block=64, path="plain", rule="batch", evict=0),
        # the mid fleet: 64 instances, 4,096 sessions x 10 turns
        dict(name="mid_fleet", kind="replay", sessions=4096, turns=10, instances=64, first=4096, grow_lo=256,
             grow_hi=4096, cap=65536, prefixes=16, prefix=2048, block=16, path="probed", rule="batch", evict=0),
        # long-context coding agents (the first 12 turns), loads updated request by request
        dict(name="long_context", kind="replay", sessions=1024, turns=12, instances=256, first=16384, grow_lo=512,
             grow_hi=8192, cap=131072, prefixes=4, prefix=8192, block=16, path="probed", rule="online", evict=0),
        # one 32,768-token prefix shared by everybody, 5 % LRU eviction after every turn
        dict(name="divergent_evict", kind="replay", sessions=8192, turns=4, instances=128, first=41472, grow_lo=512,
             grow_hi=512, cap=65536, prefixes=1, prefix=32768, block=16, path="probed", rule="batch", evict=5),
        # the throughput configuration, two batches from a saved index of 200M entries
        dict(name="throughput", kind="saved", requests=16384, instances=1024, batches=2, median=24576, entries=200000000,
             slots=1 << 28),
        # what each rule would do with one batch of the throughput configuration
        dict(name="policies", kind="policies", requests=16384, instances=1024, median=24576, first_pct=10),
        # requests routed one at a time: a fleet's batch with a tenth of the sessions starting
        dict(name="online_route", kind="online", coloc=False, requests=16384, instances=1024, median=24576,
             first_pct=10),
        dict(name="online_coloc", kind="online", coloc=True, requests=4096, instances=256, median=16384, first_pct=10),
        # session reconstruction on 1,024 users' anonymised trace
        dict(name="sessions", kind="sessions", users=1024, per_user=4, turns=8, first=2048, prefix=1024, grow_lo=256,
             grow_hi=2048, block=16),
        # LRU eviction of a large index: in place, then by rebuild
        dict(name="evict_large", kind="evict", entries=50000000, instances=1024, requests=2048, median=24576),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["replay", "saved", "policies", "online", "sessions", "evict"], [10, 2, 2, 3, 1, 1])[0]
    if kind == "replay":
        path = rng.choice(["plain", "probed"])
        sessions = _logint(rng, 1, 400) if path == "plain" else _logint(rng, 8, 8192)
        first = _logint(rng, 256, 32768)
        grow_lo = _logint(rng, 64, 1024)
        grow_hi = grow_lo + _logint(rng, 64, 6000)
        # a replay stays within about 400M tokens
        fit = int(400e6 / (sessions * (first + 4 * grow_hi)))
        turns = max(2, min(rng.randint(2, 12), fit))
        if sessions * turns * (first + turns * grow_hi / 2) > 500e6:
            sessions = max(1, int(500e6 / (turns * (first + turns * grow_hi / 2))))
        block = rng.choice([16, 16, 16, 16, 32, 64, 128])
        return dict(kind="replay", sessions=sessions, turns=turns, instances=_logint(rng, 1, 1024), first=first,
                    grow_lo=grow_lo, grow_hi=grow_hi, cap=131072, prefixes=_logint(rng, 1, 64),
                    prefix=_logint(rng, 64, first), block=block, path=path,
                    rule=rng.choice(["batch", "batch", "online"]), evict=rng.choice([0, 0, 0, 5, 10]))
    if kind == "saved":
        entries = _logint(rng, 2000000, 180000000)
        requests = min(_logint(rng, 256, 16384), max(256, entries // 2500))
        median = _logint(rng, 4096, 24576)
        slots = 0 if rng.random() < 0.5 else int((entries + 3 * requests * median // 16 * 1.4) * rng.uniform(1.15, 1.6))
        return dict(kind="saved", requests=requests, instances=_logint(rng, 8, 2048), batches=rng.choice([1, 2]),
                    median=median, entries=entries, slots=slots)
    if kind == "policies":
        return dict(kind="policies", requests=_logint(rng, 16, 16384), instances=_logint(rng, 8, 2048),
                    median=_logint(rng, 2048, 32768), first_pct=rng.randint(0, 40))
    if kind == "online":
        coloc = rng.random() < 0.5
        return dict(kind="online", coloc=coloc, requests=_logint(rng, 16, 4096 if coloc else 16384),
                    instances=_logint(rng, 8, 1024), median=_logint(rng, 2048, 32768), first_pct=rng.randint(0, 40))
    if kind == "sessions":
        return dict(kind="sessions", users=_logint(rng, 4, 1500), per_user=rng.randint(1, 4), turns=rng.randint(2, 8),
                    first=_logint(rng, 1024, 4096), prefix=rng.choice([256, 512, 1000]), grow_lo=128,
                    grow_hi=_logint(rng, 256, 3000), block=rng.choice([16, 16, 32]))
    return dict(kind="evict", entries=_logint(rng, 500000, 50000000), instances=_logint(rng, 8, 1024),
                requests=_logint(rng, 64, 2048), median=_logint(rng, 4096, 24576))


# ---------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------
def _rngs(case, seed):
    """Streams for the shape (lengths: the case's own, so every seed's outputs have the same
    sizes), the host's draws and the device's draws."""
    own = [int(v) if isinstance(v, (bool, int, float)) else len(v) for k, v in sorted(case.items()) if k != "name"]
    return (np.random.default_rng([0x5A9E] + own), np.random.default_rng([0x51E7, int(seed)]),
            torch.Generator(device=DEV).manual_seed(int(seed) * 2 + 1))


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _tokens(g, *shape):
    return torch.randint(0, VOCAB, shape, generator=g, device=DEV, dtype=torch.int32)


def _offsets(lens):
    off = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    return off


def _loads(rng, instances):
    """Queued prefill of a fleet: Poisson(50) units of 20 ms."""
    return _dev(rng.poisson(50, instances).astype(np.int64) * Q_UNIT_NS)


def _zipf(rng, n, s, size):
    p = np.arange(1, n + 1, dtype=np.float64) ** -s
    return rng.choice(n, size=size, p=p / p.sum())


def _turn_lens(case, rng):
    """int64[turns, sessions]: prompt lengths; every turn extends the one before it."""
    n, T = case["sessions"], case["turns"]
    lens = np.zeros((T, n), np.int64)
    # first turns spread around `first`, none shorter than the shared prefix
    lens[0] = np.maximum(case["prefix"], rng.integers(case["first"] * 3 // 4, case["first"] * 5 // 4 + 1, n))
    for t in range(1, T):
        lens[t] = np.minimum(case["cap"], lens[t - 1] + rng.integers(case["grow_lo"], case["grow_hi"] + 1, n))
    return lens


def _prepare_replay(case, seed):
    shape, rng, g = _rngs(case, seed)
    n, T, I, B = case["sessions"], case["turns"], case["instances"], case["block"]
    lens = _turn_lens(case, shape)
    stream = _tokens(g, n, int(lens[-1].max()))
    pre = _tokens(g, case["prefixes"], case["prefix"])
    which = _dev(_zipf(rng, case["prefixes"], 1.1, n))
    stream[:, :case["prefix"]] = pre[which]
    col = torch.arange(stream.shape[1], device=DEV, dtype=torch.int32)
    turns, nb_max, nb_sum = [], 1, 0
    for t in range(T):
        off = _offsets(lens[t])
        blk, nb = S.block_offsets(off, B)
        L = _dev(lens[t].astype(np.int32))
        turns.append(dict(
            tokens=torch.cat([stream[s:s + 512][col < L[s:s + 512, None]] for s in range(0, n, 512)]),
            tok_off=_dev(off), blk_off=_dev(blk), nb=nb, prompt_len=L,
            hist=_dev((lens[t - 1] if t else np.zeros(n)).astype(np.int32)),
            turn=torch.full((n,), t, dtype=torch.int32, device=DEV), q=_loads(rng, I), rr=t * n))
        nb_max, nb_sum = max(nb_max, nb), nb_sum + nb
    # room for every session's last prompt twice (migrations leave copies) and one more batch
    capacity = 2 * (int((lens[-1] // B).sum()) + 64) + nb_max
    st = dict(case=case, turns=turns, capacity=capacity, session=torch.arange(n, dtype=torch.int32, device=DEV),
              params=dict(DEFAULT_PARAMS, block_size=B),
              mem=torch.empty(S.index_bytes(capacity, I), dtype=torch.uint8, device=DEV),
              keys=torch.empty(nb_max, dtype=torch.uint64, device=DEV),
              ws=torch.empty(S.insert_ws_bytes(nb_max), dtype=torch.uint8, device=DEV),
              probe=torch.empty(S.probe_ws_bytes(nb_max), dtype=torch.uint8, device=DEV),
              route_ws=torch.empty(S.route_seq_ws_bytes(n), dtype=torch.uint8, device=DEV),
              matched=torch.empty((T, n, I), dtype=torch.int32, device=DEV),
              target=torch.empty((T, n), dtype=torch.int32, device=DEV),
              branch=torch.empty((T, n), dtype=torch.uint8, device=DEV),
              q_out=torch.zeros((T, I), dtype=torch.int64, device=DEV))
    return st


def _run_replay(st):
    c = st["case"]
    n, I, B, keys, ws, probe = c["sessions"], c["instances"], c["block"], st["keys"], st["ws"], st["probe"]
    idx = S.Index(st["capacity"], I, mem=st["mem"])
    for t, b in enumerate(st["turns"]):
        m, nb = st["matched"][t], b["nb"]
        if c["path"] == "plain":
            S.hash_blocks(b["tokens"], b["tok_off"], b["blk_off"], nb, block_size=B, keys=keys)
            idx.match(keys, b["blk_off"], nb, matched=m)
        else:
            idx.hash_partition(b["tokens"], b["tok_off"], b["blk_off"], nb, block_size=B, keys=keys, state=probe)
            idx.probe_lookup(probe, keys, b["blk_off"], nb)
            idx.match_probed(probe, keys, b["blk_off"], nb, matched=m)
        if c["rule"] == "online":
            S.route_seq(m, b["prompt_len"], b["hist"], b["turn"], b["q"], st["params"], b["rr"],
                        target=st["target"][t], branch=st["branch"][t], q_out=st["q_out"][t], workspace=st["route_ws"])
        else:
            S.route(m, b["prompt_len"], b["hist"], b["turn"], b["q"], st["params"], b["rr"], target=st["target"][t],
                    branch=st["branch"][t])
        if c["path"] == "plain":
            idx.insert(keys, b["blk_off"], nb, st["target"][t], st["session"], t, workspace=ws)
        else:
            idx.insert_probed(probe, n, nb, st["target"][t], st["session"], t, workspace=ws)
        if c["evict"]:
            idx.evict(c["evict"], 100)
    # the last turn's keys begin with every earlier turn's
    out = dict(matched=st["matched"], target=st["target"], branch=st["branch"],
               keys=keys[:st["turns"][-1]["nb"]].view(torch.int64))
    return dict(out, q_out=st["q_out"]) if c["rule"] == "online" else out


def _fleet_batch(shape, rng, g, requests, instances, median, lmax=131072, prefixes=64, prefix=4096, sigma=0.6,
                 prior=0.7):
    """Prompts of a large fleet: lognormal lengths, 70 % of each prompt's blocks its session's
    prior turn, which starts with one of 64 shared prefixes."""
    L = np.clip(np.rint(shape.lognormal(math.log(median), sigma, requests)), 1024, lmax).astype(np.int64)
    off = _offsets(L)
    blk, nb = S.block_offsets(off, 16)
    tokens = _tokens(g, int(off[-1]))
    pre = _tokens(g, prefixes, prefix)
    which = _dev(_zipf(rng, prefixes, 1.2, requests))
    at, Ld, col = _dev(off[:-1]), _dev(L), torch.arange(prefix, device=DEV)
    for s in range(0, requests, 2048):
        inside = col < Ld[s:s + 2048, None]
        tokens[(at[s:s + 2048, None] + col)[inside]] = pre[which[s:s + 2048]][inside]
    prior_blocks = (prior * (L // 16)).astype(np.int64)
    return dict(tokens=tokens, tok_off=_dev(off), blk_off=_dev(blk), nb=nb, L=L, prior=prior_blocks, blk_host=blk,
                prompt_len=_dev(L.astype(np.int32)), hist=_dev((prior_blocks * 16).astype(np.int32)),
                home=_dev(rng.integers(0, instances, requests).astype(np.int32)))


def _enter_prior(idx, b, session, ws):
    """The batch's prior turns on their home instances (epoch 0)."""
    keys = S.hash_blocks(b["tokens"], b["tok_off"], b["blk_off"], b["nb"])
    pb = b["prior"]
    off = _offsets(pb)
    pbd = _dev(pb)
    pos = torch.arange(int(off[-1]), device=DEV) + torch.repeat_interleave(_dev(b["blk_host"][:-1] - off[:-1]), pbd)
    pk = keys.view(torch.int64)[pos].view(torch.uint64)
    idx.insert(pk, _dev(off), int(off[-1]), b["home"], session, 0, workspace=ws)


def _enter_filler(idx, g, instances, n, ws, chunk, epochs=1):
    """n entries of other sessions: random keys no prompt has, spread over `epochs` epochs."""
    done, k = 0, 0
    while done < n:
        m = min(chunk, n - done)
        r = -(-m // 64)
        keys = torch.randint(-(1 << 63) + 1, (1 << 63) - 1, (m,), generator=g, device=DEV, dtype=torch.int64)
        keys = torch.where((keys == 0) | (keys == -1), 12345 + torch.arange(m, device=DEV), keys).view(torch.uint64)
        off = torch.clamp(torch.arange(r + 1, device=DEV, dtype=torch.int64) * 64, max=m)
        inst = torch.randint(0, instances, (r,), generator=g, device=DEV, dtype=torch.int32)
        idx.insert(keys, off, m, inst, torch.full((r,), (1 << 24) - 1, dtype=torch.int32, device=DEV), k % epochs,
                   workspace=ws)
        done, k = done + m, k + 1


def _prepare_saved(case, seed):
    shape, rng, g = _rngs(case, seed)
    R, I = case["requests"], case["instances"]
    batches = [_fleet_batch(shape, rng, g, R, I, case["median"]) for _ in range(case["batches"])]
    nb_max = max(b["nb"] for b in batches)
    capacity = case["entries"] + nb_max + sum(b["nb"] - int(b["prior"].sum()) for b in batches[1:])
    slots = case["slots"]
    if slots:  # as full as asked, within what the library takes
        slots = max(slots, int(capacity * 1.04 * 16 / 15) + 4096)
    chunk = min(16000000, case["entries"])
    ws = torch.empty(S.insert_ws_bytes(max(nb_max, chunk)), dtype=torch.uint8, device=DEV)
    idx = S.Index(capacity, I, n_slots=slots)
    for k, b in enumerate(batches):
        b.update(session=torch.arange(R, dtype=torch.int32, device=DEV) + k * R, q=_loads(rng, I), rr=k * R)
        _enter_prior(idx, b, b["session"], ws)
    n, status = idx.stats()
    if status or n > case["entries"]:
        raise RuntimeError("the prior turns need more than the case's entries: %d entries, status %d" % (n, status))
    _enter_filler(idx, g, I, case["entries"] - n, ws, chunk)
    T = case["batches"]
    return dict(case=case, idx=idx, batches=batches, snap=idx.snapshot(),
                ws=torch.empty(S.insert_ws_bytes(nb_max), dtype=torch.uint8, device=DEV),
                probe=torch.empty(S.probe_ws_bytes(nb_max), dtype=torch.uint8, device=DEV),
                keys=[torch.empty(b["nb"], dtype=torch.uint64, device=DEV) for b in batches],
                turn=torch.ones(R, dtype=torch.int32, device=DEV),
                matched=torch.empty((T, R, I), dtype=torch.int32, device=DEV),
                target=torch.empty((T, R), dtype=torch.int32, device=DEV),
                branch=torch.empty((T, R), dtype=torch.uint8, device=DEV))


def _run_saved(st):
    idx, probe = st["idx"], st["probe"]
    idx.restore(st["snap"])
    for k, b in enumerate(st["batches"]):
        m, nb, keys = st["matched"][k], b["nb"], st["keys"][k]
        idx.hash_partition(b["tokens"], b["tok_off"], b["blk_off"], nb, keys=keys, state=probe)
        idx.probe_lookup(probe, keys, b["blk_off"], nb)
        idx.match_probed(probe, keys, b["blk_off"], nb, matched=m)
        S.route(m, b["prompt_len"], b["hist"], st["turn"], b["q"], DEFAULT_PARAMS, b["rr"], target=st["target"][k],
                branch=st["branch"][k])
        idx.insert_probed(probe, st["case"]["requests"], nb, st["target"][k], b["session"], k + 1, workspace=st["ws"])
    return dict(matched=st["matched"], target=st["target"], branch=st["branch"],
                keys=[k.view(torch.int64) for k in st["keys"]])


def _rows(case, shape, rng, g):
    """Matched rows and route inputs of a fleet's batch: follow-ups hold 70 % of their prompt
    on one instance and a shared prefix on many, first turns the prefix alone."""
    R, I = case["requests"], case["instances"]
    L = np.clip(np.rint(shape.lognormal(math.log(case["median"]), 0.6, R)), 1024, 131072).astype(np.int64)
    first = rng.random(R) * 100 < case["first_pct"]
    prior = np.where(first, 0, 0.7 * (L // 16)).astype(np.int32)
    # a prefix of up to 4,096 tokens, held by a share of the instances that its use sets
    share = _dev((rng.random(R) ** 3).astype(np.float32))
    pre = _dev(np.minimum(rng.integers(16, 257, R), L // 16).astype(np.int32))
    m = torch.where(torch.rand((R, I), generator=g, device=DEV) < share[:, None], pre[:, None], 0).to(torch.int32)
    home = _dev(rng.integers(0, I, R).astype(np.int64))
    r = torch.arange(R, device=DEV)
    m[r, home] = torch.maximum(m[r, home], _dev(prior))
    slack = rng.integers(0, 3_000_000_000, I).astype(np.int64)
    slack[rng.random(I) < 0.3] = NO_DECODE
    return dict(matched=m, prompt_len=_dev(L.astype(np.int32)), hist=_dev((prior * 16).astype(np.int32)),
                turn=_dev((~first).astype(np.int32)), q=_loads(rng, I), slack=_dev(slack),
                running=_dev(rng.poisson(8, I).astype(np.int32)))


def _prepare_policies(case, seed):
    shape, rng, g = _rngs(case, seed)
    R, I = case["requests"], case["instances"]
    st = dict(_rows(case, shape, rng, g), case=case)
    t0 = np.sort(rng.integers(0, 600_000, R)).astype(np.int64)  # arrivals over ten minutes, ms
    st.update(target=torch.empty((8, R), dtype=torch.int32, device=DEV),
              branch=torch.empty((8, R), dtype=torch.uint8, device=DEV), t0=_dev(t0),
              t1=_dev(t0 + rng.integers(1_000, 40_000, R)), load=_dev(rng.integers(1, 1 << 40, I)),
              q_tok=_dev(rng.poisson(50, I).astype(np.int64) * 200))
    return st


def _run_policies(st):
    T, B = st["target"], st["branch"]
    a = (st["matched"], st["prompt_len"], st["hist"], st["turn"], st["q"])
    S.route(*a, DEFAULT_PARAMS, 7, target=T[0], branch=B[0])
    S.route_coloc(*a, st["slack"], st["running"], DEFAULT_PARAMS, 7, target=T[1], branch=B[1])
    S.route_loadaware(*a, st["load"], (1, 4), DEFAULT_PARAMS, 7, target=T[2], branch=B[2])
    for k in range(5):
        S.route_score(k, st["matched"], st["prompt_len"], st["q_tok"], st["running"], 16, (9, 10), 7, target=T[3 + k],
                      branch=B[3 + k])
    total, top, bad = S.imbalance(T[0], st["t0"], st["t1"], st["case"]["instances"], 30_000, 22)
    return dict(target=T, branch=B, total=total, top=top, bad=bad)


def _prepare_online(case, seed):
    shape, rng, g = _rngs(case, seed)
    R, I = case["requests"], case["instances"]
    need = S.route_seq_coloc_ws_bytes(R, I) if case["coloc"] else S.route_seq_ws_bytes(R)
    return dict(_rows(case, shape, rng, g), case=case, ws=torch.empty(need, dtype=torch.uint8, device=DEV))


def _run_online(st):
    a = (st["matched"], st["prompt_len"], st["hist"], st["turn"], st["q"])
    if st["case"]["coloc"]:
        target, branch, q, n = S.route_seq_coloc(*a, st["slack"], st["running"], DEFAULT_PARAMS, 3, workspace=st["ws"])
        return dict(target=target, branch=branch, q=q, n=n)
    target, branch, q = S.route_seq(*a, DEFAULT_PARAMS, 3, workspace=st["ws"])
    return dict(target=target, branch=branch, q=q)


def _prepare_sessions(case, seed):
    """Users with several sessions that start with the user's own system prefix; 5 % of the
    turns rewrite the prompt, 3 % are sent twice; requests in arrival order."""
    shape, rng, g = _rngs(case, seed)
    n, T = case["users"] * case["per_user"], case["turns"]
    user_of = np.repeat(np.arange(case["users"]), case["per_user"])
    grow = shape.integers(case["grow_lo"], case["grow_hi"] + 1, (n, T))
    compact = (shape.random((n, T)) < 0.05) & (np.arange(T) > 0)
    retry = shape.random((n, T)) < 0.03
    at = rng.uniform(0, 1000, n)[:, None] + np.cumsum(rng.exponential(5.0, (n, T)), 1)
    lens = np.zeros((n, T), np.int64)
    start = np.zeros((n, T), np.int64)  # where in the session's stream the turn's prompt begins
    lens[:, 0] = np.maximum(case["first"], case["prefix"])
    for t in range(1, T):
        end = start[:, t - 1] + lens[:, t - 1]
        start[:, t] = np.where(compact[:, t], end, start[:, t - 1])
        lens[:, t] = np.where(compact[:, t], 1024, lens[:, t - 1]) + grow[:, t]
    stream = _tokens(g, n, int((start + lens).max()))
    stream[:, :case["prefix"]] = _tokens(g, case["users"], case["prefix"])[_dev(user_of)]
    s, t = np.nonzero(np.ones((n, T), bool))
    s, t = np.concatenate([s, s[retry.ravel()]]), np.concatenate([t, t[retry.ravel()]])
    when = at[s, t] + np.concatenate([np.zeros(n * T), np.full(int(retry.sum()), 1e-3)])
    order = np.argsort(when, kind="stable")
    s, t = s[order], t[order]
    L = lens[s, t]
    off = _offsets(L)
    blk, nb = S.block_offsets(off, case["block"])
    tokens = torch.empty(int(off[-1]), dtype=torch.int32, device=DEV)
    base = _dev(s.astype(np.int64) * stream.shape[1] + start[s, t] - off[:-1])
    flat, R = stream.view(-1), len(L)
    for a in range(0, R, 4096):
        z = min(R, a + 4096)
        rep = torch.repeat_interleave(base[a:z], _dev(L[a:z]))
        tokens[off[a]:off[z]] = flat[rep + torch.arange(int(off[a]), int(off[z]), device=DEV)]
    return dict(case=case, tokens=tokens, tok_off=_dev(off), blk_off=_dev(blk), nb=nb,
                user=_dev(user_of[s].astype(np.uint32)), turn=_dev(t.astype(np.int32)),
                keys=torch.empty(max(nb, 1), dtype=torch.uint64, device=DEV),
                ws=torch.empty(S.sessions_ws_bytes(R), dtype=torch.uint8, device=DEV))


def _run_sessions(st):
    S.hash_blocks(st["tokens"], st["tok_off"], st["blk_off"], st["nb"], block_size=st["case"]["block"], keys=st["keys"])
    parent, session = S.sessions(st["keys"], st["blk_off"], st["nb"], st["user"], st["turn"], workspace=st["ws"])
    return dict(parent=parent, session=session, keys=st["keys"].view(torch.int64))


def _prepare_evict(case, seed):
    shape, rng, g = _rngs(case, seed)
    R, I, n = case["requests"], case["instances"], case["entries"]
    b = _fleet_batch(shape, rng, g, R, I, case["median"])
    prior = int(b["prior"].sum())
    capacity = max(n, 2 * prior) + b["nb"]
    chunk = 2000000
    ws = torch.empty(S.insert_ws_bytes(max(b["nb"], chunk)), dtype=torch.uint8, device=DEV)
    idx = S.Index(capacity, I)
    session = torch.arange(R, dtype=torch.int32, device=DEV)
    _enter_prior(idx, b, session, ws)
    _enter_filler(idx, g, I, max(n - prior, prior // 2), ws, chunk, epochs=9)
    keys = S.hash_blocks(b["tokens"], b["tok_off"], b["blk_off"], b["nb"])
    idx.evict(0, 1)  # takes the index's own scratch once, as a running router has it
    return dict(case=case, idx=idx, snap=idx.snapshot(), b=b, keys=keys,
                matched=torch.empty((2, R, I), dtype=torch.int32, device=DEV))


def _run_evict(st):
    idx, b = st["idx"], st["b"]
    idx.restore(st["snap"])
    idx.evict(1, 20)
    idx.match(st["keys"], b["blk_off"], b["nb"], matched=st["matched"][0])
    idx.evict(1, 3)
    idx.match(st["keys"], b["blk_off"], b["nb"], matched=st["matched"][1])
    return dict(matched=st["matched"])


_PREPARE = dict(replay=_prepare_replay, saved=_prepare_saved, policies=_prepare_policies, online=_prepare_online,
                sessions=_prepare_sessions, evict=_prepare_evict)
_RUN = dict(replay=_run_replay, saved=_run_saved, policies=_run_policies, online=_run_online, sessions=_run_sessions,
            evict=_run_evict)


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


def run(state):
    return _RUN[state["case"]["kind"]](state)


def work(case):
    """Bytes a pass cannot do without (nothing here is a contraction): tokens 4 B in, keys 8 B
    out, 4 B out per (request, instance), a 16 B entry read per block looked up and held, 8 B
    written per refreshed and 16 B per new entry; a restored index is read and written once, an
    evicted one read once.  The operations are the hash's: one multiply-add per token."""
    k = case["kind"]
    if k == "replay":
        n, T, I, B = case["sessions"], case["turns"], case["instances"], case["block"]
        grow = (case["grow_lo"] + case["grow_hi"]) / 2
        first = max(case["first"], case["prefix"])
        lens = [min(case["cap"], first + t * grow) for t in range(T)]
        tok = n * sum(lens)
        blocks, last = tok / B, n * lens[-1] / B
        held = blocks - last
        entries = last * (2.0 if case["evict"] else 1.0)
        return dict(bytes=4 * tok + 8 * blocks + 4.0 * T * n * I + 16 * held + 8 * held + 16 * last +
                    (16.0 * T * entries if case["evict"] else 0.0), flops=2 * tok)
    mean = case["median"] * math.exp(0.18) if "median" in case else 0
    if k == "saved":
        tok = case["batches"] * case["requests"] * mean
        blocks = tok / 16
        slots = case["slots"] or case["entries"] * 4 / 3
        return dict(bytes=4 * tok + 8 * blocks + 4.0 * case["batches"] * case["requests"] * case["instances"] +
                    0.7 * blocks * 24 + 0.3 * blocks * 16 + 32.0 * slots, flops=2 * tok)
    if k == "policies":
        return dict(bytes=4.0 * case["requests"] * case["instances"] + 8 * case["requests"] * 5,
                    flops=20.0 * case["requests"] * case["instances"])
    if k == "online":
        return dict(bytes=4.0 * case["requests"] * case["instances"] + case["requests"] * 17,
                    flops=4.0 * case["requests"] * case["instances"])
    if k == "sessions":
        n = case["users"] * case["per_user"]
        tok = n * sum(case["first"] + t * (case["grow_lo"] + case["grow_hi"]) / 2 for t in range(case["turns"])) * 0.95
        return dict(bytes=4 * tok + 16 * tok / case["block"], flops=2 * tok)
    tok = case["requests"] * mean
    slots = case["entries"] * 4 / 3
    return dict(bytes=32.0 * slots + 2 * 16.0 * slots + 16.0 * slots + 2 * (tok / 16 * 16 +
                4.0 * case["requests"] * case["instances"]), flops=tok)


def tolerance(case):
    return "exact"
