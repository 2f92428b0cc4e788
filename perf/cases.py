"""The workloads this library is measured on.

Three kinds of work, each through the public binding of ``libgx.so``:

* ``explore``: clear a table and explore one network into it, with a safety
  monitor or with the reachable set fetched afterwards where a case says so;
* ``put``: batches of packed state vectors through ``Table.find_or_put``;
* ``batch`` / ``serve``: many networks at once, through a batch handle or an
  exploration server.

Networks come from this repository's seeded generators (``workloads``).  The
seed of ``prepare`` picks where some processes start, offers a few transitions
twice, renames the local states and shuffles the transition lists: the product
keeps its size but for what a start no longer reaches, its levels change, and
so does every packed vector and with it every table position.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_1801_05857_amd as gx
import workloads as W

DEVICE = "cuda:0"


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest real call: a model of four small cyclic components,
        # explored as one edits it; latency and launches only
        {"name": "explore_tiny", "kind": "explore", "family": "tiny", "size": 4,
         "bucket": 32, "subgroup": 8},
        # a protocol ring (Table 1 of the paper at nine nodes): 118,098 states
        # in many thin levels
        {"name": "explore_ring9", "kind": "explore", "family": "ring", "size": 9,
         "bucket": 16, "subgroup": 4},
        # a small uneven model of two-word vectors, thousands of states
        {"name": "explore_random_small", "kind": "explore", "family": "served", "net_seed": 11,
         "log10": 4.0, "bucket": 16, "subgroup": 4},
        # an ordinary model: a few million states
        {"name": "explore_random_medium", "kind": "explore", "family": "served", "net_seed": 17,
         "log10": 6.5, "bucket": 16, "subgroup": 4},
        # the large random network of twelve 64-state processes (three-word
        # vectors), at 311 million reachable states
        {"name": "explore_random_large", "kind": "explore", "family": "large", "size": 6,
         "bucket": 16, "subgroup": 4, "slots": 1_000_000_000},
        # the same family at 250 thousand states with a safety property
        # watched, violations returned
        {"name": "explore_monitor", "kind": "explore", "family": "large", "size": 4,
         "bucket": 32, "subgroup": 4, "monitor": True},
        # the reachable set handed to the host for further analysis
        {"name": "explore_fetch_states", "kind": "explore", "family": "served", "net_seed": 7,
         "log10": 5.5, "bucket": 16, "subgroup": 4, "fetch": True},
        # a caller that feeds small batches of vectors: launch-bound
        {"name": "put_4096", "kind": "put", "words": 2, "keys": 4096, "seen": 0.5, "load": 0.25,
         "bucket": 32, "subgroup": 8, "in_flight": 1},
        # an odd-sized batch of three-word vectors, nine tenths of which the
        # table holds already: the mix an exploration makes
        {"name": "put_3word_seen", "kind": "put", "words": 3, "keys": 2_000_003, "seen": 0.9,
         "load": 0.6, "bucket": 16, "subgroup": 4, "in_flight": 1},
        # the isolated insertion at full size: 2^27 distinct two-word vectors,
        # then as many again of which seven in eight are stored
        {"name": "put_2p27", "kind": "put", "words": 2, "keys": 1 << 27, "seen": 0.875, "load": 0.5,
         "bucket": 32, "subgroup": 4, "in_flight": 1},
        # a family of uneven models explored together on resident tables
        {"name": "batch_96", "kind": "batch", "nets": 96, "net_seed": 11, "lo": 3.0, "hi": 6.5,
         "bucket": 16, "subgroup": 4, "graph": False},
        # requests of mixed width and size sent to a running server at once
        {"name": "serve_48", "kind": "serve", "nets": 48, "net_seed": 5, "lo": 3.5, "hi": 6.5,
         "bucket": 16, "subgroup": 4},
    ]


def draw(rng):
    kind = rng.choice(["explore", "explore", "explore", "put", "put", "batch", "serve"])
    bucket = rng.choice([16, 16, 32, 64])
    room = round(rng.uniform(1.5, 6.0), 2)  # table slots per reachable state, at least
    subgroup = rng.choice([8, 16]) if bucket == 64 else rng.choice([4, 4, 8])
    if kind == "explore":
        if rng.random() < 0.2:
            return {"kind": kind, "family": "ring", "size": rng.randint(4, 13), "bucket": bucket,
                    "subgroup": subgroup, "room": room}
        if rng.random() < 0.2:
            return {"kind": kind, "family": "large", "size": rng.randint(3, 4), "bucket": bucket,
                    "subgroup": subgroup, "room": room, "monitor": True,
                    "automaton": rng.randrange(1, 1 << 16)}
        return {"kind": kind, "family": "served", "net_seed": rng.randrange(1, 1 << 16),
                "log10": round(rng.uniform(3.0, 7.5), 3), "bucket": bucket, "subgroup": subgroup,
                "room": room}
    if kind == "put":
        w = rng.randint(1, 4)
        return {"kind": kind, "words": w, "keys": int(2 ** rng.uniform(6, 25)) | 1,
                "seen": round(rng.uniform(0.05, 0.97), 3),
                "load": round(rng.uniform(0.1, 0.8), 3), "bucket": bucket, "subgroup": subgroup,
                "in_flight": rng.choice([1, 1, 2])}
    lo = round(rng.uniform(3.0, 4.0), 2)
    case = {"kind": kind, "nets": rng.randint(8, 64), "net_seed": rng.randrange(1, 1 << 16),
            "lo": lo, "hi": round(rng.uniform(lo + 0.5, 6.5), 2), "bucket": rng.choice([16, 32]),
            "subgroup": rng.choice([4, 8])}
    if kind == "batch":
        case["graph"] = rng.random() < 0.25
    return case


# ---------------------------------------------------------------- networks
@functools.lru_cache(maxsize=64)
def _base(family, size, net_seed, log10):
    """(network, bound on its reachable states)"""
    if family == "tiny":
        return W.tiny_cycles(), 4096
    if family == "ring":
        return W.token_ring(size), 2 * size * 3 ** (size - 1)
    if family == "large":
        net = W.large_random_network(size)
        return net, _local_product(net)
    nets, _, bounds = W.served_networks(1, net_seed, log10, log10)
    return nets[0], max(64, bounds[0])


@functools.lru_cache(maxsize=64)
def _bases(kind, n, net_seed, lo, hi):
    if kind == "batch":
        return W.batch_networks(n, net_seed, lo, hi)
    nets, _, bounds = W.served_networks(n, net_seed, lo, hi)
    return nets, bounds


def _local_reach(net):
    """Per process, the local states reachable when a rule may fire as soon as
    every participant has a reachable state that offers its label."""
    P, R = net.n_procs, net.rules.shape[0]
    governed = [{int(net.rules[r, p]) for r in range(R) if net.rules[r, p] >= 0} for p in range(P)]
    edges = [t.tolist() for t in net.trans]
    reach = [{int(net.initial[p])} for p in range(P)]
    grew = True
    while grew:
        grew = False
        offered = [{lab for s, lab, _ in edges[p] if s in reach[p]} for p in range(P)]
        fires = [set() for _ in range(P)]
        for r in range(R):
            parts = [p for p in range(P) if net.rules[r, p] >= 0]
            if all(int(net.rules[r, p]) in offered[p] for p in parts):
                for p in parts:
                    fires[p].add(int(net.rules[r, p]))
        for p in range(P):
            for s, lab, d in edges[p]:
                if s in reach[p] and d not in reach[p] and (
                        lab in fires[p] if lab in governed[p] else True):
                    reach[p].add(d)
                    grew = True
    return reach


def _local_product(net):
    return math.prod(len(s) for s in _local_reach(net))


def _mean_successors(net):
    """Product transitions per state, averaged over the local products."""
    reach = _local_reach(net)
    P = net.n_procs
    governed = [{int(net.rules[r, p]) for r in range(net.rules.shape[0]) if net.rules[r, p] >= 0}
                for p in range(P)]
    per = [{} for _ in range(P)]
    total = 0.0
    for p in range(P):
        for s, lab, _ in net.trans[p].tolist():
            if s in reach[p]:
                per[p][lab] = per[p].get(lab, 0) + 1 / len(reach[p])
        total += sum(v for lab, v in per[p].items() if lab not in governed[p])
    for r in range(net.rules.shape[0]):
        total += math.prod(per[p].get(int(net.rules[r, p]), 0.0) for p in range(P)
                           if net.rules[r, p] >= 0)
    return total


def _starts(net):
    """Per process, the states it may start from with the same local states
    reachable (every label firing) as from its initial state."""
    out = []
    for p in range(net.n_procs):
        succ = {}
        for s, _, d in net.trans[p].tolist():
            succ.setdefault(s, set()).add(d)

        def reach(s):
            seen, todo = {s}, [s]
            while todo:
                for d in succ.get(todo.pop(), ()):
                    if d not in seen:
                        seen.add(d)
                        todo.append(d)
            return seen

        first = int(net.initial[p])
        out.append([s for s in sorted(reach(first)) if first in reach(s)])
    return out


def _varied(net, rng, move=True):
    """The network with a quarter of its processes started elsewhere and a
    transition of half of them offered twice (move), every process's local
    states renamed and its transitions listed in another order."""
    trans, initial = [], []
    P = len(net.n_states)
    starts = _starts(net) if move else None
    moved = set(rng.permutation(P)[: max(1, P // 4)].tolist()) if move else set()
    for p in range(P):
        name = rng.permutation(int(net.n_states[p])).astype(np.uint32)
        t = net.trans[p]
        if move and len(t) and rng.random() < 0.5:
            t = np.concatenate([t, t[rng.integers(len(t))][None]])
        t = np.stack([name[t[:, 0]], t[:, 1], name[t[:, 2]]], axis=1) if len(t) else t
        trans.append(t[rng.permutation(len(t))])
        first = starts[p][rng.integers(len(starts[p]))] if p in moved else int(net.initial[p])
        initial.append(int(name[first]))
    return gx.Network(net.n_states, np.asarray(initial, np.uint32), trans, net.n_labels, net.rules)


def _tiny(rng):
    """Four cycles of eight states that meet in state 0 in pairs, as
    ``workloads.tiny_cycles``, with other starts and other meeting targets."""
    net = W.tiny_cycles()
    trans = [t.copy() for t in net.trans]
    for t in trans:
        t[t[:, 1] == 1, 2] = rng.integers(2, 7)
    return gx.Network(net.n_states, rng.integers(5, 9, 4).astype(np.uint32) % 8, trans,
                      net.n_labels, net.rules)


def _ring(net, rng):
    """A ring whose other nodes are anywhere before the token's arrival."""
    initial = net.initial.copy()
    initial[1:] = rng.integers(0, 3, len(initial) - 1)
    return gx.Network(net.n_states, initial, net.trans, net.n_labels, net.rules)


def _network_of(case):
    return _base(case["family"], case.get("size", 0), case.get("net_seed", 0),
                 case.get("log10", 0.0))


def _networks_of(case):
    return _bases(case["kind"], case["nets"], case["net_seed"], case["lo"], case["hi"])


# ---------------------------------------------------------------- vectors
def _distinct(n, w, first):
    """n distinct vectors of w words, bit 31 of every word clear: a bijection
    of the counters first .. first + n - 1 (of 31 bits for one word, 62 for
    more)."""
    c = torch.arange(n, dtype=torch.int64, device=DEVICE) + first
    if w == 1:
        m = (1 << 31) - 1
        for a, s in ((0x2545F491, 15), (0x6F4F2A35, 13)):
            c = (c * a) & m
            c = c ^ (c >> s)
        return c.to(torch.int32).reshape(n, 1)
    m = (1 << 62) - 1
    cols = []
    for _ in range(0, w, 2):
        for a, s in ((0x1FB21C651E98DF25, 29), (0x16E8FEB86659FD93, 32)):
            c = (c * a) & m
            c = c ^ (c >> s)
        cols += [c & 0x7FFFFFFF, c >> 31]
    out = torch.empty((n, w), dtype=torch.int32, device=DEVICE)
    for k in range(w):
        out[:, k] = cols[k].to(torch.int32)
    return out


def _put_sizes(case):
    """(vectors of the first call, of the second, of the second that are new)"""
    n = case["keys"]
    new = n - int(round(case["seen"] * n))
    return n, n, new


# ---------------------------------------------------------------- states
def prepare(case, seed):
    kind = case["kind"]
    rng = np.random.default_rng(seed)
    if kind == "explore":
        net, bound = _network_of(case)
        if case["family"] == "tiny":
            net = _tiny(rng)
        elif case["family"] == "ring":
            net = _ring(net, rng)
        net = _varied(net, rng, move=case["family"] not in ("tiny", "ring") and not case.get("monitor"))
        monitor = None
        if case.get("monitor"):
            acts = list(range(net.rules.shape[0] + net.n_labels))
            n_mon, first, trans = W.random_monitor(case.get("automaton", 3), acts, 4, 4)
            net, proc, flags = gx.add_monitor(net, (n_mon, first, trans), [3])
            monitor = (proc, flags)
            bound *= 4
        view = gx.network_view(net)
        slots = case.get("slots") or max(1 << 16, int(case.get("room", 2.0) * bound))
        if case["family"] == "tiny":
            slots = 1 << 16
        table = gx.Table(gx.network_words(view), case["bucket"], slots,
                         subgroup=case["subgroup"], max_hashes=32)
        return {"kind": kind, "view": view, "table": table, "monitor": monitor,
                "fetch": bool(case.get("fetch"))}
    if kind == "put":
        n, n2, new = _put_sizes(case)
        w = case["words"]
        first = int(rng.integers(0, 1 << (20 if w == 1 else 40)))
        both = _distinct(n + new, w, first)
        gen = torch.Generator(device=DEVICE)
        gen.manual_seed(int(seed))
        second = both[new:][torch.randperm(n2, device=DEVICE, generator=gen)].contiguous()
        table = gx.Table(w, case["bucket"], max(64, int((n + new) / case["load"])),
                         subgroup=case["subgroup"], keys_per_subgroup=case["in_flight"],
                         max_hashes=64)
        return {"kind": kind, "table": table, "first": both[:n].contiguous(), "second": second,
                "status": [torch.zeros(k, dtype=torch.uint8, device=DEVICE) for k in (n, n2)],
                "n_new": torch.zeros(1, dtype=torch.int64, device=DEVICE)}
    nets, bounds = _networks_of(case)
    views = [gx.network_view(_varied(net, rng)) for net in nets]
    if kind == "batch":
        batch = gx.Batch(views, [2 * b for b in bounds], max_hashes=32,
                         bucket_words=case["bucket"], subgroup=case["subgroup"],
                         keys_per_subgroup=1, use_graph=case["graph"], max_levels=512)
        return {"kind": kind, "batch": batch}
    server = gx.Server(12 << 30, max_hashes=32, bucket_words=case["bucket"],
                       subgroup=case["subgroup"], keys_per_subgroup=1)
    return {"kind": kind, "server": server, "views": views, "bounds": bounds}


def _room(a, rows, dtype):
    """The rows of a, zeros after them up to a multiple of ``rows`` (how many
    levels or deadlocks there are depends on the start)."""
    n = max(1, -(-len(a) // rows)) * rows
    out = np.zeros((n,) + a.shape[1:], dtype)
    out[: len(a)] = a
    return out


def _together(results):
    """The results of many explorations as a few arrays."""
    return {"n_states": np.array([r.n_states for r in results], np.int64),
            "n_transitions": np.array([r.n_transitions for r in results], np.int64),
            "levels": np.stack([_room(r.levels, 128, np.int64)[:128] for r in results]),
            "n_levels": np.array([len(r.levels) for r in results], np.int64),
            "n_deadlocks": np.array([len(r.deadlocks) for r in results], np.int64),
            "deadlocks": _room(np.concatenate([r.deadlocks.reshape(-1) for r in results]), 1 << 14,
                               np.int32)}


def run(state):
    kind = state["kind"]
    if kind == "explore":
        table = state["table"]
        table.clear()
        r = gx.explore(state["view"], table, monitor=state["monitor"])
        out = {"n_states": r.n_states, "n_transitions": r.n_transitions,
               "levels": _room(r.levels, 128, np.int64),
               "deadlocks": _room(r.deadlocks, 256, np.int32)}
        if state["monitor"] is not None:
            out["violations"] = r.violations.view(np.int32)
        if state["fetch"]:
            out["states"] = table.dump().view(np.int32)
        return out
    if kind == "put":
        table, (st1, st2), n_new = state["table"], state["status"], state["n_new"]
        table.clear()
        n_new.zero_()
        table.find_or_put(state["first"], st1, n_new)
        table.find_or_put(state["second"], st2, n_new)
        return {"first": st1, "second": st2, "n_new": n_new}
    if kind == "batch":
        state["batch"].run()
        got = state["batch"].results()
        return _together([r for _, r in got])
    server = state["server"]
    ids = [server.submit(v, b) for v, b in zip(state["views"], state["bounds"])]
    return _together([server.poll(i)[1] for i in ids])


# ---------------------------------------------------------------- floors
def _explore_bytes(net, states, words):
    """Every reachable state stored once and read once as a frontier state,
    every successor's words compared with a stored vector's."""
    return 4 * words * states * (2 + _mean_successors(net))


def _words(net):
    word = used = 0
    for n in net.n_states:
        b = max(1, int(n - 1).bit_length())
        if used + b > 31:
            word, used = word + 1, 0
        used += b
    return word + 1


def work(case):
    """Bytes of one pass; nothing here multiplies, so no operations are
    counted.  Sizes of random networks are those of the products of their
    locally reachable states."""
    kind = case["kind"]
    if kind == "put":
        n, n2, new = _put_sizes(case)
        w = case["words"]
        # vectors and statuses of both calls; the table filled once, its slots
        # cleared before
        return {"bytes": float((n + n2) * (4 * w + 1) + (n + new) * 4 * w * (1 + 1 / case["load"])),
                "flops": 0.0}
    if kind == "explore":
        net, bound = _network_of(case)
        states = bound if case["family"] in ("tiny", "ring") else _local_product(net)
        return {"bytes": float(_explore_bytes(net, states, _words(net))), "flops": 0.0}
    nets, _ = _networks_of(case)
    return {"bytes": float(sum(_explore_bytes(n, _local_product(n), _words(n)) for n in nets)),
            "flops": 0.0}


# ---------------------------------------------------------------- exact
def exact(case, seed):
    """Closed forms where there are some: the statuses of distinct vectors,
    the sizes of the products of cycles and of a ring."""
    if case["kind"] == "put":
        n, n2, new = _put_sizes(case)
        return {"first": np.full(n, 1, np.uint8),  # each of them new
                "second": None, "n_new": np.array([n + new], np.int64)}
    if case["kind"] == "explore" and case["family"] in ("tiny", "ring") and not case.get("monitor"):
        n = case["size"]
        return {"n_states": 8 ** n if case["family"] == "tiny" else 2 * n * 3 ** (n - 1),
                "n_transitions": None, "levels": None, "deadlocks": None}
    return None
