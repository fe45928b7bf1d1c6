"""Performance cases of the eviction hot path, through the Python binding of the C ABI.

Each case is one call, or one short sequence of calls, that a Tree-of-Thoughts
server makes while it searches: scoring of blocks, keep-counts, the decoding
step's attention, the entropy signal, and the Transition events that restore
and evict blocks.  Tree shapes and geometries are those of the synthetic
configurations (paper_2605_22106_amd/synth.py) or lie between them; `draw`
gives more of the same ranges.  All inputs are seeded and made on the GPU.

Kinds
  score        arbor_score: window queries of observers against their chains
  allocate     arbor_allocate: keep-counts of every block under the budget
  decode       arbor_tree_decode_attn, or with credit ..._scored
  uncertainty  arbor_uncertainty over rows of boundary logits
  transition   the search jumps to another frontier and back: allocate,
               rehydrate, select + compact, twice
  walk         arbor_walk: a sequence of single-leaf Transition events, scored
"""
from __future__ import annotations

import math
import random

import torch

from paper_2605_22106_amd import _lib as L
from paper_2605_22106_amd import synth

P = synth.PAGE_SIZE


def listed():
    b8 = dict(branching=4, depth=3, root=1024, node=256, heads=8, group=4, dim=128)
    b70 = dict(branching=4, depth=4, root=4096, node=512, heads=8, group=8, dim=128)
    dpts = dict(branching=4, depth=4, root=1024, node=128, heads=8, group=4, dim=128)
    deep = dict(branching=3, depth=8, root=1024, node=64, heads=8, group=4, dim=128)
    tiny = dict(branching=2, depth=2, root=64, node=32, heads=4, group=1, dim=64)
    return [
        # the smallest tree, fp32: what a call costs in launches and latency
        dict(name="score_tiny", kind="score", **tiny, ragged=False, kept=1.0, shape=0, layers=1,
             slices=1, window=8, observers=7, dtype="f32"),
        # the eviction event of the 8B-shaped tree: every block's window replayed
        dict(name="score_8b", kind="score", **b8, ragged=False, kept=1.0, shape=0, layers=32,
             slices=2, window=32, observers=85, dtype="bf16"),
        # the same on the 70B-shaped tree (four of its layers): the largest replay
        dict(name="score_70b", kind="score", **b70, ragged=False, kept=1.0, shape=0, layers=4,
             slices=2, window=32, observers=341, dtype="bf16"),
        # a search step of a wide frontier: 16 new leaves score a tree of ragged
        # blocks of which an earlier event has evicted a part
        dict(name="score_frontier", kind="score", **dpts, ragged=True, kept=0.4, shape=11,
             layers=8, slices=2, window=8, observers=16, dtype="bf16"),
        # keep-counts of a deep tree of 9,841 blocks
        dict(name="allocate_deep", kind="allocate", branching=3, depth=8, root=1024, node=64,
             ragged=False, shape=0, active=1, rho=0.2),
        # one decoding step of four leaves, all 32 layers of the 8B shape
        dict(name="decode_8b", kind="decode", **b8, ragged=False, kept=1.0, shape=0, layers=32,
             calls=1, leaves=4, scored=False, dtype="bf16", out="bf16"),
        # eight leaves of the 70B shape, a quarter of its layers, fp32 outputs
        dict(name="decode_70b", kind="decode", **b70, ragged=False, kept=1.0, shape=0, layers=20,
             calls=1, leaves=8, scored=False, dtype="bf16", out="f32"),
        # a model's own loop: one call for each layer, here four of them, 16
        # ragged leaves, each call crediting its layer's weights to A
        dict(name="decode_layers", kind="decode", **dpts, ragged=True, kept=1.0, shape=12,
             layers=4, calls=4, leaves=16, scored=True, dtype="bf16", out="bf16"),
        # the entropy signal of every block of the 8B tree, whole vocabulary
        dict(name="uncertainty_rows", kind="uncertainty", rows=85, vocab=128256, top_k=0,
             dtype="bf16"),
        # top-40 entropy of the 16 blocks that a frontier has just closed, fp32
        dict(name="uncertainty_topk", kind="uncertainty", rows=16, vocab=128256, top_k=40,
             dtype="f32"),
        # backtracking between two frontiers of the 8B tree at a 25 % budget
        dict(name="transition_8b", kind="transition", **b8, ragged=False, shape=0, layers=32,
             active=4, rho=0.25, dtype="bf16"),
        # the controller over eight events of a random walk in the deep tree
        dict(name="walk_deep", kind="walk", **deep, ragged=False, shape=3, layers=4, steps=8,
             window=32, rho=0.2, dtype="bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _nodes(case):
    return sum(case["branching"] ** d for d in range(case["depth"] + 1))


def draw(rng):
    """One more case of the ranges that the listed ones span."""
    while True:
        kind = rng.choice(["score", "score", "score", "allocate", "decode", "decode", "decode",
                           "uncertainty", "uncertainty", "transition", "walk"])
        if kind == "uncertainty":
            c = dict(kind=kind, rows=_log(rng, 1, 128), vocab=8 * _log(rng, 1000, 19000),
                     top_k=rng.choice([0, 0, _log(rng, 2, 250)]), dtype=rng.choice(["bf16", "f32"]))
            return c
        c = dict(kind=kind, branching=rng.randint(2, 5), depth=rng.randint(1, 8),
                 root=_log(rng, 40, 4096), node=_log(rng, 20, 512))
        if not 3 <= _nodes(c) <= (9841 if kind in ("allocate", "walk") else 400):
            continue
        tokens = c["root"] + c["node"] * (_nodes(c) - 1)
        if tokens > 700_000 or (kind not in ("allocate", "walk") and tokens > 180_000):
            continue
        c.update(ragged=rng.random() < 0.7, shape=rng.randrange(1 << 16))
        if kind == "allocate":
            c.update(active=_log(rng, 1, 16), rho=round(rng.uniform(0.15, 0.6), 3))
            return c
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        if kind == "walk":
            dtype = "bf16"
        c.update(heads=rng.choice([4, 8]), group=rng.choice([1, 4, 4, 8]),
                 dim=rng.choice([64, 128, 128]), dtype=dtype)
        token_bytes = 2 * c["heads"] * c["dim"] * (2 if dtype == "bf16" else 4)
        room = (12 << 30) // (tokens * token_bytes)      # layers that make a pool of 12 GiB
        if room < 2:
            continue
        if kind == "score":
            c.update(kept=rng.choice([1.0, round(rng.uniform(0.2, 0.9), 3)]),
                     layers=min(room, rng.choice([1, 4, 8, 32])), window=_log(rng, 1, 32))
            c.update(slices=min(2, c["layers"]),
                     observers=rng.choice([_nodes(c), _log(rng, 1, _nodes(c))]))
            if work(c)["flops"] * (1 if dtype == "bf16" else 8) > 1.2e12:
                continue
        elif kind == "decode":
            calls = rng.choice([1, 1, 4])
            c.update(kept=rng.choice([1.0, 1.0, round(rng.uniform(0.2, 0.9), 3)]),
                     layers=min(room, rng.choice([4, 8, 16, 32])) if calls == 1 else 4,
                     calls=calls, leaves=_log(rng, 1, 24), scored=rng.random() < 0.4,
                     out=rng.choice(["bf16", "f32"]))
            if c["layers"] > room or c["layers"] < calls:
                continue
        elif kind == "transition":
            c.update(layers=min(room // 2, rng.choice([1, 4, 8, 32])), active=_log(rng, 1, 8),
                     rho=round(rng.uniform(0.2, 0.7), 3))
            there, back = _fronts(c, _tree(c)[0])
            if set(there) == set(back):
                continue
        else:
            if c["depth"] < 3:
                continue
            c.update(layers=min(room // 2, 4), steps=rng.randint(4, 12), window=_log(rng, 1, 32),
                     rho=round(rng.uniform(0.15, 0.5), 3))
        if c["layers"] >= 1:
            return c


# ---- the tree of a case (host side, from the case alone) ---------------------

def _tree(case):
    """parent, n (tokens of each block), children-free deepest leaves in id order."""
    parent, n = synth.complete_tree(case["branching"], case["depth"], case["root"], case["node"])
    if case["ragged"]:
        r = random.Random(case["shape"])
        n = [max(1, round(x * r.uniform(0.3, 1.0))) for x in n]
    return parent, n


def _chain(parent, i):
    out = []
    while i >= 0:
        out.append(i)
        i = parent[i]
    return out[::-1]


def _deepest(parent, count, offset=0.0):
    """`count` leaves spread evenly over the deepest level (repeated where it has fewer)."""
    d = synth.tree_depths(parent)
    lv = [i for i in range(len(parent)) if d[i] == max(d)]
    return [lv[int((k + offset) * len(lv) / count) % len(lv)] for k in range(count)]


def _resident(case, parent, n, full=()):
    """Tokens that each block holds: a share `kept` of it where an event has evicted."""
    if case.get("kept", 1.0) >= 1.0:
        return list(n)
    r = random.Random(case["shape"] + 1)
    full = set(full)
    return [x if i in full else min(x, max(1, round(x * case["kept"] * r.uniform(0.4, 1.6))))
            for i, x in enumerate(n)]


def _observers(case, parent):
    v = len(parent)
    if case["observers"] >= v:
        return list(range(v))
    # the newest blocks: a frontier's leaves, in creation order
    return sorted(set(_deepest(parent, case["observers"]))) or [v - 1]


def _slices(case):
    if case["slices"] == 1:
        return [0]
    return [case["layers"] // 2, case["layers"] - 1]


def _dt(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _size(name):
    return 2 if name == "bf16" else 4


# ---- states on the GPU -------------------------------------------------------

def _gen(seed, purpose):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 7919 + purpose)
    return g


def _kv(case, seed, parent, n, c, store):
    """The paged pool with c[i] of block i's n[i] tokens resident, pages shuffled;
    with `store` also the token-major record of every token."""
    dev = "cuda"
    V, N = len(parent), sum(n)
    Lr, H, D = case["layers"], case["heads"], case["dim"]
    g = _gen(seed, 1)
    nt = torch.tensor(n, device=dev)
    ct = torch.tensor(c, device=dev)
    tok_off = torch.zeros(V + 1, dtype=torch.int64, device=dev)
    tok_off[1:] = nt.cumsum(0)
    page_off = torch.zeros(V + 1, dtype=torch.int64, device=dev)
    page_off[1:] = ((nt + P - 1) // P).cumsum(0)
    pages = int(page_off[-1])
    perm = torch.randperm(pages, generator=g, device=dev)
    # logical pages in use, the rest on the free stack
    node_of_page = torch.repeat_interleave(torch.arange(V, device=dev), page_off.diff())
    q = torch.arange(pages, device=dev) - page_off[node_of_page]
    used = q < ((ct + P - 1) // P)[node_of_page]
    page_table = torch.where(used, perm, -torch.ones_like(perm)).to(torch.int32)
    free = perm[~used].to(torch.int32)
    free_stack = torch.full((pages,), -1, dtype=torch.int32, device=dev)
    free_stack[:free.numel()] = free
    # the resident positions of each block: c[i] of n[i] at random, ascending
    node = torch.repeat_interleave(torch.arange(V, device=dev), nt)
    pos = torch.arange(N, device=dev) - tok_off[node]
    key = torch.rand(N, generator=g, device=dev, dtype=torch.float64)
    rank = torch.empty(N, dtype=torch.int64, device=dev)
    rank[torch.argsort(node + key)] = pos            # rank of a token's key within its block
    keep = rank < ct[node]
    count = keep.to(torch.int64).cumsum(0)
    first = torch.zeros(V, dtype=torch.int64, device=dev)
    first[1:] = ct.cumsum(0)[:-1]
    tok = torch.nonzero(keep).flatten()
    slot = count[tok] - 1 - first[node[tok]]
    phys = page_table[page_off[node[tok]] + slot // P].to(torch.int64)
    slot_pos = torch.full((pages, P), -1, dtype=torch.int32, device=dev)
    slot_pos[phys, slot % P] = pos[tok].to(torch.int32)
    # values: normal, 2 % of the keys heavy (x 4)
    heavy = torch.rand(N, generator=g, device=dev) < 0.02
    dt = _dt(case["dtype"])
    out = {}
    if store:
        hk = torch.randn((N, Lr, H, D), generator=g, device=dev, dtype=dt)
        hk.mul_(torch.where(heavy, 4.0, 1.0).to(dt)[:, None, None, None])
        hv = torch.randn((N, Lr, H, D), generator=g, device=dev, dtype=dt)
        src = torch.zeros(pages * P, dtype=torch.int64, device=dev)
        src[phys * P + slot % P] = tok
        out["host_k"], out["host_v"] = hk, hv
        kv = []
        for h in (hk, hv):
            t = torch.empty((Lr, pages, H, P, D), dtype=dt, device=dev)
            for l in range(Lr):
                t[l] = h[:, l][src].view(pages, P, H, D).transpose(1, 2)
            kv.append(t)
        k, v = kv
    else:
        k = torch.randn((Lr, pages, H, P, D), generator=g, device=dev, dtype=dt)
        v = torch.randn((Lr, pages, H, P, D), generator=g, device=dev, dtype=dt)
        scale = torch.ones((pages, P), device=dev, dtype=dt)
        hs = heavy[tok]
        scale[phys[hs], (slot % P)[hs]] = 4.0
        k.mul_(scale[None, :, None, :, None])
    i32 = torch.int32
    out["kv"] = L.KVState(torch.tensor(parent, dtype=i32, device=dev), nt.to(i32), tok_off,
                          page_off, ct.to(i32), page_table, k, v, slot_pos, free_stack,
                          torch.tensor([free.numel()], dtype=i32, device=dev), Lr, H,
                          case["group"], D, P, L.BF16 if dt == torch.bfloat16 else L.F32, N)
    return out


def _workspace(kv, **sizes):
    return torch.empty(L.arbor_workspace_size(kv, **sizes), dtype=torch.uint8, device="cuda")


def _i32(values):
    return torch.tensor(values, dtype=torch.int32, device="cuda")


def _context(parent, n):
    """Tokens of the longest chain."""
    total = [0] * len(n)
    for i, x in enumerate(n):
        total[i] = x + (total[parent[i]] if i else 0)
    return max(total)


def _params(case):
    return dict(synth.DEFAULT_PARAMS)


def prepare(case, seed):
    kind = case["kind"]
    dev = "cuda"
    st = dict(case=case, status=torch.zeros(1, dtype=torch.int32, device=dev))
    g = _gen(seed, 2)
    if kind == "uncertainty":
        R, Vc = case["rows"], case["vocab"]
        z = torch.randn((R, Vc), generator=g, device=dev)
        z.mul_(torch.tensor([(0.5, 2.0, 3.0, 2.0)[r % 4] for r in range(R)], device=dev)[:, None])
        peaked = torch.arange(0, R, 3, device=dev)
        z[peaked, torch.randint(Vc, (peaked.numel(),), generator=g, device=dev)] += 12.0
        st["logits"] = z.to(_dt(case["dtype"]))
        st["u"] = torch.zeros(R, device=dev)
        st["ws"] = torch.empty(L.arbor_uncertainty_workspace_size(
            R, Vc, L.BF16 if case["dtype"] == "bf16" else L.F32), dtype=torch.uint8, device=dev)
        return st
    parent, n = _tree(case)
    V, N = len(parent), sum(n)
    st["params"] = _params(case)
    if kind == "allocate":
        full = dict(case, layers=1, heads=1, group=1, dim=64, dtype="bf16")
        st.update(_kv(full, seed, parent, n, n, False))
        st["active"] = _i32(_deepest(parent, case["active"]))
        st["budget"] = _budget(case, parent, n)
        st["s"] = torch.rand(V, generator=g, device=dev)
        st["ws"] = _workspace(st["kv"])
    elif kind == "score":
        c = _resident(case, parent, n)
        st.update(_kv(case, seed, parent, n, c, False))
        obs = _observers(case, parent)
        Hq = case["heads"] * case["group"]
        st["observers"] = _i32(obs)
        st["slices"] = _slices(case)
        st["q_win"] = torch.randn((len(obs), case["slices"], Hq, case["window"], case["dim"]),
                                  generator=g, device=dev).to(_dt(case["dtype"]))
        st["v_sig"] = torch.rand(V, generator=g, device=dev)
        st["u_sig"] = torch.rand(V, generator=g, device=dev)
        st["A"] = torch.zeros(N, device=dev)
        st["rows"] = torch.zeros(V, dtype=torch.int64, device=dev)
        st["a"] = torch.zeros(V, device=dev)
        st["s"] = torch.zeros(V, device=dev)
        st["ws"] = _workspace(st["kv"], max_context=_context(parent, n), max_observers=len(obs),
                              window=case["window"], n_slice=case["slices"])
    elif kind == "decode":
        leaves = _deepest(parent, case["leaves"])
        path = set(x for leaf in leaves for x in _chain(parent, leaf))
        c = _resident(case, parent, n, path if case["kept"] >= 1.0 else ())
        st.update(_kv(case, seed, parent, n, c, False))
        Hq = case["heads"] * case["group"]
        per = case["layers"] // case["calls"]
        st["leaves"] = _i32(leaves)
        dt = _dt(case["dtype"])
        st["q"] = [torch.randn((len(leaves), per, Hq, case["dim"]), generator=g,
                               device=dev).to(dt) for _ in range(case["calls"])]
        st["out"] = [torch.zeros(q.shape, dtype=_dt(case["out"]), device=dev) for q in st["q"]]
        st["lse"] = [torch.zeros(q.shape[:3], device=dev) for q in st["q"]]
        st["A"] = torch.zeros(N, device=dev)
        st["rows"] = torch.zeros(V, dtype=torch.int64, device=dev)
        st["ws"] = _workspace(st["kv"], max_context=_context(parent, n),
                              max_leaves=len(leaves), max_layers=per, n_slice=2)
    else:
        st.update(_kv(case, seed, parent, n, n, True))
        st["budget"] = _budget(case, parent, n)
        st["s"] = torch.rand(V, generator=g, device=dev)
        st["A"] = torch.rand(N, generator=g, device=dev)
        i32 = torch.int32
        st["k"] = torch.zeros(V, dtype=i32, device=dev)
        st["delta"] = torch.zeros(V, dtype=i32, device=dev)
        st["on_path"] = torch.zeros(V, dtype=torch.uint8, device=dev)
        st["sel"] = torch.zeros(N, dtype=i32, device=dev)
        if kind == "transition":
            st["fronts"] = [_i32(f) for f in _fronts(case, parent)]
            st["ws"] = _workspace(st["kv"])
        else:
            st["targets"] = _i32(_targets(case, parent))
            steps = st["targets"].numel()
            Hq = case["heads"] * case["group"]
            st["q_win"] = torch.randn((steps, 2, Hq, case["window"], case["dim"]), generator=g,
                                      device=dev).to(_dt(case["dtype"]))
            st["v_sig"] = torch.rand(V, generator=g, device=dev)
            st["u_sig"] = torch.rand(V, generator=g, device=dev)
            st["rows"] = torch.zeros(V, dtype=torch.int64, device=dev)
            st["a"] = torch.zeros(V, device=dev)
            st["stats"] = torch.zeros((steps, 4), dtype=torch.int64, device=dev)
            st["ws"] = _workspace(st["kv"], max_context=_context(parent, n), max_observers=1,
                                  window=case["window"], n_slice=2)
    return st


def _fronts(case, parent):
    """Two sets of active leaves, in different subtrees where there is room."""
    return [_deepest(parent, case["active"]), _deepest(parent, case["active"], 0.5)]


def _targets(case, parent):
    start = _deepest(parent, 1)[0]
    t = synth.walk_targets(parent, 4 * case["steps"], 0.3, case["shape"], start)
    return t[:case["steps"]]


def _budget(case, parent, n):
    """rho of all tokens, at least the longest chains and the floors of the rest."""
    need = 0
    if case["kind"] in ("allocate", "transition"):
        fronts = _fronts(case, parent) if case["kind"] == "transition" else [
            _deepest(parent, case["active"])]
        for f in fronts:
            path = set(x for leaf in f for x in _chain(parent, leaf))
            need = max(need, sum(n[x] for x in path))
    else:
        need = _context(parent, n)
    floors = sum(max(min(8, x), int(0.05 * x)) for x in n)
    return max(int(case["rho"] * sum(n)), need + floors + len(n))


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "uncertainty":
        L.arbor_uncertainty(st["logits"], case["top_k"], st["u"], st["status"], st["ws"])
        return dict(u=st["u"], status=st["status"])
    kv, p = st["kv"], st["params"]
    if kind == "allocate":
        V = kv.num_nodes
        if "k" not in st:
            st["k"] = torch.zeros(V, dtype=torch.int32, device="cuda")
            st["delta"] = torch.zeros(V, dtype=torch.int32, device="cuda")
            st["on_path"] = torch.zeros(V, dtype=torch.uint8, device="cuda")
        L.arbor_allocate(kv, st["active"], st["budget"], st["s"], p, st["k"], st["delta"],
                         st["on_path"], st["status"], st["ws"])
        return dict(k=st["k"], delta=st["delta"], on_path=st["on_path"], status=st["status"])
    if kind == "score":
        L.arbor_score(kv, st["observers"], st["q_win"], case["window"], st["slices"], st["v_sig"],
                      st["u_sig"], st["A"], st["rows"], st["a"], st["s"], p, st["status"],
                      st["ws"])
        return dict(A=st["A"], rows=st["rows"], a=st["a"], s=st["s"], status=st["status"])
    if kind == "decode":
        per = case["layers"] // case["calls"]
        for i in range(case["calls"]):
            l0 = i * per
            if case["scored"]:
                sl = [l0 + per - 1] if per == 1 else [l0 + per // 2, l0 + per - 1]
                L.arbor_tree_decode_attn_scored(kv, st["leaves"], l0, l0 + per, st["q"][i],
                                                st["out"][i], st["lse"][i], 0.0, sl, 0, st["A"],
                                                st["rows"], st["status"], st["ws"])
            else:
                L.arbor_tree_decode_attn(kv, st["leaves"], l0, l0 + per, st["q"][i],
                                         st["out"][i], st["lse"][i], 0.0, st["status"], st["ws"])
        return dict(out=st["out"], lse=st["lse"], A=st["A"], rows=st["rows"], status=st["status"])
    if kind == "transition":
        # to the other frontier and back
        for f in (st["fronts"][1], st["fronts"][0]):
            L.arbor_allocate(kv, f, st["budget"], st["s"], p, st["k"], st["delta"],
                             st["on_path"], st["status"], st["ws"])
            L.arbor_rehydrate(kv, st["on_path"], st["host_k"], st["host_v"], st["status"],
                              st["ws"])
            L.arbor_select_compact(kv, st["A"], st["k"], p, st["sel"], st["status"], st["ws"])
        return dict(k=st["k"], delta=st["delta"], on_path=st["on_path"], kv_k=kv.k, kv_v=kv.v,
                    n_kept=kv.n_kept, page_table=kv.page_table, slot_pos=kv.slot_pos,
                    free_top=kv.free_top, status=st["status"])
    L.arbor_walk(kv, st["targets"], st["budget"], p, st["A"], st["s"], st["k"], st["delta"],
                 st["on_path"], st["sel"], st["status"], st["ws"], host_k=st["host_k"],
                 host_v=st["host_v"], pressure_margin=0, q_win=st["q_win"],
                 window=case["window"], slice_layers=[case["layers"] // 2, case["layers"] - 1],
                 v_in=st["v_sig"], u_in=st["u_sig"], rows_seen=st["rows"], a_out=st["a"],
                 stats=st["stats"])
    return dict(A=st["A"], rows=st["rows"], a=st["a"], s=st["s"], stats=st["stats"], k=st["k"],
                kv_k=kv.k, kv_v=kv.v, n_kept=kv.n_kept, page_table=kv.page_table,
                slot_pos=kv.slot_pos, free_top=kv.free_top, status=st["status"])


# ---- what a pass cannot do without ---------------------------------------------

def _score_work(case, parent, n, c, obs, S, window, union=True):
    """Bytes and 2 d flops per (window row, visible key): the keys of the slice once,
    the window queries once, A read and written."""
    H, G, D, e = case["heads"], case["group"], case["dim"], _size(case["dtype"])
    seen, pairs, rows = set(), 0, 0
    total = [0] * len(n)
    for i in range(len(n)):
        total[i] = c[i] + (total[parent[i]] if i else 0)
    for j in obs:
        w = min(window, n[j])
        # the block's own keys up to each row (as resident tokens spread evenly)
        pairs += w * (total[j] - c[j]) + int(w * c[j] * (1 - (w - 1) / (2.0 * n[j])))
        rows += w
        seen.update(_chain(parent, j))
    keys = sum(c[i] for i in seen)
    return dict(bytes=S * (keys * H * D * e + rows * H * G * D * e) + 8 * sum(n) + 32 * len(n),
                flops=2.0 * D * H * G * S * pairs)


def work(case):
    kind = case["kind"]
    if kind == "uncertainty":
        el = case["rows"] * case["vocab"]
        return dict(bytes=el * _size(case["dtype"]) + 4 * case["rows"], flops=4.0 * el)
    parent, n = _tree(case)
    V = len(n)
    if kind == "allocate":
        return dict(bytes=V * (4 * 4 + 4 + 4 + 1), flops=20.0 * V)
    H, G, D, e = case["heads"], case["group"], case["dim"], _size(case["dtype"])
    if kind == "score":
        return _score_work(case, parent, n, _resident(case, parent, n), _observers(case, parent),
                           case["slices"], case["window"])
    if kind == "decode":
        leaves = _deepest(parent, case["leaves"])
        path = set(x for leaf in leaves for x in _chain(parent, leaf))
        c = _resident(case, parent, n, path if case["kept"] >= 1.0 else ())
        union = sum(c[i] for i in path)
        chain = sum(c[x] for leaf in leaves for x in _chain(parent, leaf))
        io = case["leaves"] * case["layers"] * H * G * (D * (e + _size(case["out"])) + 4)
        return dict(bytes=2 * union * H * D * e * case["layers"] + io,
                    flops=4.0 * D * chain * H * G * case["layers"])
    token = 2 * case["layers"] * H * D * e
    budget = _budget(case, parent, n)
    if kind == "transition":
        paths = [set(x for leaf in f for x in _chain(parent, leaf)) for f in _fronts(case, parent)]
        back = 0
        for a, b in ((0, 1), (1, 0)):
            new = sum(n[x] for x in paths[b] - paths[a])
            # what the blocks of the new path had kept at this budget
            off = sum(n) - sum(n[x] for x in paths[a])
            share = min(1.0, (budget - sum(n[x] for x in paths[a])) / max(1, off))
            back += new * (1 - share) * (1 + share)   # restored, and as many kept rows moved in
        return dict(bytes=2.0 * back * token + 2 * 45 * V, flops=40.0 * V)
    b = f = 0.0
    prev = set(_chain(parent, _targets(case, parent)[-1]))
    for t in _targets(case, parent):
        path = _chain(parent, t)
        s = _score_work(case, parent, n, n, [t], 2, case["window"])
        share = min(1.0, (budget - sum(n[x] for x in path)) / max(1, sum(n)))
        b += s["bytes"] - 8 * sum(n) + 8 * sum(n[x] for x in path) + 45 * V
        b += 2.0 * token * sum(n[x] for x in path if x not in prev) * (1 - share)
        f += s["flops"] + 20.0 * V
        prev = set(path)
    return dict(bytes=b, flops=f)


def tolerance(case):
    kind = case["kind"]
    if kind in ("allocate", "transition"):
        return "exact"          # counts, layouts and copied rows
    if kind == "decode" and case["out"] == "bf16":
        # an fp32 result that lies at a rounding boundary may take the next bf16 value
        # (one part in 128 at most), which few do
        return {"rel": 5e-4, "max": 1e-2}
    # fp32 sums of fp32 terms: up to 4.2e-7 from the 64-bit values over these cases
    return {"rel": 2e-6, "max": 1e-4}


# ---- the same in 64 bits ----------------------------------------------------------

def _rows_of(kv, layer, chain, which):
    """Resident rows of the blocks of a chain, root first: [H][tokens][d] in fp64."""
    c = kv.n_kept.tolist() if not hasattr(kv, "_c") else kv._c
    kv._c = c
    if not hasattr(kv, "_po"):
        kv._po = kv.page_off.tolist()
    idx = []
    for i in chain:
        pg = kv.page_table[kv._po[i]:kv._po[i] + (c[i] + P - 1) // P].to(torch.int64)
        idx.append((pg[:, None] * P + torch.arange(P, device="cuda")[None, :]).flatten()[:c[i]])
    idx = torch.cat(idx)
    t = which[layer][idx // P, :, idx % P]              # [tokens][H][d]
    return t.permute(1, 0, 2).to(torch.float64).contiguous(), idx


def _exact_score(case, seed):
    st = prepare(case, seed)
    kv = st["kv"]
    parent, n = _tree(case)
    V, N = len(n), sum(n)
    obs = _observers(case, parent)
    H, G, D, W = case["heads"], case["group"], case["dim"], case["window"]
    to = kv.tok_off.tolist()
    A = torch.zeros(N, dtype=torch.float64, device="cuda")
    rows = [0] * V
    for o, j in enumerate(obs):
        chain = _chain(parent, j)
        w = min(W, n[j])
        for si, layer in enumerate(st["slices"]):
            k, idx = _rows_of(kv, layer, chain, kv.k)
            pos = kv.slot_pos.flatten()[idx].to(torch.int64)
            cnt = torch.tensor([kv._c[x] for x in chain], device="cuda")
            node = torch.repeat_interleave(torch.tensor(chain, device="cuda"), cnt)
            q = st["q_win"][o, si].to(torch.float64)[:, :w].reshape(H, G * w, D)
            z = torch.bmm(q, k.transpose(1, 2).contiguous()) / math.sqrt(D)
            u = n[j] - w + torch.arange(w, device="cuda")
            hide = (node == j)[None, :] & (pos[None, :] > u[:, None])       # [w][tokens]
            z.view(H, G, w, -1).masked_fill_(hide, -math.inf)
            pr = torch.softmax(z, -1).sum(dim=(0, 1))
            anc = node != j
            A.index_add_(0, torch.tensor(to, device="cuda")[node[anc]] + pos[anc], pr[anc])
        for x in chain[:-1]:
            rows[x] += len(st["slices"]) * H * G * w
    r = torch.tensor(rows, dtype=torch.float64, device="cuda")
    node = torch.repeat_interleave(torch.arange(V, device="cuda"), kv.n_full.to(torch.int64))
    mass = torch.zeros(V, dtype=torch.float64, device="cuda").index_add_(0, node, A)
    a = torch.where(r > 0, mass / r.clamp(min=1), torch.zeros_like(mass))
    th = st["params"]["theta"]
    s = torch.sigmoid(th[0] * st["v_sig"].double() + th[1] * st["u_sig"].double() + th[2] * a)
    return dict(A=A, rows=None, a=a, s=s, status=None)


def _exact_decode(case, seed):
    st = prepare(case, seed)
    kv = st["kv"]
    parent, n = _tree(case)
    H, G, D = case["heads"], case["group"], case["dim"]
    per = case["layers"] // case["calls"]
    leaves = _deepest(parent, case["leaves"])
    to = kv.tok_off
    A = torch.zeros(sum(n), dtype=torch.float64, device="cuda")
    outs, lses = [], []
    for i in range(case["calls"]):
        out = torch.zeros(st["q"][i].shape, dtype=torch.float64, device="cuda")
        lse = torch.zeros(st["q"][i].shape[:3], dtype=torch.float64, device="cuda")
        credited = [per - 1] if per == 1 else [per // 2, per - 1]
        for b, leaf in enumerate(leaves):
            chain = _chain(parent, leaf)
            for lr in range(per):
                k, idx = _rows_of(kv, i * per + lr, chain, kv.k)
                v, _ = _rows_of(kv, i * per + lr, chain, kv.v)
                q = st["q"][i][b, lr].to(torch.float64).reshape(H, G, D)
                z = torch.bmm(q, k.transpose(1, 2).contiguous()) / math.sqrt(D)
                pr = torch.softmax(z, -1)
                out[b, lr] = torch.bmm(pr, v).reshape(H * G, D)
                lse[b, lr] = torch.logsumexp(z, -1).flatten()
                if case["scored"] and lr in credited:
                    cnt = torch.tensor([kv._c[x] for x in chain], device="cuda")
                    node = torch.repeat_interleave(torch.tensor(chain, device="cuda"), cnt)
                    pos = kv.slot_pos.flatten()[idx].to(torch.int64)
                    anc = node != leaf
                    A.index_add_(0, to[node[anc]] + pos[anc], pr.sum(dim=(0, 1))[anc])
        outs.append(out)
        lses.append(lse)
    return dict(out=outs, lse=lses, A=A if case["scored"] else None, rows=None, status=None)


def exact(case, seed):
    kind = case["kind"]
    if kind == "score":
        return _exact_score(case, seed)
    if kind == "decode":
        return _exact_decode(case, seed)
    if kind == "uncertainty":
        z = prepare(case, seed)["logits"].to(torch.float64)
        lp = torch.log_softmax(z, -1)
        if 0 < case["top_k"] < case["vocab"]:
            top = torch.topk(lp, case["top_k"], dim=-1).values
            rest = (1.0 - top.exp().sum(-1)).clamp(min=0.0)
            h = -(top.exp() * top).sum(-1) - torch.special.xlogy(rest, rest)
        else:
            h = -(lp.exp() * lp).sum(-1)
        return dict(u=1.0 - h / math.log(case["vocab"]), status=None)
    # counts, layouts and bitwise copies; a walk's values follow from its decisions
    return None
