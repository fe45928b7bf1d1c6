"""GPU parity of arbor_allocate on trees beyond the one-workgroup kernel (512
blocks), bit-exact against the oracle: at the edges of its node state (blocks
in registers up to 10,240, links in LDS up to 16,384), with scores spread over
decades, equal (all prices tie) or near zero, and under floor protection."""
import numpy as np
import pytest
import torch

from oracle import arbor_oracle as O
from paper_2605_22106_amd import _lib as L
from paper_2605_22106_amd import synth
from tests.gpu_helpers import check_rc, status, to_gpu, workspace
from tests.test_gpu_parity import PARAMS

pytestmark = pytest.mark.gpu


def _run(kv, act, budget, s, p, ws):
    V = kv.num_nodes
    k = torch.empty(V, dtype=torch.int32, device="cuda")
    dl = torch.empty_like(k)
    onp = torch.empty(V, dtype=torch.uint8, device="cuda")
    stt = status()
    check_rc(L.arbor_allocate(kv, act, budget, torch.tensor(s, device="cuda"), p, k, dl, onp, stt,
                              ws))
    torch.cuda.synchronize()
    return k.cpu().numpy(), dl.cpu().numpy(), onp.cpu().numpy(), int(stt)


@pytest.mark.parametrize("V,max_n", [(513, 300), (10240, 33), (10241, 17), (16384, 9), (16385, 9)])
def test_allocate_large_edges(V, max_n):
    parent, n_full = synth.random_tree(V, max_n, V)
    rng = np.random.default_rng(V)
    leaves = sorted(set(range(V)) - set(parent))
    active = sorted(rng.choice(leaves, size=3, replace=False).tolist())
    st = synth.build_state(parent, n_full, layers=1, kv_heads=1, q_per_kv=1, head_dim=64,
                           dtype="f32", seed=V, active=active, host_store=False)
    kv = to_gpu(st)
    nf, nk, par = st["n_full"].numpy(), st["n_kept"].numpy(), st["parent"].numpy()
    ws = workspace(kv)
    act = torch.tensor(active, dtype=torch.int32, device="cuda")
    total = int(nk.sum())
    u = rng.random(V)
    scores = dict(uniform=u, equal=np.full(V, 0.5), low=u ** 9, two=np.where(u < 0.5, 0.25, 0.75))
    for name, s in scores.items():
        s = s.astype(np.float32)
        for rho, extra in ((0.3, {}), (0.6, dict(k_protect=3, lambda_delta=0.0)), (0.02, {})):
            p = dict(PARAMS, **extra)
            want = O.allocate(par, nf, nk, active, int(rho * total), s, p)
            k, dl, onp, sg = _run(kv, act, int(rho * total), s, p, ws)
            assert sg == want[3], (name, rho)
            assert np.array_equal(k, want[0]), (name, rho)
            assert np.array_equal(dl, want[1]) and np.array_equal(onp, want[2]), (name, rho)
    off = next(i for i in range(V - 1, 0, -1) if not want[2][i])
    for bad, code in ((np.nan, L.ENONFINITE), (1.5, L.EINVAL)):
        s = u.astype(np.float32)
        s[off] = bad
        assert _run(kv, act, total // 2, s, PARAMS, ws)[3] == code
    out = torch.tensor([active[0], V], dtype=torch.int32, device="cuda")
    assert _run(kv, out, total // 2, u.astype(np.float32), PARAMS, ws)[3] == L.EINVAL


def _near_ties(prices):
    """Ranks E whose price (the cut) lies among more than 1,536 prices within 1e-13 of one
    another: the edges and the middle of each run of equal doubles of such a group."""
    last = np.searchsorted(prices, prices * (1.0 + 1e-13), side="right")
    out, i = [], 0
    while i < len(prices):
        if last[i] - i > 1536:
            runs = np.flatnonzero(np.diff(prices[i:last[i]])) + i + 1
            edges = [i, *runs.tolist(), int(last[i])]
            for a, b in zip(edges, edges[1:]):
                out += [a, (a + b) // 2, b - 1]
            i = int(last[i])
        else:
            i += 1
    return sorted(set(out))


@pytest.mark.parametrize("branching,depth,lo,hi", [(5, 5, 20, 64), (4, 6, 10, 64), (3, 8, 5, 33)])
def test_allocate_large_near_ties(branching, depth, lo, hi):
    """Equal scores over ragged blocks put one rational price a few roundings apart in
    thousands of blocks: a search on rounded counts cannot confirm its bracket there and is
    done again on exact ones.  The sizes lie between those that fill the thread's registers,
    so some of a thread's blocks are padding."""
    parent, _ = synth.complete_tree(branching, depth, 1, 1)
    V = len(parent)
    rng = np.random.default_rng(V)
    n_full = [200] + rng.integers(lo, hi + 1, V - 1).tolist()
    active = [V - 1]
    st = synth.build_state(parent, n_full, layers=1, kv_heads=1, q_per_kv=1, head_dim=64,
                           dtype="f32", seed=V, active=active, host_store=False)
    kv = to_gpu(st)
    nf, nk, par = st["n_full"].numpy(), st["n_kept"].numpy(), st["parent"].numpy()
    ws = workspace(kv)
    act = torch.tensor(active, dtype=torch.int32, device="cuda")
    s = np.full(V, 0.5, np.float32)
    s_gpu = torch.tensor(s, device="cuda")
    d, on_path, delta = O.geometry(par, active)
    k = torch.empty(V, dtype=torch.int32, device="cuda")
    dl, onp, stt = torch.empty_like(k), torch.empty(V, dtype=torch.uint8, device="cuda"), status()
    for extra in ({}, dict(lambda_delta=0.0), dict(lambda_delta=0.0, k_min=0, l_tail=0, r_min=0.0)):
        p = dict(PARAMS, **extra)
        off = np.flatnonzero(~np.asarray(on_path, bool))
        F = np.array([O.floor_count(nf[i], nk[i], p) for i in off])
        W = np.array([O.value_geometry_weight(s[i], d[i], delta[i], p, False) for i in off]) * nf[off]
        owner = np.repeat(np.arange(len(off)), nk[off] - F)
        j = np.concatenate([np.arange(f + 1, c + 1) for f, c in zip(F, nk[off])])
        price = j / W[owner]
        order = np.sort(price)
        base = int(nf[np.asarray(on_path, bool)].sum() + F.sum())
        ranks = _near_ties(order)
        assert ranks
        # (every one of a few, else spread over them)
        ranks = [ranks[x] for x in np.unique(np.linspace(0, len(ranks) - 1, 60).astype(int))]
        for x, E in enumerate(ranks):
            want = nf.copy()
            want[off] = F + np.bincount(owner[price < order[E]], minlength=len(off))
            if x == 0:
                assert np.array_equal(want, O.allocate(par, nf, nk, active, base + E, s, p)[0])
            k.fill_(-77)
            check_rc(L.arbor_allocate(kv, act, base + E, s_gpu, p, k, dl, onp, stt, ws))
            torch.cuda.synchronize()
            assert int(stt) == L.OK, (extra, E)
            got = k.cpu().numpy()
            assert np.array_equal(got, want), (extra, E, int((got == -77).sum()))
