"""GPU parity of arbor_walk (Alg. 2's event-driven controller run on the
device over a walk of Transition events) against the oracle's walk.

* Without scoring (fixed s and A), a whole 30-event walk in ONE call --
  allocate, lazy rehydration from pinned host memory, eviction, and Pressure
  at B - delta -- against O.walk: pool state, page tables, free stack and
  per-event statistics bit-exact.
* With scoring, event by event: each call's A and s against the oracle's
  score within 1e-4 (fed the GPU's A, rows_seen, s from the event before, so
  that the integer decisions compare bit-exactly), the state bit-exact.
* The same scored walk in one call equals it issued event by event, bitwise.
"""
import math

import numpy as np
import pytest
import torch

from oracle import arbor_oracle as O
from paper_2605_22106_amd import _lib as L
from paper_2605_22106_amd import synth
from tests.gpu_helpers import assert_same_pool, check_rc, gpu_to_oracle, status, to_gpu, workspace
from tests.helpers import np_float, oracle_state

pytestmark = pytest.mark.gpu

BASE = dict(alpha_max=math.inf, gamma=2.0, lambda_d=0.0, lambda_delta=0.5, eta=0.8, r_min=0.05,
            k_min=2, l_tail=4, theta=(1.0, 1.0, 1.0), select_mode=0, score_self_window=0)
W = 8


def _case(seed, steps=30):
    parent, n_full = synth.complete_tree(3, 3, 160, 48)
    st = synth.build_state(parent, n_full, layers=2, kv_heads=2, q_per_kv=2, head_dim=128,
                           dtype="bf16", seed=seed, shuffle_pages=True, spare_pages=6,
                           window=W, slice_layers=[0, 1], active=[13])
    targets = synth.walk_targets(parent, steps, 0.3, seed, 13)
    g = torch.Generator().manual_seed(seed)
    q = torch.randn((len(targets), 2, 4, W, 128), generator=g).to(torch.bfloat16)
    return st, parent, targets, q


class Bufs:
    def __init__(self, kv, st, steps):
        V, N = kv.num_nodes, kv.num_tokens
        self.k = torch.empty(V, dtype=torch.int32, device="cuda")
        self.delta = torch.empty_like(self.k)
        self.on_path = torch.empty(V, dtype=torch.uint8, device="cuda")
        self.sel = torch.empty(N, dtype=torch.int32, device="cuda")
        self.stats = torch.full((steps, 4), -9, dtype=torch.int64, device="cuda")
        self.rows = torch.zeros(V, dtype=torch.int64, device="cuda")
        self.a = torch.empty(V, device="cuda")
        self.ws = workspace(kv, max_context=160 + 3 * 48, max_observers=1, window=W, n_slice=2)
        self.hk = st["host_k"].pin_memory()
        self.hv = st["host_v"].pin_memory()


def _walk(kv, st, b, targets, budget, p, A, s, stt, margin, q=None):
    kw = {}
    if q is not None:
        kw = dict(q_win=q.cuda().contiguous(), window=W, slice_layers=[0, 1],
                  v_in=st["v_sig"].cuda(), u_in=st["u_sig"].cuda(), rows_seen=b.rows, a_out=b.a)
    check_rc(L.arbor_walk(kv, torch.tensor(targets, dtype=torch.int32, device="cuda"), budget, p,
                          A, s, b.k, b.delta, b.on_path, b.sel, stt, b.ws, host_k=b.hk,
                          host_v=b.hv, pressure_margin=margin, stats=b.stats[:len(targets)],
                          **kw))
    torch.cuda.synchronize()


@pytest.mark.parametrize("seed,margin", [(0, 0), (1, 40)])
def test_walk_in_one_call_matches_oracle(seed, margin):
    st, parent, targets, _ = _case(seed)
    kv = to_gpu(st)
    N = st["num_tokens"]
    rng = np.random.default_rng(seed)
    s_np = rng.random(len(parent)).astype(np.float32)
    A_np = rng.random(N).astype(np.float32)
    budget = int(0.25 * N)
    b = Bufs(kv, st, len(targets))
    stt = status()
    _walk(kv, st, b, targets, budget, BASE, torch.tensor(A_np, device="cuda"),
          torch.tensor(s_np, device="cuda"), stt, margin)
    ost = oracle_state(st)
    out = O.walk(ost, targets, budget, s_np, A_np, np.zeros(len(parent), np.int64), BASE,
                 np_float(st["host_k"]), np_float(st["host_v"]), pressure_margin=margin)
    assert int(stt) == out[5]
    assert np.array_equal(b.stats.cpu().numpy(), out[4])
    assert_same_pool(gpu_to_oracle(kv), out[0])
    assert out[4][:, 1].sum() > 0, "the walk rehydrates"
    if margin:
        assert out[4][:, 3].sum() > 0, "Pressure fires"


def test_scored_walk_event_by_event():
    st, parent, targets, q = _case(2, steps=16)
    kv = to_gpu(st)
    N = st["num_tokens"]
    budget = int(0.25 * N)
    b = Bufs(kv, st, 1)
    A = torch.zeros(N, device="cuda")
    s = torch.full((len(parent),), 0.5, device="cuda")
    stt = status()
    hk, hv = np_float(st["host_k"]), np_float(st["host_v"])
    for e, leaf in enumerate(targets):
        ost = gpu_to_oracle(kv)
        A0, s0, r0 = A.cpu().numpy(), s.cpu().numpy(), b.rows.cpu().numpy()
        _walk(kv, st, b, [leaf], budget, BASE, A, s, stt, 30, q[e:e + 1])
        assert int(stt) >= 0, e
        A1, s1 = A.cpu().numpy(), s.cpu().numpy()
        # the oracle's event on the same state, scores and queries
        k, _, on_path, _ = O.allocate(ost["parent"], ost["n_full"], ost["n_kept"], [leaf], budget,
                                      s0, BASE)
        ost, rs = O.rehydrate(ost, on_path, hk, hv)
        assert rs == O.OK
        Ao, ro, _, so = O.score(ost, [leaf], np_float(q[e:e + 1]), W, [0, 1], 2,
                                st["v_sig"].numpy(), st["u_sig"].numpy(), A0, r0)
        g, o = A1.astype(np.float64), Ao.astype(np.float64)
        assert np.all(np.abs(g - o) <= 1e-4 * np.abs(o) + 1e-30), e
        assert np.all(np.abs(s1.astype(np.float64) - so) <= 1e-4 * np.abs(so) + 1e-30), e
        assert np.array_equal(b.rows.cpu().numpy(), ro)
        # the integer decisions on the GPU's own A and s
        sel, _ = O.select(ost, A1, k, BASE["l_tail"])
        ost = O.compact(ost, k, sel)
        if int(np.sum(ost["n_kept"])) >= budget - 30:
            k2, _, _, _ = O.allocate(ost["parent"], ost["n_full"], ost["n_kept"], [leaf],
                                     budget - 30, s1, BASE)
            sel, _ = O.select(ost, A1, k2, BASE["l_tail"])
            ost = O.compact(ost, k2, sel)
        assert_same_pool(gpu_to_oracle(kv), ost)


def test_scored_walk_in_one_call_equals_event_by_event():
    st, parent, targets, q = _case(3, steps=20)
    N = st["num_tokens"]
    budget = int(0.25 * N)
    res = []
    for per_event in (False, True):
        kv = to_gpu(st)
        b = Bufs(kv, st, len(targets))
        A = torch.zeros(N, device="cuda")
        s = torch.full((len(parent),), 0.5, device="cuda")
        stt = status()
        if per_event:
            rows = []
            for e, leaf in enumerate(targets):
                _walk(kv, st, b, [leaf], budget, BASE, A, s, stt, 25, q[e:e + 1])
                rows.append(b.stats[0].cpu().numpy().copy())
            stats = np.array(rows)
        else:
            _walk(kv, st, b, targets, budget, BASE, A, s, stt, 25, q)
            stats = b.stats.cpu().numpy()
        res.append((gpu_to_oracle(kv), A.cpu().numpy(), s.cpu().numpy(), stats, int(stt)))
    (p0, A0, s0, t0, c0), (p1, A1, s1, t1, c1) = res
    assert c0 == c1 and c0 >= 0
    assert np.array_equal(t0, t1)
    assert np.array_equal(A0.view(np.uint32), A1.view(np.uint32))
    assert np.array_equal(s0.view(np.uint32), s1.view(np.uint32))
    assert_same_pool(p0, p1)


def test_walk_without_free_pages_keeps_the_events_statistics():
    """An event whose rehydration finds too few pages fails, changes nothing in the
    pool, and still has its statistics; the events after it have none."""
    st, parent, _, _ = _case(3)
    kv = to_gpu(st)
    N = st["num_tokens"]
    s = torch.full((len(parent),), 0.5, device="cuda")
    A = torch.rand(N, device="cuda")
    budget = int(0.25 * N)
    b = Bufs(kv, st, 3)
    stt = status()
    _walk(kv, st, b, [13], budget, BASE, A, s, stt, 0)
    assert int(stt) >= 0
    kv.free_top.zero_()
    before = gpu_to_oracle(kv)
    leaf = len(parent) - 1
    k, _, on_path, _ = O.allocate(before["parent"], before["n_full"], before["n_kept"], [leaf],
                                  budget, s.cpu().numpy(), BASE)
    c, n = np.asarray(before["n_kept"]), np.asarray(before["n_full"])
    want = [int(k.sum()), int((n - c)[(np.asarray(on_path) != 0) & (c < n)].sum()),
            int(np.maximum(c - k, 0).sum()), 0]
    b.stats.fill_(-9)
    _walk(kv, st, b, [leaf, 13], budget, BASE, A, s, stt, 0)
    assert int(stt) == L.ENOPAGES
    assert want[1] > 0 and b.stats[0].tolist() == want
    assert b.stats[1].tolist() == [-9] * 4
    assert_same_pool(gpu_to_oracle(kv), before)
