"""GPU parity of arbor_score over its two launch shapes: few observers (16-row
groups and more key splits, up to 128 workgroups of the other shape) and many,
for 1 to 5 row groups, both dtypes and crediting modes; and one observer over a
tree beyond the setup's LDS.  fp32 outputs within 1e-4 of the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import arbor_oracle as O
from paper_2605_22106_amd import _lib as L
from paper_2605_22106_amd import synth
from tests.gpu_helpers import check_rc, status, to_gpu, workspace
from tests.helpers import np_float, oracle_state
from tests.test_gpu_parity import PARAMS, _close, _gpu_score

pytestmark = pytest.mark.gpu


def _both(st, kv, ost, obs, p):
    q = torch.randn((len(obs), len(st["slice_layers"]), st["kv_heads"] * st["q_per_kv"],
                     st["window"], st["head_dim"]),
                    generator=torch.Generator().manual_seed(len(obs))).to(st["k"].dtype)
    V = kv.num_nodes
    A, rows, a, s, sg = _gpu_score(st, kv, p, observers=torch.tensor(obs, dtype=torch.int32),
                                   q_win=q)
    Ao, ro, ao, so = O.score(ost, obs, np_float(q), st["window"], st["slice_layers"],
                             st["q_per_kv"], st["v_sig"].numpy(), st["u_sig"].numpy(),
                             np.zeros(st["num_tokens"], np.float32), np.zeros(V, np.int64),
                             theta=p["theta"], self_window=p["score_self_window"])
    assert sg == L.OK
    _close(A, Ao)
    assert np.array_equal(rows, ro)
    _close(a, ao)
    _close(s, so)


@pytest.mark.parametrize("G,window,dtype,d,sw", [(1, 3, "bf16", 128, 0), (4, 4, "bf16", 64, 1),
                                                 (4, 8, "bf16", 128, 1), (8, 33, "bf16", 128, 0),
                                                 (1, 16, "f32", 128, 1), (2, 33, "f32", 64, 0)])
def test_score_few_and_many_observers(G, window, dtype, d, sw):
    parent, n_full = synth.random_tree(40, 60, 3)
    n_full[0] = 333                                 # an uneven share of sub-pages per split
    st = synth.build_state(parent, n_full, layers=2, kv_heads=4, q_per_kv=G, head_dim=d,
                           dtype=dtype, seed=G, shuffle_pages=True, window=window, active=[39],
                           heavy_frac=0.05, host_store=False)
    kv, ost = to_gpu(st), oracle_state(st)
    p = dict(PARAMS, score_self_window=sw)
    # 2 x 4 planes: 16 observers of one slab are 128 workgroups, 17 more
    for obs in ([0], [39], [7, 39, 12], list(range(16)), list(range(23, 40)), list(range(40))):
        _both(st, kv, ost, obs, p)


@pytest.mark.parametrize("sw", [0, 1])
def test_score_one_observer_of_a_large_tree(sw):
    V = 2100
    parent, n_full = synth.random_tree(V, 24, 9)
    st = synth.build_state(parent, n_full, layers=1, kv_heads=2, q_per_kv=2, head_dim=64,
                           dtype="bf16", seed=1, shuffle_pages=True, window=5, active=[V - 1],
                           observers=[V - 1], host_store=False)
    kv, ost = to_gpu(st), oracle_state(st)
    p = dict(PARAMS, score_self_window=sw)
    for obs in ([V - 1], [0], [1]):
        _both(st, kv, ost, obs, p)
    # a malformed block off the chain is still refused, and nothing changes
    off = next(i for i in range(V - 1, 0, -1) if i != V - 1)
    kv.n_kept[off] = n_full[off] + 1
    A0 = np.random.default_rng(0).random(st["num_tokens"]).astype(np.float32)
    A, rows, _, _, sg = _gpu_score(st, kv, p, A0=A0, observers=torch.tensor([1], dtype=torch.int32))
    assert sg == L.EINVAL
    assert np.array_equal(A, A0) and not rows.any()


@pytest.mark.parametrize("n_root,n_obs", [(1, 33), (15, 300), (16, 34), (17, 257), (64, 63),
                                          (65, 300), (129, 40), (2048, 33), (2049, 33), (65, 16),
                                          (65, 17), (2049, 17)])
def test_score_root_parts_of_many_observers(n_root, n_obs):
    """More than 16 observers: the root's chunks are reduced in parts of 16 slots and
    groups of four observers, 256 observers at a time; beyond 2,048 slots uncut."""
    parent, n_full = synth.random_tree(n_obs + 1, 20, n_obs)
    n_full[0] = n_root
    st = synth.build_state(parent, n_full, layers=2, kv_heads=2, q_per_kv=2, head_dim=64,
                           dtype="bf16", seed=n_root, shuffle_pages=True, window=3,
                           active=[n_obs], host_store=False)
    kv, ost = to_gpu(st), oracle_state(st)
    for sw in (0, 1):
        _both(st, kv, ost, list(range(1, n_obs + 1)),
              dict(PARAMS, score_self_window=sw))


@pytest.mark.parametrize("deep,small,malformed,code", [
    (True, False, False, L.EUNSUPPORTED), (True, False, True, L.EINVAL),
    (False, True, False, L.EWORKSPACE), (False, True, True, L.EINVAL),
    (False, False, True, L.EINVAL), (True, True, True, L.EINVAL)])
def test_score_one_observer_error_codes(deep, small, malformed, code):
    """One observer over a large tree: the blocks are checked by other workgroups than its
    chain and the workspace, and a malformed block comes first whatever finds out first."""
    V, tail = 4200, 64 if deep else 40                 # a chain of tail + 1 blocks, then leaves
    parent = [-1] + list(range(tail)) + [0] * (V - 1 - tail)
    n_full = [200] + [20] * tail + [2] * (V - 1 - tail)
    st = synth.build_state(parent, n_full, layers=1, kv_heads=2, q_per_kv=2, head_dim=64,
                           dtype="bf16", seed=1, window=5, active=[tail], observers=[tail],
                           host_store=False)
    kv = to_gpu(st)
    if malformed:
        kv.n_kept[V - 3] = n_full[V - 3] + 1
    ws = workspace(kv, max_observers=1, window=5, n_slice=1)
    if small:                                          # room for the offsets and chains only
        ws = ws[:20 * V + st["num_tokens"] // 8 + 16 * 256]
    g = torch.Generator().manual_seed(3)
    A0, rows0 = torch.rand(st["num_tokens"], generator=g), torch.arange(V)
    a0, s0 = torch.rand(V, generator=g), torch.rand(V, generator=g)
    for _ in range(20):
        A, rows, a, s, stt = A0.cuda(), rows0.cuda(), a0.cuda(), s0.cuda(), status()
        check_rc(L.arbor_score(kv, st["observers"].cuda(), st["q_win"].cuda().contiguous(), 5, [0],
                               st["v_sig"].cuda(), st["u_sig"].cuda(), A, rows, a, s, PARAMS, stt,
                               ws))
        torch.cuda.synchronize()
        assert int(stt) == code
        for x, y in ((A, A0), (rows, rows0), (a, a0), (s, s0)):
            assert torch.equal(x.cpu(), y)
