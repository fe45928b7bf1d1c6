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
