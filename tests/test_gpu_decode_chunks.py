"""GPU parity of the tree decode over its chunk sizes and row blocks: the plan
cuts a chain node's slots into chunks of 64 to 1,024 by the number of units,
and its rows (leaves below it times G) into blocks of 16.  |g - o| <= 2e-3 for
fp32 outputs and 1e-4 relative for A, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import arbor_oracle as O
from paper_2605_22106_amd import _lib as L
from paper_2605_22106_amd import synth
from tests.gpu_helpers import check_rc, status, to_gpu, workspace
from tests.helpers import oracle_state

pytestmark = pytest.mark.gpu


def _tree(root, nodes):
    """root -> three children -> two leaves each, with the given token counts."""
    parent = [-1, 0, 0, 0, 1, 1, 2, 2, 3, 3]
    return parent, [root] + nodes


# (layers, root tokens, leaves, G, dtype): one plane set of 8 kv heads per
# layer, so that 1 layer gives few units (64-slot chunks), 8 layers under many
# rows a middle size, and 64 layers at least 4,096 units of 1,024 slots
CASES = [(1, 1, [4], 4, "bf16"), (1, 63, [4, 9], 8, "bf16"), (1, 1100, [4, 5, 6, 9], 4, "bf16"),
         (1, 64, [1, 4, 8], 1, "f32"), (8, 1025, [4, 5, 6, 7, 8, 9] * 3, 8, "bf16"),
         (8, 700, [4], 1, "f32"), (64, 2049, [4, 5, 6, 9, 9], 8, "bf16"),
         (64, 1024, [7], 4, "bf16"), (64, 2049, [4, 5, 9], 4, "f32"), (24, 1025, [4, 6], 8, "f32"), (2, 300, [4, 5, 6, 7, 8, 9, 1, 0] * 9, 2, "bf16")]


@pytest.mark.parametrize("layers,root,leaves,G,dtype", CASES)
def test_decode_chunks(layers, root, leaves, G, dtype):
    nodes = [70, 128, 1, 65, 16, 257, 33, 640, 15]
    parent, n_full = _tree(root, nodes)
    d = 64 if layers > 1 else 128
    st = synth.build_state(parent, n_full, layers=layers, kv_heads=8, q_per_kv=G, head_dim=d,
                           dtype=dtype, seed=root + layers, shuffle_pages=True, heavy_frac=0.05,
                           active=leaves, host_store=False)
    kv = to_gpu(st)
    Hq, nb = 8 * G, len(leaves)
    q = st["q_dec"].cuda().contiguous()
    lt = torch.tensor(leaves, dtype=torch.int32, device="cuda")
    ws = workspace(kv, max_leaves=nb, max_layers=layers, n_slice=1)
    outs = []
    for scored in (False, True):
        out = torch.full((nb, layers, Hq, d), 7.0, device="cuda")
        lse = torch.full((nb, layers, Hq), 7.0, device="cuda")
        A = torch.zeros(kv.num_tokens, device="cuda")
        rows = torch.zeros(kv.num_nodes, dtype=torch.int64, device="cuda")
        stt = status()
        if scored:
            check_rc(L.arbor_tree_decode_attn_scored(kv, lt, 0, layers, q, out, lse, 0.0,
                                                     [layers - 1], 1, A, rows, stt, ws))
        else:
            check_rc(L.arbor_tree_decode_attn(kv, lt, 0, layers, q, out, lse, 0.0, stt, ws))
        torch.cuda.synchronize()
        assert int(stt) == L.OK
        outs.append((out, lse))
    # the plain and the scored call agree bitwise, at every layer
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    # the last and the first layer against the oracle on that layer
    for lr in {0, layers - 1}:
        one = oracle_state(dict(st, k=st["k"][lr:lr + 1], v=st["v"][lr:lr + 1]))
        ql = q[:, lr:lr + 1].float().cpu().numpy()
        o, ls = O.tree_decode_attn(one, leaves, 0, 1, ql, G)
        assert np.max(np.abs(outs[0][0][:, lr].cpu().numpy() - o[:, 0])) <= 2e-3
        assert np.max(np.abs(outs[0][1][:, lr].cpu().numpy() - ls[:, 0])) <= 2e-3
        if lr == layers - 1:
            Ao, ro = O.decode_credit(one, leaves, 0, ql, G, [0], np.zeros(kv.num_tokens, np.float32),
                                     np.zeros(kv.num_nodes, np.int64), self_window=1)
            assert np.allclose(A.cpu().numpy(), Ao, rtol=1e-4, atol=1e-30)
            assert np.array_equal(rows.cpu().numpy(), ro)


@pytest.mark.parametrize("node,d,step", [(512, 128, 16), (1024, 64, 8), (1500, 64, 8)])
def test_decode_long_chunks_are_as_accurate_as_short_ones(node, d, step):
    """64 layers in one call (chunks of 1,024 slots) and in calls of `step` layers (256
    slots): the fp32 outputs of the first are no further from 64 bits (the two per cent are
    the spread of a norm over 262,144 rounded values and more).  Heavy keys spread the
    logits, so that most weights lie far below their row's max."""
    layers, G = 64, 8
    parent = [-1, 0, 0, 1, 1, 2, 2]
    n_full = [2 * node + 40] + [node] * 6
    leaves = [3, 4, 5, 6] * 2
    st = synth.build_state(parent, n_full, layers=layers, kv_heads=8, q_per_kv=G, head_dim=d,
                           dtype="bf16", seed=node, shuffle_pages=True, heavy_frac=0.02,
                           active=leaves, host_store=False)
    kv = to_gpu(st)
    q = st["q_dec"].cuda().contiguous()
    lt = torch.tensor(leaves, dtype=torch.int32, device="cuda")
    ws = workspace(kv, max_leaves=len(leaves), max_layers=layers)
    stt = status()
    whole, each = (torch.empty((len(leaves), layers, 8 * G, d), device="cuda") for _ in range(2))
    check_rc(L.arbor_tree_decode_attn(kv, lt, 0, layers, q, whole, None, 0.0, stt, ws))
    for l in range(0, layers, step):
        out = torch.empty((len(leaves), step, 8 * G, d), device="cuda")
        check_rc(L.arbor_tree_decode_attn(kv, lt, l, l + step, q[:, l:l + step].contiguous(), out,
                                          None, 0.0, stt, ws))
        each[:, l:l + step] = out
    torch.cuda.synchronize()
    assert int(stt) == L.OK
    po, P = st["page_off"].tolist(), st["page_size"]
    num = torch.zeros(2, dtype=torch.float64)
    den = 0.0
    for b, chain in enumerate(([0, 1, 3], [0, 1, 4], [0, 2, 5], [0, 2, 6])):
        idx = torch.cat([(kv.page_table[po[i]:po[i + 1]].long()[:, None] * P +
                          torch.arange(P, device="cuda")).flatten()[:n_full[i]] for i in chain])
        for l in range(layers):
            k, v = (t[l].transpose(1, 2).reshape(-1, 8, d)[idx].double().transpose(0, 1).contiguous()
                    for t in (kv.k, kv.v))
            z = torch.bmm(q[b, l].view(8, G, d).double(), k.transpose(1, 2).contiguous()) / d ** 0.5
            o = torch.bmm(torch.softmax(z, -1), v).view(8 * G, d)
            den += float((o * o).sum())
            for x, t in enumerate((whole, each)):
                num[x] += float((t[b, l].double() - o).square().sum())
    err = (num / den).sqrt().tolist()
    assert err[0] <= 1.02 * err[1], err


def test_decode_credit_of_many_leaves_in_long_chunks():
    """Row blocks and chunks beyond the credit's workgroups (the plan's list of live 64-slot
    pieces): 40 leaves, blocks of 40 to 300 slots, 64 layers, two slices of which one listed
    twice, against the oracle; and an eighth of the layers, whose chunks are shorter."""
    parent = [-1] + [0] * 5 + [1 + i // 8 for i in range(40)]
    n_full = [1500] + [128, 300, 40, 65, 260] + [40 + 7 * i for i in range(40)]
    leaves, G, d = list(range(6, 46)), 4, 64
    for layers in (64, 8):
        st = synth.build_state(parent, n_full, layers=layers, kv_heads=8, q_per_kv=G, head_dim=d,
                               dtype="bf16", seed=layers, shuffle_pages=True, heavy_frac=0.05,
                               active=leaves, host_store=False)
        kv = to_gpu(st)
        q = st["q_dec"].cuda().contiguous()
        lt = torch.tensor(leaves, dtype=torch.int32, device="cuda")
        ws = workspace(kv, max_leaves=len(leaves), max_layers=layers, n_slice=3)
        out = torch.empty((len(leaves), layers, 8 * G, d), device="cuda")
        A = torch.zeros(kv.num_tokens, device="cuda")
        rows, stt = torch.zeros(kv.num_nodes, dtype=torch.int64, device="cuda"), status()
        check_rc(L.arbor_tree_decode_attn_scored(kv, lt, 0, layers, q, out, None, 0.0,
                                                 [1, layers - 1, 1], 0, A, rows, stt, ws))
        torch.cuda.synchronize()
        assert int(stt) == L.OK
        pick = [1, layers - 1]
        two = oracle_state(dict(st, k=st["k"][pick], v=st["v"][pick]))
        Ao, ro = O.decode_credit(two, leaves, 0, q[:, pick].float().cpu().numpy(), G, [0, 1, 0],
                                 np.zeros(kv.num_tokens, np.float32),
                                 np.zeros(kv.num_nodes, np.int64), self_window=0)
        assert np.allclose(A.cpu().numpy(), Ao, rtol=1e-4, atol=1e-30)
        assert np.array_equal(rows.cpu().numpy(), ro)
