"""GPU parity of arbor_rehydrate at the edges of its 64-position segments: the
resident count and the block size around multiples of 64, for every row size,
bit-exact against the oracle."""
import numpy as np
import pytest
import torch

from oracle import arbor_oracle as O
from paper_2605_22106_amd import _lib as L
from paper_2605_22106_amd import synth
from tests.gpu_helpers import assert_same_pool, check_rc, gpu_to_oracle, status, to_gpu, workspace
from tests.helpers import np_float, oracle_state
from tests.test_gpu_parity import PARAMS, _event, rand_A

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 128)])
def test_rehydrate_segments(dtype, d):
    n = [700, 64, 64, 65, 127, 128, 129, 300, 300, 1, 320, 512]
    keep = [700, 0, 63, 64, 65, 1, 128, 64, 190, 0, 257, 511]
    parent = [-1] + [0] * 3 + [1] * 8
    st = synth.build_state(parent, n, layers=2, kv_heads=2, q_per_kv=1, head_dim=d, dtype=dtype,
                           seed=d, shuffle_pages=True, spare_pages=3, active=[11])
    kv, ost = to_gpu(st), oracle_state(st)
    A = rand_A(st["num_tokens"], 2)
    k = np.array(keep)
    sel, _ = O.select(ost, A, k, PARAMS["l_tail"])
    ost = O.compact(ost, k, sel)
    _event(st, kv, A, k, PARAMS)
    ws = workspace(kv)
    for on in (np.array([1, 0, 1, 0, 1, 0, 1, 0, 1, 0, 1, 0], np.uint8), np.ones(12, np.uint8)):
        ost, _ = O.rehydrate(ost, on, np_float(st["host_k"]), np_float(st["host_v"]))
        stt = status()
        check_rc(L.arbor_rehydrate(kv, torch.tensor(on, device="cuda"), st["host_k"].cuda(),
                                   st["host_v"].cuda(), stt, ws))
        torch.cuda.synchronize()
        assert int(stt) == L.OK
        assert_same_pool(gpu_to_oracle(kv), ost)


def _restore(n, keep, layers, kv_heads, d=64):
    """State, tree and oracle state with keep[i] of block i's n[i] tokens resident."""
    parent = [-1] + [0] * (len(n) - 1)
    st = synth.build_state(parent, n, layers=layers, kv_heads=kv_heads, q_per_kv=1, head_dim=d,
                           dtype="bf16", seed=len(n), shuffle_pages=True, active=[1])
    kv = to_gpu(st)
    A = rand_A(st["num_tokens"], 2)
    _event(st, kv, A, np.array(keep), PARAMS)
    return st, kv, A


def test_rehydrate_long_blocks():
    """Blocks of thousands of tokens: a segment's resident slots are found by a search
    of 64 probes a round (one round from 65 resident slots, two from 4,097)."""
    n = [70, 5000, 9001, 9001, 4160, 4161, 8200]
    keep = [70, 4097, 8999, 70, 4095, 4096, 65]
    st, kv, A = _restore(n, keep, 1, 2)
    ost = oracle_state(st)
    sel, _ = O.select(ost, A, np.array(keep), PARAMS["l_tail"])
    ost = O.compact(ost, np.array(keep), sel)
    on = np.ones(len(n), np.uint8)
    ost, _ = O.rehydrate(ost, on, np_float(st["host_k"]), np_float(st["host_v"]))
    stt = status()
    check_rc(L.arbor_rehydrate(kv, torch.tensor(on, device="cuda"), st["host_k"].cuda(),
                               st["host_v"].cuda(), stt, workspace(kv)))
    torch.cuda.synchronize()
    assert int(stt) == L.OK
    assert_same_pool(gpu_to_oracle(kv), ost)


def test_rehydrate_time_grows_with_the_block():
    """One plane of a block of four times the tokens takes about four times as long
    (sixteen times if every segment visited every resident slot)."""
    us = []
    for n in (12288, 49152):
        st, kv, _ = _restore([16, n], [16, n - n // 8], 1, 1)
        hk, hv, ws = st["host_k"].cuda(), st["host_v"].cuda(), workspace(kv)
        on = torch.ones(2, dtype=torch.uint8, device="cuda")
        saved = [x.clone() for x in (kv.n_kept, kv.page_table, kv.slot_pos, kv.free_stack,
                                     kv.free_top)]
        stt, best = status(), float("inf")
        for _ in range(4):
            for x, y in zip((kv.n_kept, kv.page_table, kv.slot_pos, kv.free_stack, kv.free_top),
                            saved):
                x.copy_(y)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            check_rc(L.arbor_rehydrate(kv, on, hk, hv, stt, ws))
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        assert int(stt) == L.OK and kv.n_kept.tolist() == [16, n]
        us.append(1e3 * best)
    assert us[1] < 8 * us[0], us
