"""GPU parity of arbor_uncertainty's chunked top-K at the edges of its paths:
candidates ranked or radix-selected (K around the limit, values that all tie),
chunks in registers or streamed again, chunks with fewer than K values.
Against fp64 torch, within 1e-5 absolute (fp32 sums of a row's terms)."""
import math

import pytest
import torch

from paper_2605_22106_amd import _lib as L
from tests.gpu_helpers import check_rc, status

pytestmark = pytest.mark.gpu


def _want(z, k):
    lp = torch.log_softmax(z.double(), -1)
    if 0 < k < z.shape[1]:
        top = torch.topk(lp, k, dim=-1).values
        rest = (1.0 - top.exp().sum(-1)).clamp(min=0.0)
        h = -(top.exp() * top).sum(-1) - torch.special.xlogy(rest, rest)
    else:
        h = -(lp.exp() * lp).sum(-1)
    return 1.0 - h / math.log(z.shape[1])


@pytest.mark.parametrize("rows,vocab,dtype", [(1, 16, "f32"), (3, 4096, "f32"), (1, 8192, "bf16"),
                                              (17, 50008, "bf16"), (64, 262144, "f32"),
                                              (64, 262272, "f32"), (700, 16392, "bf16")])
def test_topk_edges(rows, vocab, dtype):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(vocab)
    z = torch.randn(rows, vocab, generator=g, device="cuda") * 2.0
    z[0] = 0.5                                       # every value ties
    if rows > 1:
        z[1] = torch.round(z[1] * 2.0) / 2.0         # long runs of ties
    if rows > 2:
        z[2, : vocab // 2] += 9.0                    # the top K in half of the chunks
    z = z.to(dt)
    ws = torch.empty(L.arbor_uncertainty_workspace_size(rows, vocab, L.BF16 if dtype == "bf16"
                                                        else L.F32),
                     dtype=torch.uint8, device="cuda")
    for k in (0, 1, 2, 40, 84, 85, 86, 200, 256):
        if k >= vocab:
            continue
        got = []
        for _ in range(2):
            u, st = torch.full((rows,), 9.0, device="cuda"), status()
            check_rc(L.arbor_uncertainty(z, k, u, st, ws))
            torch.cuda.synchronize()
            assert int(st) == L.OK
            got.append(u)
        assert torch.equal(got[0], got[1]), k        # reproducible
        assert float((got[0].double() - _want(z, k)).abs().max()) <= 1e-5, k
