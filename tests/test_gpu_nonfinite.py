"""A NaN or infinity reaches only what depends on it.  The causal forms work on
tiles, where a masked weight is a zero that a product still multiplies with the
masked element's value; so a non-finite input at one position is planted and
every result that must not depend on it is compared, bit for bit, with the
result of the same call on finite inputs."""

import pytest
import torch

from fmm_testlib import TORCH_DT, log
from paper_2108_02347_amd import binding

pytestmark = pytest.mark.gpu

BAD = [float("nan"), float("inf")]


def _tensors(n, shape, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn(*shape, device="cuda", generator=g).to(TORCH_DT[dtype])
            for _ in range(n)]


@pytest.mark.parametrize("joint", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,rank", [(16, 1), (32, 2), (64, 3), (128, 2)])
def test_backward_query_side_reaches_no_later_key(d, rank, dtype, joint):
    # dk_j and dv_j sum over the rows i >= j.  The near field works on 32 rows
    # at a time, so the keys from 32 on (of a 64-row tile, and the tiles after
    # it) are held to independence from row 5.
    H, N, kw = 2, 200, 7
    q, k, v, g = _tensors(4, (1, H, N, d), dtype, 7000 + d + rank)
    w = torch.zeros(H, device="cuda")
    want = binding.backward(q, k, v, g, w, w, kw, rank, 1, joint=joint)
    for bad in BAD:
        for name in ("q", "dout"):
            log(f"{name}[5] = {bad}, d={d} rank={rank} {dtype} joint={joint}")
            q2, g2 = q.clone(), g.clone()
            (q2 if name == "q" else g2)[:, 0, 5] = bad
            got = binding.backward(q2, k, v, g2, w, w, kw, rank, 1, joint=joint)
            for what, a, b in zip(("dk", "dv"), got[1:3], want[1:3]):
                assert torch.equal(a[:, 0, 32:], b[:, 0, 32:]), what
                assert torch.equal(a[:, 1], b[:, 1]), what
