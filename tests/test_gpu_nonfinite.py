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


@pytest.mark.parametrize("n_linear", [0, 1])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_fast_weight_key_side_reaches_no_earlier_row(d, dtype, n_linear):
    # out_i and dq_i depend on the positions j <= i only: position 9 is planted,
    # the middle of a 16-position chunk, and 40, of a later one
    H, N, kw = 2, 75, 6
    q, k, v, g = _tensors(4, (1, H, N, d), dtype, 7100 + d + n_linear)
    beta = torch.rand(1, H, N, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(d))
    w = torch.zeros(H, device="cuda")
    want = binding.forward_fastweight(q, k, v, beta, w, w, kw, n_linear)
    want_dq = binding.backward_fastweight(q, k, v, beta, g, w, w, kw, n_linear)[0]
    for bad in BAD:
        for name in ("k", "beta"):
            for j in (9, 40):
                log(f"{name}[{j}] = {bad}, d={d} {dtype} n_linear={n_linear}")
                k2, b2 = k.clone(), beta.clone()
                (k2 if name == "k" else b2)[:, 0, j] = bad
                got = binding.forward_fastweight(q, k2, v, b2, w, w, kw, n_linear)
                assert torch.equal(got[:, 0, :j], want[:, 0, :j])
                assert torch.equal(got[:, 1], want[:, 1])
                assert not torch.isfinite(got[:, 0, j].float()).all()
                if name == "beta":  # (k also enters the near field's dq, 32 keys at a time)
                    dq = binding.backward_fastweight(q, k2, v, b2, g, w, w, kw, n_linear)[0]
                    assert torch.equal(dq[:, 0, :j], want_dq[:, 0, :j])
                    assert torch.equal(dq[:, 1], want_dq[:, 1])
