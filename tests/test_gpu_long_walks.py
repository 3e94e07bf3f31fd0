"""Walks of three and more 64-row tiles per workgroup: the non-causal apply, row
and key passes take one tile each until B H N exceeds 32768, so shapes beyond
that are run whole and two of their slices (the first and the last) compared with
the float64 oracle.  128 slices of 699 rows: four row segments per slice, three
of three tiles and a last one of two, the second ragged, in the state segments of
the causal forms as in the apply split.  The bands lie on both sides of the
128-row rings (non-causal 32, causal 64)."""

import pytest
import torch

from fmm_testlib import TOL, TORCH_DT, log, slice_errors
from oracle import fmm_ref as ref
from paper_2108_02347_amd import binding

pytestmark = pytest.mark.gpu

B, H, N = 64, 2, 699
ENDS = [0, B - 1]


def _tiles():
    rows = -(-N // -(-512 // (B * H)))  # about 512 workgroups
    return -(-rows // 64)


def _inputs(d, dtype, seed):
    """q, k, v, dout, w_near, w_far on the GPU, drawn there (a whole shape in
    float64 on the host would take most of the tests' time)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = [(torch.randn(B, H, N, d, device="cuda", generator=g) * s).to(TORCH_DT[dtype])
         for s in (2.0 / d ** 0.5,) * 3 + (1.0,)]
    return x + [torch.randn(H, device="cuda", generator=g) for _ in range(2)]


def _ends(x):
    return x[ENDS].double().cpu().numpy()


def _host(x):
    return x.double().cpu().numpy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [16, 32, 64])
@pytest.mark.parametrize("causal,kw", [(0, 32), (0, 33), (1, 64), (1, 65)])
def test_backward(causal, kw, d, dtype):
    assert _tiles() == 3
    q, k, v, g, wn, wf = _inputs(d, dtype, 6000 + d + kw)
    rank = 3 if kw in (33, 64) else 2
    log(f"backward {B}x{H} slices of {N}, d={d} k={kw} r={rank} causal={causal} {dtype}")
    got = binding.backward(q, k, v, g, wn, wf, kw, rank, causal, joint=rank == 3)
    want = ref.fmm_attention_backward_stream(*map(_ends, (q, k, v)), *map(_host, (wn, wf)),
                                             _ends(g), kw, rank, bool(causal),
                                             norm="joint" if rank == 3 else "map")
    errs = [slice_errors(_ends(a), b).max() for a, b in zip(got[:3], want[:3])]
    log("  " + " ".join(f"{e:.2e}" for e in errs))
    assert max(errs) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,rank,joint", [(32, 3, True), (64, 2, True), (128, 2, False),
                                          (128, 1, True)])
@pytest.mark.parametrize("causal", [0, 1])
def test_general_apply(causal, d, rank, joint, dtype):
    # k_wide and, for bf16 heads of 128, k_wide128 with rings of one and two units
    # of band
    assert _tiles() == 3
    q, k, v, _, wn, wf = _inputs(d, dtype, 6300 + d + rank)
    for kw in (20, 33, 64):
        log(f"forward {B}x{H} slices of {N}, d={d} k={kw} r={rank} joint={joint} "
            f"causal={causal} {dtype}")
        got = binding.forward(q, k, v, wn, wf, kw, rank, causal, joint=joint)
        want = ref.fmm_attention_stream(*map(_ends, (q, k, v)), *map(_host, (wn, wf)), kw, rank,
                                        bool(causal), norm="joint" if joint else "map")
        err = slice_errors(_ends(got), want).max()
        log(f"  {err:.2e}")
        assert err <= TOL[dtype]


@pytest.mark.parametrize("causal,kw", [(0, 20), (1, 64)])
def test_backward_width_128(causal, kw):
    q, k, v, g, wn, wf = _inputs(128, "bf16", 6600 + kw)
    log(f"backward {B}x{H} slices of {N}, d=128 k={kw} causal={causal}")
    got = binding.backward(q, k, v, g, wn, wf, kw, 2, causal)
    want = ref.fmm_attention_backward_stream(*map(_ends, (q, k, v)), *map(_host, (wn, wf)),
                                             _ends(g), kw, 2, bool(causal))
    errs = [slice_errors(_ends(a), b).max() for a, b in zip(got[:3], want[:3])]
    log("  " + " ".join(f"{e:.2e}" for e in errs))
    assert max(errs) <= TOL["bf16"]
