"""bf16 heads of 128 (k_wide128) against the float64 oracle where its dispatch
and its ring turn: both forms, one and two maps, both normalisations, bands at
and past the ring's units, one tile, ragged tails and several segments.  The
causal walks turn the ring here; the non-causal ones take one tile per workgroup
at these lengths, longer ones are in test_gpu_long_walks.py."""

import numpy as np
import pytest
import torch

from fmm_testlib import TOL, check_full, log, slice_errors, upload
from oracle import fmm_ref as ref
from paper_2108_02347_amd import binding
from paper_2108_02347_amd.inputs import make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("rank", [1, 2])
@pytest.mark.parametrize("kw", [0, 31, 32, 33, 64, 65])
def test_bands(kw, rank, causal):
    for i, n in enumerate((1, 63, 65, 700, 1345)):
        check_full(1, 2, n, 128, kw, rank, causal, "bf16", 3000 + 10 * kw + i, std=0.3)


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("rank", [1, 2])
def test_joint(rank, causal):
    q, k, v, wn, wf = make_inputs(2, 2, 777, 128, "bf16", 0.2, 3100 + rank)
    log(f"joint d=128 rank={rank} causal={causal}")
    out = binding.forward(*upload(q, k, v, wn, wf, "bf16"), 40, rank, causal, joint=True)
    torch.cuda.synchronize()
    want = ref.fmm_attention_stream(q, k, v, wn, wf, 40, rank, bool(causal), norm="joint")
    err = slice_errors(out.float().cpu().numpy().astype(np.float64), want).max()
    log(f"  {err:.2e}")
    assert err <= TOL["bf16"]
