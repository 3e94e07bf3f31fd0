"""The layer's own projection and weight-gradient kernels (E = 32, 64, 96, 128,
both storage types) at token counts where their tiles and chunks end: fewer
than a 64-token tile, a partial last one, several 256-token chunks with a
ragged last one across batches; and the length of their fp32 sums."""

import numpy as np
import pytest

from fmm_testlib import log
from perf import cases
from test_gpu_layer import check_layer, check_layer_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("E,H", [(32, 1), (64, 4), (96, 3), (128, 8)])
def test_tiles_and_chunks(E, H, dtype):
    for i, (B, N) in enumerate(((1, 5), (3, 67), (2, 643))):
        check_layer(B, N, E, H, 9, 2, i % 2, dtype, 3200 + E + i)
        check_layer_backward(B, N, E, H, 9, 2, i % 2, dtype, 5500 + E + i)


@pytest.mark.parametrize("B,H,N,d,name,most", [
    (32, 2, 4096, 16, "dw_out", 4.26e-7),  # many tokens: 512 of them per chunk
    (32, 2, 4096, 32, "dw_out", 4.62e-7),
    (1, 8, 200, 16, "dx", 4.41e-7),        # the longest contraction, 3 E = 384
])
def test_fp32_sums_as_exact_as_rocblas(B, H, N, d, name, most):
    # most: the error (relative 2-norm, causal) with rocBLAS products in the
    # place of these kernels; one chain of additions per sum gave 4.92, 5.18 and
    # 4.68e-7.  Geometric mean over three inputs, which differ by 3 %
    case = dict(call="layer_train", dtype="f32", B=B, H=H, N=N, d=d, band=20, rank=2, causal=True,
                joint=False, std=1.0)
    errs = []
    for seed in (1, 2, 3):
        got = cases.run(cases.prepare(case, seed))[name].double()
        want = cases.exact(case, seed)[name]
        errs.append(float((got - want).norm() / want.norm()))
    log(f"{name} E={H * d}, {B * N} tokens: {errs}")
    assert np.exp(np.log(errs).mean()) <= most
