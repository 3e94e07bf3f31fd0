"""What the calls take of the library-owned workspace, held to limits set
through FMM_ATTN_WS_LIMIT."""

import ctypes

import pytest
import torch

from fmm_testlib import TORCH_DT, log
from paper_2108_02347_amd import binding

pytestmark = pytest.mark.gpu


def _align(x):
    return (x + 255) // 256 * 256


def _preferred(B, H, N, d, kw, rank, causal, dtype):
    """Workspace of the plan that a forward call takes if it may."""
    f = binding.lib()._ZN3fmm23forward_workspace_bytesEiiiiiiii  # fmm::forward_workspace_bytes
    f.restype = ctypes.c_size_t
    return f(B, H, N, d, kw, rank, causal, int(dtype == "bf16"))


def _randn(seed, dtype, *shape, std=1.0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(*shape, device="cuda", generator=g) * std).to(TORCH_DT[dtype])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_layer_takes_only_the_arrays_it_uses(monkeypatch, dtype):
    # with the library's own products: q, k, v and o, in the backward also their
    # gradients; none of the nine arrays that only the rocBLAS form needs
    B, H, N, d, kw = 32, 2, 1024, 16, 5
    E = H * d
    x, dy = (_randn(i, dtype, B, N, E) for i in (1, 2))
    w_qkv, w_out = (_randn(i, dtype, E, c, std=E ** -0.5) for i, c in ((3, 3 * E), (4, E)))
    w = torch.zeros(H, device="cuda")
    array = _align(B * N * E * x.element_size())
    limit = 4 * array + _preferred(B, H, N, d, kw, 1, 0, dtype)
    log(f"layer {dtype}: {limit} bytes forward, {13 * array} backward")
    monkeypatch.setenv("FMM_ATTN_WS_LIMIT", str(limit))
    binding.layer_forward(x, w_qkv, w_out, H, w, w, kw, 1, 0)
    monkeypatch.setenv("FMM_ATTN_WS_LIMIT", str(13 * array))
    binding.layer_backward(x, w_qkv, w_out, dy, H, w, w, kw, 1, 0)
    torch.cuda.synchronize()
