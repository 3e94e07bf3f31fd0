"""The forward's split into state segments, seen through the workspace of its
plan: one record of rank * d * (d + 1) floats per segment and one per slice.  No
GPU is used."""

import ctypes

import pytest

from paper_2108_02347_amd import binding


def plan_bytes(B, H, N, d, rank, causal, bf16):
    f = binding.lib()._ZN3fmm23forward_workspace_bytesEiiiiiiii  # fmm::forward_workspace_bytes
    f.restype = ctypes.c_size_t
    return f(B, H, N, d, 5, rank, causal, int(bf16))


def segments(B, H, N, d, rank, causal=1):
    rec = rank * d * (d + 1) * 4
    return max(plan_bytes(B, H, N, d, rank, causal, t) for t in (0, 1)) // rec - B * H


@pytest.mark.parametrize("B,H,N,d,rank,most", [
    # one slice: no more segments than its combine walks at once (fp32 causal:
    # one per CU); 64-row segments of these took twice as long
    (1, 1, 20000, 16, 2, 256), (1, 1, 30000, 32, 2, 256),
    # several: at most one workgroup per CU, not a second round that is mostly
    # idle (376 workgroups: 1.2 to 1.3 times as long as 232 or 250)
    (2, 4, 9000, 64, 2, 256), (1, 2, 40000, 64, 2, 256), (2, 4, 9000, 128, 1, 256),
])
def test_shorter_segments_stay_within_one_round(B, H, N, d, rank, most):
    assert 150 <= segments(B, H, N, d, rank) <= most


def test_segments_fill_the_chip():
    # 16 workgroups with a quarter-size record rule; at least four times as many
    assert segments(1, 2, 5000, 64, 2) >= 64
    # and within the no-allocation call's array wherever the quarter rule was
    assert plan_bytes(2, 4, 16381, 128, 2, 1, 1) <= binding.noalloc_max_bytes()
