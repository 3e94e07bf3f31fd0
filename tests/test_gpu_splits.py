"""Work splits of the non-causal calls: the row segments walked by the apply,
row and key passes are chosen apart from the state segments, so shapes whose
two splits differ (short and long slices, a ragged last segment, a last
segment of one row) are compared with the float64 oracle.  Their row segments
are one tile long; longer ones are in test_gpu_long_walks.py."""

import pytest

from fmm_testlib import check_full
from test_gpu_backward import check_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rank", [1, 3])
@pytest.mark.parametrize("B,H,N,d", [(4, 2, 1025, 32), (1, 3, 4161, 16), (1, 2, 2111, 64)])
def test_backward_walk_apart_from_state_segments(B, H, N, d, rank, dtype):
    check_backward(B, H, N, d, 20, rank, 0, dtype, 2600 + N + rank, std=2.0 / d ** 0.5,
                   joint=rank == 3)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("B,H,N,d", [(1, 1, 65, 128), (2, 1, 1281, 128), (1, 2, 2049, 64),
                                     (1, 1, 4095, 16)])
def test_forward_few_state_segments(B, H, N, d, causal, dtype):
    # fewer segments than CUs: shorter state segments than the record rule's
    check_full(B, H, N, d, 20, 2, causal, dtype, 2700 + N + causal, std=1.0 / d ** 0.5)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_backward_few_state_segments(dtype):
    check_backward(1, 2, 1153, 64, 20, 2, 1, dtype, 2800, std=0.25)
    check_backward(1, 1, 700, 128, 5, 2, 1, dtype, 2801, std=0.18)
