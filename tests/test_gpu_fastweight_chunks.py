"""The chunked fast-weight kernels where chunks, passes and ranges end: lengths
around the 16-position chunk against the float64 oracle; a forward whose
slices take two passes against calls on its parts, bit for bit; and one slice
of more chunks than a pass holds, whose state crosses from one range to the
next."""

import numpy as np
import pytest
import torch

from fmm_testlib import log
from paper_2108_02347_amd import binding
from test_gpu_fastweight import check_fw, check_fw_backward

pytestmark = pytest.mark.gpu

PASS_FLOATS = (1 << 30) // 4  # workspace of one forward pass
CHUNK_FLOATS = 5 * 16 * 16 + 16 * 16 + 16 + 2 * 16  # of one chunk at d = 16


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_chunk_edges(d, dtype):
    for i, n in enumerate((15, 16, 17, 33, 65)):
        check_fw(1, 3, n, d, 4, i % 2, dtype, 4800 + d + i)
        check_fw_backward(1, 3, n, d, 4, i % 2, dtype, 4900 + d + i)


def _inputs(B, H, N, d, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v = (torch.randn(B, H, N, d, device="cuda", generator=g) for _ in range(3))
    beta = torch.rand(B, H, N, device="cuda", generator=g)
    return q, k, v, beta, torch.randn(H, device="cuda", generator=g)


def test_slices_in_two_passes():
    H, N, d = 8, 16, 16
    B = PASS_FLOATS // CHUNK_FLOATS // H + 37  # one chunk per slice
    q, k, v, beta, w = _inputs(B, H, N, d, 1)
    log(f"two passes: {B * H} slices of {N}")
    out = binding.forward_fastweight(q, k, v, beta, w, w, 3, 1)
    for b0 in (0, B // 2, B - 50):
        part = [x[b0:b0 + 50].contiguous() for x in (q, k, v, beta)]
        assert torch.equal(out[b0:b0 + 50], binding.forward_fastweight(*part, w, w, 3, 1))


def test_state_carried_between_ranges():
    # writes stop after 64 positions, so W stays as it is and only z grows:
    # fw_i = W_63 p(q_i) / (z_i . p(q_i)).  Error: z is a running sum of N / 16
    # = 170000 chunk sums, each addition off by at most half a unit of z (3e-8
    # to 6e-8 of it) and mostly to either side: sqrt(N / 16) 6e-8 = 2.5e-5, and
    # four times that as the bound
    d = 16
    N = PASS_FLOATS // CHUNK_FLOATS * 16 + 1000
    q, k, v, beta, _ = _inputs(1, 1, N, d, 2)
    beta[:, :, 64:] = 0
    near, far = (torch.full((1,), x, device="cuda") for x in (-float("inf"), float("inf")))
    log(f"one slice of {N}")
    out = binding.forward_fastweight(q, k, v, beta, near, far, 0, 0)[0, 0]

    def p(x):
        f = torch.where(x > 0, x + 1, x.double().exp())
        return f / f.sum(-1, keepdim=True)

    W = np.zeros((d, d))
    pk = p(k[0, 0, :64].double()).cpu().numpy()
    for i in range(64):
        u = v[0, 0, i].double().cpu().numpy() - W @ pk[i]
        W += float(beta[0, 0, i]) * np.outer(u, pk[i])
    z = torch.cumsum(p(k[0, 0].double()), 0)
    rows = torch.cat([torch.arange(64, 200), torch.arange(N - 1200, N)]).cuda()
    pq = p(q[0, 0, rows].double())
    want = pq @ torch.from_numpy(W).cuda().T / (z[rows] * pq).sum(-1, keepdim=True)
    err = (out[rows].double() - want).norm(dim=-1) / want.norm(dim=-1)
    log(f"  worst row {err.max():.2e}")
    assert float(err.max()) < 1e-4


def _dbeta_stepwise(q, k, v, beta, f, t):
    """dbeta of sum(f * fw) by the recurrence, one step per position, in the
    arithmetic of t; all slices [S, N, d] together."""
    q, k, v, beta, f = (np.asarray(x).astype(t) for x in (q, k, v, beta, f))

    def p(x):
        phi = np.where(x > 0, x + t(1), np.exp(np.minimum(x, t(0))))
        return phi / phi.sum(-1, keepdims=True)

    def dot(x, y):  # [S, d, d] or [S, 1, d] times [S, d]
        return np.matmul(x, y[..., None])[..., 0]

    pq, pk = p(q), p(k)
    s, n, d = q.shape
    w, z = np.zeros((s, d, d), t), np.zeros((s, d), t)
    e, den = [], []
    for i in range(n):
        e.append(v[:, i] - dot(w, pk[:, i]))
        w = w + (beta[:, i, None] * e[-1])[..., None] * pk[:, i, None]
        z = z + pk[:, i]
        den.append((z * pq[:, i]).sum(-1, keepdims=True))
    g, db = np.zeros((s, d, d), t), np.zeros((s, n), t)
    for i in range(n - 1, -1, -1):
        g = g + (f[:, i] / den[i])[..., None] * pq[:, i, None]
        lam = dot(g, pk[:, i])
        db[:, i] = (lam * e[i]).sum(-1)
        g = g - (beta[:, i, None] * lam)[..., None] * pk[:, i, None]
    return db


@pytest.mark.parametrize("N,d", [(64, 16), (100, 32), (48, 64), (33, 128)])
def test_dbeta_no_less_exact_than_single_steps(N, d):
    # the yardstick is the recurrence itself in fp32: solving a chunk's
    # triangular system must not lose what stepping through it keeps.  Errors
    # are per slice (2-norm, relative), their geometric mean over 96 slices: it
    # varies by about 0.5 / sqrt(96) = 5 % between inputs
    S = 96
    q, k, v, beta, _ = _inputs(S, 1, N, d, 900 + d)
    dout = torch.randn(S, 1, N, d, device="cuda",
                       generator=torch.Generator(device="cuda").manual_seed(d))
    near, far = (torch.full((1,), x, device="cuda") for x in (-float("inf"), float("inf")))
    got = binding.backward_fastweight(q, k, v, beta, dout, near, far, 0, 0)[3]
    got = got[:, 0].double().cpu().numpy()
    x = [y[:, 0].cpu().numpy() for y in (q, k, v, beta, dout)]
    want, step = _dbeta_stepwise(*x, np.float64), _dbeta_stepwise(*x, np.float32)
    err = [np.exp(np.log(np.linalg.norm(y - want, axis=1)
                         / np.linalg.norm(want, axis=1)).mean()) for y in (got, step)]
    log(f"dbeta N={N} d={d}: {err[0]:.3e}, in single steps {err[1]:.3e}")
    assert err[0] <= err[1]
