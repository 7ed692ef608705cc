"""Caller matrices whose rows or columns differ by many powers of two, with zero blocks between them: FP32 factors
without refinement keep their accuracy, since scaling by powers of two commutes with every rounding of an
FP32 LU (up to the choice of pivots, which stay within their blocks here)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

N, P, Q, T = 1024, slice(0, 128), slice(128, 256), slice(256, 1024)


def _matrix(kind, p, first, rng):
    S = slice(256 + first, 256 + first + 64)  # a few columns past the first group of panels
    m = 0.7 * (rng.normal(size=(N, N)) + 1j * rng.normal(size=(N, N))) / np.sqrt(2 * N) + np.eye(N)
    x = rng.normal(size=(N, 3)) + 1j * rng.normal(size=(N, 3))
    m[P, Q] = m[Q, P] = 0
    if kind == "rows":
        # rows P, 2^p times larger, reach the trailing columns in S only; the rows below do not touch them
        keep = m[P, S].copy()
        m[P, T] = 0
        m[P, S] = keep
        m[T, P] = 0
        m[P] *= 2.0 ** p
    else:
        # columns S, 2^p times larger, which rows P do not reach
        m[P, S] = 0
        m[:, S] *= 2.0 ** p
        x[S] /= 2.0 ** p
    return m, x


@pytest.mark.parametrize("p", [0, 20, 40, 60])
@pytest.mark.parametrize("kind,first", [("rows", 300), ("columns", 300), ("columns", 224)])
def test_blocks_of_unlike_scale(kind, first, p):
    import paper_2311_12134_amd as lsms
    print("[gpu] LU of blocks of unlike scale", kind, first, p, flush=True)
    m, x = _matrix(kind, p, first, np.random.default_rng(7))
    ctx = lsms.Context(0)
    got = torch.from_numpy(m @ x).cuda()
    info = ctx.batched_lu_solve([torch.from_numpy(m).cuda()], [got], precision="split")
    assert int(info.abs().max()) == 0
    unit = np.abs(x).max(axis=1, keepdims=True)
    err = np.linalg.norm((got.cpu().numpy() - x) / unit) / np.linalg.norm(x / unit)
    # the backward error of an LU, about n^(1/2) eps32, times the condition (below 20)
    assert err <= 20 * np.sqrt(N) * 2.0 ** -24, err
    ctx.close()
