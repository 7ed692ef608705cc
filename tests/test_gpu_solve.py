"""The group solves at the edges of their shapes: groups of 2 .. 4 panels, last groups of one to all of their panels,
rows that every panel of a group moves.  (Transposed solves: the adjoint's tests.)"""
import numpy as np
import pytest
import torch

import paper_2311_12134_amd as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[2, 3, 4])
def ctx(request):
    c = P.Context(0)
    for knob in ("group_f32", "group_f64"):
        c.set_knob(knob, request.param)
    yield c
    c.close()


def _scattered(n, rng, chains):
    """A well-conditioned matrix with its rows out of place: at random, or (chains) each panel's 64 rows where
    the next panel's belong and the first's at the end, so that a row moves with every panel of a group."""
    m = 0.3 * (rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))) / np.sqrt(n) + np.eye(n)
    return m[np.roll(np.arange(n), 64) if chains else rng.permutation(n)].copy()


@pytest.mark.parametrize("chains", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "split"])
def test_forward_solves(ctx, precision, chains):
    """Backward error of an LU solve with partial pivoting: n eps times the growth, below 10 sqrt(n) eps here."""
    rng = np.random.default_rng(3)
    eps = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    sizes = [1, 64, 65, 128, 192, 193, 256, 300, 384, 449, 512, 513, 600, 769]
    mats = [_scattered(n, rng, chains) for n in sizes]
    rhs = [rng.normal(size=(n, 16)) + 1j * rng.normal(size=(n, 16)) for n in sizes]
    x = [torch.from_numpy(b).cuda() for b in rhs]
    info = ctx.batched_lu_solve([torch.from_numpy(m).cuda() for m in mats], x, precision=precision).cpu().numpy()
    assert (info == 0).all()
    for m, b, v in zip(mats, rhs, x):
        v = v.cpu().numpy()
        back = np.linalg.norm(m @ v - b) / (np.linalg.norm(m) * np.linalg.norm(v))
        assert back <= 10 * np.sqrt(len(m)) * eps, (len(m), back)
