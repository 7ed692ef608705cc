"""The symmetric factorization by itself: without pivoting an exact zero on the diagonal has to be reported, so that
lsms_tau_solve recomputes the system by an LU with pivoting."""
import numpy as np
import pytest
import torch

import internal_kernels as ik

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tall_rows", [64, 4096])  # panels as a diagonal block and L21, and whole
@pytest.mark.parametrize("n", [64, 192, 320])
def test_exact_zero_pivots_are_reported_at_their_column(n, tall_rows):
    """[[0, 1], [1, 0]] on the diagonal: before any elimination, in the leaves of the first and of later panels and in the
    last column, beside systems without one; and a zero that the elimination leaves."""
    print("[gpu] zero pivots of the symmetric form", n, tall_rows, flush=True)
    rng = np.random.default_rng(n)
    cols = [c for c in (0, 5, 31, 32, 62, 64, 100, 150, 190, 256, 318) if c + 1 < n]
    mats = []
    for c in cols:
        m = np.eye(n) * (1 + 0j)
        m[c, c] = m[c + 1, c + 1] = 0
        m[c, c + 1] = m[c + 1, c] = 1
        mats.append(m)
    left = np.eye(n) * (1 + 0j)
    left[3, n - 1] = left[n - 1, 3] = 1  # 1 - 1 * 1
    regular = 0.1 * (rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))) / np.sqrt(n)
    regular = regular + regular.T + np.eye(n)
    s = ik.Systems(mats + [left, regular, np.eye(n) * (1 + 0j)])
    ik.ldlt(s, tall_rows)
    assert s.info.cpu().tolist() == [c + 1 for c in cols] + [n, 0, 0]
    # the factors of the regular system: L below the diagonal, U above; the panels' diagonal blocks hold inverses
    f = s.results()[-2].astype(np.complex128)
    assert np.isfinite(f).all()


def test_many_systems_as_few():
    """600 systems in one call, whose panels of 64 rows take one wavefront each, and the same three by themselves."""
    rng = np.random.default_rng(4)
    mats = []
    for n in (64, 128, 192):
        m = 0.3 * (rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))) / np.sqrt(n)
        mats.append(m + m.T + np.eye(n))
    mats[1][70, 70] = mats[1][70, :70] @ np.linalg.solve(mats[1][:70, :70], mats[1][:70, 70])  # nearly singular minor
    few, many = ik.Systems(mats), ik.Systems(mats * 200)
    ik.ldlt(few, 64)
    ik.ldlt(many, 64)
    want = few.results()
    assert many.info.cpu().tolist() == few.info.cpu().tolist() * 200
    for i, got in enumerate(many.results()):
        assert np.array_equal(got, want[i % 3], equal_nan=True)
