"""The split-mode wide update from pairs of FP16 numbers (the default tiling for blocks of at
least 512 rows) against NumPy in 64 bits and against the FP32 matrix-core tilings: FP32 factors
without refinement, so the update's own error shows."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# with four panels per group the first wide update has npad - 256 rows: 448 (the FP32 tiling's last
# size), 512 and 576 (the rule's first two, an even and an odd number of 64-row halves), and
# sizes whose later groups cross the rule; uneven batches share a launch
BATCHES = {"edges": [704, 768, 832], "uneven": [1100, 833, 769, 700, 65, 1], "long": [1800]}


def _solve(ctx, tiling, mats, rhs):
    x = [torch.from_numpy(b).cuda() for b in rhs]
    ctx.set_gemm_tiling(tiling)
    try:
        info = ctx.batched_lu_solve([torch.from_numpy(m).cuda() for m in mats], x, precision="split").cpu().numpy()
    finally:
        ctx.set_gemm_tiling(-1)
    return [v.cpu().numpy() for v in x], list(info)


@pytest.fixture(scope="module")
def ctx():
    import paper_2311_12134_amd as P
    c = P.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("batch", sorted(BATCHES))
@pytest.mark.parametrize("scale", ["plain", "rows", "columns", "tiny", "huge"])
def test_pairs_are_no_less_exact_than_fp32(ctx, batch, scale):
    """Rows or columns 2^-30 .. 2^30 apart and whole systems near the ends of FP32's range: the pair
    update's error must not exceed the FP32 matrix cores' by more than the scatter between two
    roundings (a factor of 1.5), and stay within n eps32 of a well-conditioned solve."""
    print("[gpu] half2", batch, scale, flush=True)
    rng = np.random.default_rng(len(batch) + len(scale))
    mats, rhs = [], []
    for n in BATCHES[batch]:
        m = 0.7 * (rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))) / np.sqrt(2 * n) + np.eye(n)
        x = rng.normal(size=(n, 3)) + 1j * rng.normal(size=(n, 3))
        if scale == "rows":
            m = m * np.exp2(rng.integers(-30, 31, (n, 1)))
        elif scale == "columns":
            # x_j as small as its column is large, so that every column counts alike in B (an unknown
            # whose column vanishes in B's rounding is beyond any LU); powers of two commute with
            # every rounding of the LU, so the plain system's bound holds
            c = np.exp2(rng.integers(-30, 31, (1, n)))
            m, x = m * c, x / c.T
        elif scale in ("tiny", "huge"):
            m = m * (2.0 ** -110 if scale == "tiny" else 2.0 ** 110)
        mats.append(m)
        rhs.append(m @ x)
    (pair, info), (fp32, info32) = _solve(ctx, 19, mats, rhs), _solve(ctx, 2, mats, rhs)
    assert not any(info) and not any(info32)
    for m, b, p, f in zip(mats, rhs, pair, fp32):
        ref = np.linalg.solve(m, b)
        # columns of unlike scale: each unknown relative to the size it has
        unit = np.abs(ref).max(axis=1, keepdims=True)
        err = [np.linalg.norm((v - ref) / unit) / np.linalg.norm(ref / unit) for v in (p, f)]
        assert err[0] <= 1.5 * err[1] + 1e-12, (len(m), err)
        # backward error of the LU, about n^(1/2) eps32, times the condition: |M^-1| |M| < 20 here; rows
        # of unlike scale meet pivots of unlike rows, which may grow it tenfold more
        assert err[0] <= 20 * np.sqrt(len(m)) * 2.0 ** -24 * (100 if scale == "rows" else 1), (len(m), err)


def test_zero_blocks_and_non_finite_rows(ctx):
    """The identity (L21 and U12 all zero) is solved exactly; a NaN in one system of a batch stays
    in that system."""
    rng = np.random.default_rng(3)
    eye = np.eye(900, dtype=np.complex128)
    good = 0.7 * (rng.normal(size=(900, 900)) + 1j * rng.normal(size=(900, 900))) / 43 + eye
    bad = good.copy()
    bad[800, 5] = np.nan
    b = rng.integers(-100, 100, (900, 2)) + 1j * rng.integers(-100, 100, (900, 2))
    (x, info), (x32, info32) = (_solve(ctx, t, [eye, bad, good], [b, b, b]) for t in (19, 2))
    assert info == info32 and info[0] == info[2] == 0
    assert np.array_equal(x[0], b)
    assert np.array_equal(np.isnan(x[1]), np.isnan(x32[1])) and np.isnan(x[1]).any()
    assert np.abs(good @ x[2] - b).max() <= 1e-4 * np.abs(b).max()
