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


@pytest.mark.parametrize("radius", [1.7, 2.1, 2.2])
def test_symmetric_factorization(radius):
    """The lower-triangle form of the update at edges of its 128-row tiles: LIZ of a finite bcc cluster, so the
    systems of one batch differ in size (up to 832, 1088 and 1472 rows), against the FP64 LU.  Refined to a backward
    error of 1e-14, the solutions differ by that times the condition (below 1e3 here)."""
    import paper_2311_12134_amd as P
    a = 5.7
    grid = np.array([(i, j, k) for i in range(5) for j in range(5) for k in range(5)], dtype=np.float64)
    pos = np.concatenate([grid, grid + 0.5]) * a
    inner = [62, 187, 0, 31, 124, 93, 186]
    ctx = P.Context(0)
    liz = P.build_liz(pos, None, radius * a, centres=inner)
    assert len(set(np.diff(liz.ptr)[inner])) > 2
    atom, dpos = liz.to_device(ctx.device)
    phase = torch.from_numpy(np.random.default_rng(4).uniform(-0.5, 0.5, (len(pos), 4))).cuda()
    want = ctx.tau_solve(liz, atom, dpos, phase, 0.65, 0.01, precision="fp64")[:2]
    ctx.set_symmetric(True)
    tp, tm, info, berr = ctx.tau_solve(liz, atom, dpos, phase, 0.65, 0.01, precision="split")
    assert int(info.abs().max()) == 0 and float(berr.min()) >= 0  # no system fell back to the FP64 LU
    for got, ref in zip((tp, tm), want):
        assert float((got - ref).norm() / ref.norm()) <= 1e-11
    ctx.close()
