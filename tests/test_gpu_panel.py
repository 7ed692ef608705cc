"""The panel factorization at the edges of its shapes: heights where the workgroup size, the row
slots per thread or the leaf width change, pivots that move every row far, ties, exact zeros."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# heights of the first panel (n rounded up to 64): one row slot of 256 and of 512 threads, 2 .. 8 slots
SIZES = [1, 63, 64, 65, 256, 257, 320, 512, 513, 768, 769, 1024, 1025, 1536, 1537, 2048, 2049, 2561]


@pytest.fixture(scope="module")
def ctx():
    import paper_2311_12134_amd as P
    c = P.Context(0)
    yield c
    c.close()


def _solve(ctx, mats, rhs, precision):
    x = [torch.from_numpy(b).cuda() for b in rhs]
    info = ctx.batched_lu_solve([torch.from_numpy(m).cuda() for m in mats], x, precision=precision).cpu().numpy()
    return [v.cpu().numpy() for v in x], info


@pytest.mark.parametrize("precision", ["fp64", "split"])
@pytest.mark.parametrize("kind", ["reversed", "ties"])
def test_panel_shapes(ctx, precision, kind):
    """reversed: a well-conditioned matrix with its rows in reverse order, so that every column's pivot
    comes from the other end; ties: entries of equal magnitude only.  The backward error of an LU with
    partial pivoting is n eps times the growth (below 10 n^(1/2) for these)."""
    rng = np.random.default_rng(5)
    eps = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    for lo in range(0, len(SIZES), 6):  # uneven batches
        print("[gpu] panel shapes", kind, precision, SIZES[lo:lo + 6], flush=True)
        mats, rhs = [], []
        for n in SIZES[lo:lo + 6]:
            if kind == "reversed":
                m = (0.5 * (rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))) / np.sqrt(n) + np.eye(n))[::-1]
            else:
                m = np.array([1, 1j, -1, -1j])[rng.integers(0, 4, (n, n))]
            mats.append(m.copy())
            rhs.append(rng.normal(size=(n, 2)) + 1j * rng.normal(size=(n, 2)))
        got, info = _solve(ctx, mats, rhs, precision)
        for m, b, x, i in zip(mats, rhs, got, info):
            n = len(m)
            if kind == "ties" and i != 0:
                assert np.linalg.matrix_rank(m) < n, n  # small ones may be singular
                continue
            back = np.linalg.norm(m @ x - b) / (np.linalg.norm(m) * np.linalg.norm(x))
            assert i == 0 and back <= 10 * np.sqrt(n) * eps, (n, i, back)


@pytest.mark.parametrize("precision", ["fp64", "split"])
def test_zero_pivot_is_reported_at_its_column(ctx, precision):
    """A zero column met in the first and in the second leaf of the first and of a later panel."""
    rng = np.random.default_rng(6)
    cols = [0, 5, 40, 63, 64, 150, 299]
    mats, rhs = [], []
    for c in cols:
        m = rng.normal(size=(300, 300)) + 1j * rng.normal(size=(300, 300))
        m[:, c] = 0
        mats.append(m)
        rhs.append(np.ones((300, 1), dtype=np.complex128))
    _, info = _solve(ctx, mats, rhs, precision)
    assert list(info) == [c + 1 for c in cols]


def test_multiples_of_the_pivot_row_cancel_as_with_a_division(ctx):
    """Constant real and imaginary 2 x 2 matrices in FP64: the second pivot is v - (v (1 / v)) v with a correctly
    rounded 1 / v, an exact zero for most v."""
    values = [v * f for v in range(1, 300) for f in (1, 1j, -1, 0.1)]
    _, info = _solve(ctx, [np.full((2, 2), v, dtype=np.complex128) for v in values],
                     [np.ones((2, 1), dtype=np.complex128)] * len(values), "fp64")
    size = np.abs(np.array(values))
    assert np.array_equal(info, np.where(size * (1.0 / size) == 1.0, 2, 0))


@pytest.mark.parametrize("chunk", [2048, 64])  # with 64, panels of more than 128 rows by tournament
def test_infinite_pivots_in_fp64(ctx, chunk):
    """An infinite entry on the diagonal takes its unknown out of the system: that one is 0 and the others are those of
    the system without it (backward error of the LU, n eps, times a condition below 20)."""
    rng = np.random.default_rng(7)
    ctx.set_tslu_chunk(chunk)
    try:
        for n in (8, 70, 300, 700):
            for where in ([0], [5], [n - 1], [0, 3, n // 2]):
                print("[gpu] infinite pivots", chunk, n, where, flush=True)
                m = 0.5 * (rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))) / np.sqrt(2 * n) + np.eye(n)
                keep = np.setdiff1d(np.arange(n), where)
                ref = np.linalg.solve(m[np.ix_(keep, keep)], np.ones((len(keep), 1)))
                m[where, where] = np.inf
                (x,), info = _solve(ctx, [m], [np.ones((n, 1), dtype=np.complex128)], "fp64")
                assert info[0] == 0 and (x[where] == 0).all()
                assert np.abs(x[keep] - ref).max() <= 20 * n * 2.0 ** -53 * np.abs(ref).max()
    finally:
        ctx.set_tslu_chunk(2048)


@pytest.mark.parametrize("precision", ["fp64", "split"])
def test_many_small_systems_as_few(ctx, precision):
    """600 systems of up to 64 rows in one call, whose FP32 panels take one wavefront each, and in two calls: bitwise the
    same, singular ones and ties among them."""
    rng = np.random.default_rng(8)
    mats, rhs = [], []
    for i in range(600):
        n = 64 if i % 3 == 0 else int(rng.integers(1, 65))
        m = rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))
        if i % 7 == 0:
            m = rng.integers(-1, 2, (n, n)) + 1j * rng.integers(-1, 2, (n, n))
        if i % 11 == 0:
            m[:, rng.integers(n)] = 0
        mats.append(m.astype(np.complex128))
        rhs.append(rng.normal(size=(n, 2)) + 1j * rng.normal(size=(n, 2)))
    x, info = _solve(ctx, mats, rhs, precision)
    halves = [_solve(ctx, mats[h], rhs[h], precision) for h in (slice(0, 300), slice(300, 600))]
    assert np.array_equal(info, np.concatenate([h[1] for h in halves])) and (info != 0).any() and (info == 0).any()
    for a, b in zip(x, halves[0][0] + halves[1][0]):
        assert np.array_equal(a, b, equal_nan=True)
    eps = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    for m, b, v, i in zip(mats, rhs, x, info):
        if i == 0 and np.linalg.matrix_rank(m) == len(m):
            back = np.linalg.norm(m @ v - b) / (np.linalg.norm(m) * np.linalg.norm(v))
            assert back <= 10 * np.sqrt(len(m)) * eps, (len(m), back)


def test_few_tall_systems_look_ahead_bitwise(ctx):
    """One LIZ of 259 members (n = 4160, tournament panels), where the next group's first panel runs on a stream of
    its own, against graph replay, which keeps one stream."""
    import paper_2311_12134_amd as P
    cells, a = 8, 5.7
    grid = np.array([(i, j, k) for i in range(cells) for j in range(cells) for k in range(cells)], dtype=np.float64)
    pos = np.concatenate([grid, grid + 0.5]) * a
    liz = P.build_liz(pos, np.eye(3) * cells * a, 3.001 * a, centres=[0])
    assert liz.ptr[1] == 259
    atom, dpos = liz.to_device(ctx.device)
    phase = torch.from_numpy(np.random.default_rng(2).uniform(-0.6, 0.6, (len(pos), 4))).cuda()
    got = []
    for graphs in (False, True, True, False):
        ctx.set_graphs(graphs)
        tp, tm, info, _ = ctx.tau_solve(liz, atom, dpos, phase, 0.65, 0.005, precision="split")
        torch.cuda.synchronize()
        assert int(info.abs().max()) == 0
        got.append((tp.clone(), tm.clone()))
    ctx.set_graphs(False)
    for tp, tm in got[1:]:
        assert torch.equal(tp, got[0][0]) and torch.equal(tm, got[0][1])
