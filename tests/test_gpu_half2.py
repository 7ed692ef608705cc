"""The split-mode wide update from pairs of FP16 numbers (the default tiling of lsms_tau_solve for blocks of at
least 512 rows): the kernels by themselves against NumPy in 64 bits and against an FP32 matrix-core tiling, then
whole solves."""
import numpy as np
import pytest
import torch

import internal_kernels as ik

pytestmark = pytest.mark.gpu
U = 2.0 ** -24

# sizes of the systems (multiples of 64) and columns of the group; rows to either side of the 128-row
# tiles, an odd and an even number of 64-row halves, systems inside the group and one that is all group
BATCHES = {"edges": ([704, 768, 832], 256), "uneven": ([1088, 832, 768, 704, 320, 256, 64], 256),
           "long": ([1792], 256), "two panels": ([768, 640], 128), "three panels": ([960, 704, 192], 192)}


def _matrix(rng, n):
    return rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))


def _updated(mats, kd, update, **kw):
    s = ik.Systems(mats)
    update(s, kd, **kw)
    return s.results()


def _reference(m, kd):
    """The updated block and the sums of moduli |L21| |U12| that scale its rounding."""
    d = m.astype(np.complex64).astype(np.complex128)
    return d[kd:, kd:] - d[kd:, :kd] @ d[:kd, kd:], np.abs(d[kd:, :kd]) @ np.abs(d[:kd, kd:]), np.abs(d[kd:, kd:])


def _bound(sums, c, kd):
    """Operands to 2^-23 each and a dropped product of 2^-22: 2^-21 = 8 U of the sums; 16 products per
    rounding, three of the four parts of a product each for two real sums: 6 kd / 16 roundings of U; the block's
    old values and the difference once more; a real and an imaginary part."""
    return np.sqrt(2) * U * ((8 + 6 * kd / 16) * sums + 2 * (c + sums))


@pytest.mark.parametrize("batch", sorted(BATCHES))
@pytest.mark.parametrize("scale", ["plain", "rows", "columns", "tiny", "huge"])
def test_update_against_float64_and_fp32(batch, scale):
    """Rows or columns 2^-30 .. 2^30 apart and whole systems near the ends of FP32's range.  Every entry
    within the bound of its own sums; over a system of random entries the error must not exceed the FP32 matrix
    cores' by more than the scatter between two roundings (a factor of 1.5)."""
    print("[gpu] pair update", batch, scale, flush=True)
    sizes, kd = BATCHES[batch]
    rng = np.random.default_rng(len(batch) + len(scale))
    mats = []
    for n in sizes:
        m = _matrix(rng, n)
        if scale in ("rows", "columns"):
            d = np.exp2(rng.integers(-30, 31, n))
            # of the whole matrix: row i of L21 and of A22 by d_i, row q of U12 by d_q and column q of L21 by 1 / d_q
            m = m * d[:, None] if scale == "rows" else m * d[None, :]
            if scale == "rows":
                m[kd:, :kd] /= d[None, :kd]
            else:
                m[:kd, kd:] /= d[:kd, None]
        elif scale in ("tiny", "huge"):  # products of two near the ends of the range
            m *= 2.0 ** -60 if scale == "tiny" else 2.0 ** 55
        mats.append(m)
    for at_once in (1, len(mats)):  # groups of jobs through the scratch
        pair = _updated(mats, kd, ik.pair_update, jobs_at_once=at_once)
        fp32 = _updated(mats, kd, ik.fp32_update)
        for m, p, f in zip(mats, pair, fp32):
            if len(m) <= kd:
                assert np.array_equal(p, m.astype(np.complex64))
                continue
            ref, sums, c = _reference(m, kd)
            assert np.array_equal(p[:kd], m[:kd].astype(np.complex64))
            assert np.array_equal(p[:, :kd], m[:, :kd].astype(np.complex64))
            err, err32 = np.abs(p[kd:, kd:] - ref), np.abs(f[kd:, kd:] - ref)
            assert (err <= _bound(sums, c, kd)).all(), (len(m), (err / sums).max() / U)
            assert np.linalg.norm(err / sums) <= 1.5 * np.linalg.norm(err32 / sums), len(m)


@pytest.mark.parametrize("p", [20, 40, 60])
@pytest.mark.parametrize("first", [0, 100, 300, 700])
def test_rows_whose_large_entries_lie_in_few_columns(p, first):
    """Rows of U12 2^p times larger than the others in 64 columns and zero elsewhere: their scale has to come
    from those columns, or the other rows' entries there are lost for rows of L21 that touch only those."""
    n, kd = 1024, 256
    rng = np.random.default_rng(first + p)
    m = _matrix(rng, n)
    keep = m[:128, kd + first:kd + first + 64] * 2.0 ** p
    m[:128, kd:] = 0
    m[:128, kd + first:kd + first + 64] = keep
    m[kd:, :128] *= 2.0 ** -p
    m[kd::2, :128] = 0
    ref, sums, c = _reference(m, kd)
    err = np.abs(_updated([m], kd, ik.pair_update)[0][kd:, kd:] - ref)
    assert (err <= _bound(sums, c, kd)).all(), (err / sums).max() / U


@pytest.mark.parametrize("value", [1 + 2.0 ** -11, 1 + 2.0 ** -11 + 2.0 ** -23, 1 + 2.0 ** -12, 1.5])
def test_unfavourable_operands(value):
    """All entries alike and halfway between two FP16 numbers, so that every dropped product has the same sign and
    the largest size, 2^-22 of the product (random operands: a tenth of that on average)."""
    n, kd = 768, 256
    m = np.full((n, n), value) * np.exp2(np.random.default_rng(1).integers(-3, 4, (n, n))) * (1 + 0j)
    ref, sums, c = _reference(m, kd)
    err = np.abs(_updated([m], kd, ik.pair_update)[0][kd:, kd:] - ref)
    assert (err <= _bound(sums, c, kd)).all(), (err / sums).max() / U


def test_update_in_two_parts_and_lower_half_are_bitwise_the_same():
    """The look-ahead's split at the next panel's columns; the symmetric form's tiles on and below the diagonal
    (of a tile on the diagonal the 64 x 64 block above it stays as it is)."""
    rng = np.random.default_rng(2)
    kd = 256
    mats = [_matrix(rng, n) * np.exp2(rng.integers(-8, 9, (n, n))) for n in (1088, 832, 320)]
    whole = _updated(mats, kd, ik.pair_update)
    s = ik.Systems(mats)
    ik.pair_update(s, kd, c_end=kd + 64)
    ik.pair_update(s, kd, c_begin=kd + 64)
    lower = _updated(mats, kd, ik.pair_update, lower=True)
    for m, w, two, low in zip(mats, whole, s.results(), lower):
        assert np.array_equal(w, two)
        i, j = np.indices(m.shape)
        kept = (i < kd) | (j < kd) | ((j - kd) // 64 > (i - kd) // 64)
        assert np.array_equal(low, np.where(kept, m.astype(np.complex64), w))


def test_zero_blocks_and_non_finite_rows():
    """L21 and U12 all zero change nothing; a NaN or an infinity in one system of a batch stays in that
    system, and makes the entries NaN that depend on it."""
    rng = np.random.default_rng(3)
    n, kd = 896, 256
    eye = np.eye(n) * (1 + 0j)
    good = _matrix(rng, n)
    bad = [good.copy() for _ in range(3)]
    bad[0][kd + 7, 5] = np.nan
    bad[1][5, kd + 9] = np.nan
    bad[2][5, kd + 9] = np.inf
    out = _updated([eye, bad[0], good, bad[1], bad[2]], kd, ik.pair_update)
    alone = _updated([good], kd, ik.pair_update)[0]
    assert np.array_equal(out[0], eye.astype(np.complex64)) and np.array_equal(out[2], alone)
    for got, where in ((out[1], np.s_[7, :]), (out[3], np.s_[:, 9]), (out[4], np.s_[:, 9])):
        hit = np.zeros((n - kd, n - kd), bool)
        hit[where] = True
        assert np.array_equal(np.isnan(got[kd:, kd:]), hit)
        # the other entries within the bound (the NaN's or infinity's own row or column has no scale of its own)
        ref, sums, c = _reference(good, kd)
        assert (np.abs(got[kd:, kd:] - ref) <= _bound(sums, c, kd))[~hit].all()


def _cluster(radius):
    """LIZ of a finite bcc cluster, so that the systems of one batch differ in size."""
    import paper_2311_12134_amd as P
    a = 5.7
    grid = np.array([(i, j, k) for i in range(5) for j in range(5) for k in range(5)], dtype=np.float64)
    pos = np.concatenate([grid, grid + 0.5]) * a
    inner = [62, 187, 0, 31, 124, 93, 186]
    liz = P.build_liz(pos, None, radius * a, centres=inner)
    assert len(set(np.diff(liz.ptr)[inner])) > 2
    return liz, torch.from_numpy(np.random.default_rng(4).uniform(-0.5, 0.5, (len(pos), 4))).cuda()


@pytest.mark.parametrize("radius", [1.7, 2.1, 2.2])
def test_unrefined_solutions(radius):
    """tau_solve without corrections returns the FP32 factors' solution (any backward error is accepted): with
    pairs no less exact than with an FP32 tiling, up to the scatter between two roundings (a factor of 1.5), in
    systems of up to 832, 1088 and 1472 rows, and a system in a wave of unlike ones as exact as by itself."""
    import paper_2311_12134_amd as P
    from paper_2311_12134_amd.api import Liz
    liz, phase = _cluster(radius)
    ctx = P.Context(0)
    atom, dpos = liz.to_device(ctx.device)
    want = ctx.tau_solve(liz, atom, dpos, phase, 0.65, 0.01, precision="fp64")[0].cpu().numpy()

    def errors(tiling):
        ctx.set_gemm_tiling(tiling)
        tp, _, info, berr = ctx.tau_solve(liz, atom, dpos, phase, 0.65, 0.01, precision="split", refine_tol=1.0,
                                          max_refine=0)
        assert int(info.abs().max()) == 0 and 0 < float(berr.max()) < 1e-5
        d = tp.cpu().numpy() - want
        return np.array([np.linalg.norm(d[b:e]) / np.linalg.norm(want[b:e])
                         for b, e in zip(liz.ptr[:-1], liz.ptr[1:]) if e > b])

    pair, fp32 = errors(19), errors(2)
    assert (pair != fp32).any()
    assert (pair <= 1.5 * fp32.max()).all(), (pair, fp32)
    ctx.set_gemm_tiling(19)
    for c in np.flatnonzero(np.diff(liz.ptr)):  # by itself, where a small system keeps to the FP32 tiling
        part, b = slice(liz.ptr[c], liz.ptr[c + 1]), np.zeros(len(liz.ptr), np.int64)
        b[c + 1:] = liz.ptr[c + 1] - liz.ptr[c]
        one = Liz(b, liz.atom[part], liz.pos[part])
        a1, p1 = one.to_device(ctx.device)
        tp = ctx.tau_solve(one, a1, p1, phase, 0.65, 0.01, precision="split", refine_tol=1.0, max_refine=0)[0]
        assert np.linalg.norm(tp.cpu().numpy() - want[part]) <= 1.5 * fp32.max() * np.linalg.norm(want[part])
    ctx.close()


@pytest.mark.parametrize("radius", [1.7, 2.1, 2.2])
def test_symmetric_factorization(radius):
    """The lower-triangle form of the update at edges of its 128-row tiles: LIZ of a finite bcc cluster, so the
    systems of one batch differ in size (up to 832, 1088 and 1472 rows), against the FP64 LU.  Refined to a backward
    error of 1e-14, the solutions differ by that times the condition (below 1e3 here)."""
    import paper_2311_12134_amd as P
    liz, phase = _cluster(radius)
    ctx = P.Context(0)
    atom, dpos = liz.to_device(ctx.device)
    want = ctx.tau_solve(liz, atom, dpos, phase, 0.65, 0.01, precision="fp64")[:2]
    ctx.set_symmetric(True)
    tp, tm, info, berr = ctx.tau_solve(liz, atom, dpos, phase, 0.65, 0.01, precision="split")
    assert int(info.abs().max()) == 0 and float(berr.min()) >= 0  # no system fell back to the FP64 LU
    for got, ref in zip((tp, tm), want):
        assert float((got - ref).norm() / ref.norm()) <= 1e-11
    ctx.close()
