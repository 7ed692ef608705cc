"""The FP64 update's small tiles (launches of few tiles) against the 64 x 64 ones, bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[128], [193, 65, 1], [320, 300, 257], [700, 641, 640, 64], [1100] * 4 + [833] * 5])
def test_few_tiles_match_the_large_tile_bitwise(sizes):
    """Row and column counts that are odd multiples of 64 and of 32-row tiles, uneven batches, the widths of
    narrow (64 columns) and wide updates; tiling 5 never takes the small tile."""
    import paper_2311_12134_amd as P
    rng = np.random.default_rng(len(sizes))
    mats = [rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n)) for n in sizes]
    rhs = [rng.normal(size=(n, 3)) + 1j * rng.normal(size=(n, 3)) for n in sizes]
    ctx = P.Context(0)
    got = []
    for tiling in (-1, 5):
        for knob in ("f64_wide", "f64_narrow"):
            ctx.set_knob(knob, tiling)
        x = [torch.from_numpy(b).cuda() for b in rhs]
        info = ctx.batched_lu_solve([torch.from_numpy(m).cuda() for m in mats], x, precision="fp64")
        assert int(info.abs().max()) == 0
        got.append([v.cpu().numpy() for v in x])
    ctx.close()
    for a, b, m, r in zip(*got, mats, rhs):
        assert (a == b).all()
        assert np.linalg.norm(m @ a - r) <= 1e-11 * np.linalg.norm(m) * np.linalg.norm(a)
