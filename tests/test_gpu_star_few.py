"""Star contours have a kernel for few contours and one for many: a contour's result does not depend on its company,
so the same contours evolved alone and among more than the first kernel takes must agree bit for bit, for direction
tables and ray counts on either side of what it keeps in registers.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch   # before the library: the process then has one HIP runtime
    assert torch.cuda.is_available(), "GPU tests need a GPU"


def _evolve(p, dirs, raw, cen, ids, lanes, layout):
    from paper_1804_06304_amd import snk
    ctx = snk.Context(0)
    ctx.set_params(p)
    ctx.set_launch(lanes, 0, layout)
    ctx.set_star(0.3)
    ctx.set_directions(dirs)
    ctx.load_volume(raw)
    ctx.prepass()
    ctx.load_seeds(cen, ids=ids)
    ctx.evolve(7)    # in two calls: radii and draws carry over
    ctx.evolve(12)
    out, radii = ctx.get_state(), ctx.get_star_radii()
    ctx.close()
    return out, radii


# 64 lanes keep tables of up to 384 directions and 128 rays
@pytest.mark.parametrize("dim,lanes,D,M,layout", [(3, 128, 642, 64, 0), (3, 64, 162, 32, 1), (3, 64, 642, 32, 0),
                                                  (3, 64, 162, 130, 0), (3, 128, 162, 34, 2), (2, 128, 64, 16, 0),
                                                  (2, 64, 64, 18, 1)])
def test_few_equals_many(dim, lanes, D, M, layout):
    rng = np.random.default_rng(5)
    shape = (40, 44, 48) if dim == 3 else (1, 90, 80)
    raw = rng.integers(0, 250, shape).astype(np.uint8)
    p = synth.Params(dim=dim, sigma_pre=1.0, dR=0.8, r_max=9.0, r_init=4.0, n_rays=M, n_dirs=D, conv_window=0)
    n = 8 * 256 // (lanes // 64) + 1
    cen = rng.uniform(0.0, 1.0, (n, 3)) * (np.array(shape[::-1]) - 1.0)
    cen[:, dim:] = 0.0
    ids = np.arange(n, dtype=np.uint32)
    dirs = synth.directions_for(dim, D)
    many, many_r = _evolve(p, dirs, raw, cen, ids, lanes, layout)
    few, few_r = _evolve(p, dirs, raw, cen[::53], ids[::53], lanes, layout)
    assert np.array_equal(few_r, many_r[::53], equal_nan=True)
    for k in few:
        assert np.array_equal(few[k], many[k][::53], equal_nan=True), k
