"""Automatic boxes of 256 lanes in 3D: two waves do their work where the balls fit the box that 8 contours of a CU leave
each other, four waves with the larger box of fewer contours where they do not. The bits are those of no box.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch   # before the library: the process then has one HIP runtime
    assert torch.cuda.is_available(), "GPU tests need a GPU"


def _run(R, M, lanes=0, tile=-1, iters=20, n=2600):
    from paper_1804_06304_amd import snk
    rng = np.random.default_rng(3)
    shape = (44, 60, 66)
    z, y, x = np.meshgrid(*(np.arange(s) for s in shape), indexing="ij")
    raw = np.clip(100 + 60 * np.sin(x / 5.0) * np.cos(y / 6.0) * np.cos(z / 4.0) + rng.normal(0, 8, shape), 0, 255).astype(np.uint8)
    cen = rng.uniform(0, 1, (n, 3)) * (np.array(shape[::-1]) - 1.0)   # 2,600: 11 per CU, beyond 10 of two waves
    p = synth.Params(dim=3, i_offset=20.0, i_scale=1 / 160.0, dR=0.75, r_init=R, r_max=2 * R, n_dirs=162, n_rays=M)
    ctx = snk.Context(0)
    ctx.set_params(p)
    ctx.set_directions(synth.directions_for(3, 162))
    ctx.set_launch(lanes, 2 if lanes else 0, 0)
    ctx.set_tile(tile)
    ctx.load_volume(raw)
    ctx.load_seeds(cen)
    ctx.evolve(iters)
    t = ctx.get_timing()
    ctx.finalize()
    out = ctx.read()
    ctx.close()
    return t, out


# a ball of R takes about (2 R + dR + 2)^3 voxels of a box; 8 contours leave each other some 4,400, 4 twice that
@pytest.mark.parametrize("R,M,least,most", [(6.0, 64, 4000, 4800), (8.0, 64, 6600, 16384), (8.0, 70, 6600, 16384),
                                            (14.0, 64, 4800, 16384)])
def test_box_of_256_lanes(R, M, least, most):
    t, out = _run(R, M)
    assert t["lanes_per_contour"] == 256 and least <= t["tile_voxels"] <= most, t
    _, ref = _run(R, M, 256, 0)
    for k in out:
        assert np.array_equal(out[k], ref[k]), k


@pytest.mark.parametrize("R,M,n,iters,box", [(6.0, 64, 2600, 15, False), (6.0, 64, 2600, 16, True), (8.0, 64, 2600, 5, False),
                                             (14.0, 64, 2600, 5, True), (6.0, 32, 5200, 15, False), (6.0, 32, 5200, 16, True),
                                             (6.0, 64, 2000, 5, True), (6.0, 64, 16000, 6, False), (6.0, 64, 16000, 7, True)])
def test_short_launches_take_no_box(R, M, n, iters, box):
    """More contours than can be resident, launches too short to repay the staging; balls beyond the box stage nothing."""
    t, out = _run(R, M, iters=iters, n=n)
    assert (t["tile_voxels"] > 0) == box, t
    _, ref = _run(R, M, t["lanes_per_contour"], 0, iters, n)
    for k in out:
        assert np.array_equal(out[k], ref[k]), k
