"""Launches at the limit of the LDS that they are accepted by: the kernels take up to 5.5 KB more than the rule counts
(most with 102 rays), the largest boxes and ray counts are launched, and the next larger ones refused.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch   # before the library: the process then has one HIP runtime
    assert torch.cuda.is_available(), "GPU tests need a GPU"


def _evolved(dim, M, lanes, tile, n=20):
    from paper_1804_06304_amd import snk
    rng = np.random.default_rng(dim)
    shape = (1, 80, 90) if dim == 2 else (30, 40, 44)
    raw = rng.integers(0, 200, shape).astype(np.uint8)
    p = synth.Params(dim=dim, i_scale=1 / 160.0, r_init=6.5, r_max=14.0, n_dirs=64 if dim == 2 else 162, n_rays=M)
    ctx = snk.Context(0)
    ctx.set_params(p)
    ctx.set_directions(synth.directions_for(dim, p.n_dirs))
    ctx.set_launch(lanes, 2, 0)
    ctx.set_tile(tile)
    ctx.load_volume(raw)
    ctx.load_seeds(rng.uniform(0, 1, (12, 3)) * (np.array(shape[::-1]) - 1.0))
    try:
        ctx.evolve(n)
        out = ctx.get_state()
        assert ctx.get_timing()["tile_voxels"] == tile
    except snk.SnkError as e:
        assert "LDS" in str(e)
        out = None
    ctx.close()
    return out


@pytest.mark.parametrize("dim,lanes,largest", [(2, 64, 15520), (2, 128, 15504), (2, 256, 14624), (3, 64, 15520),
                                               (3, 128, 15500), (3, 256, 14616)])
def test_largest_box(dim, lanes, largest):
    out, ref = _evolved(dim, 102, lanes, largest), _evolved(dim, 102, lanes, 0)
    assert _evolved(dim, 102, lanes, largest + 1, 1) is None
    for k in ref:
        assert np.array_equal(out[k], ref[k]), k


@pytest.mark.parametrize("dim,lanes,most", [(2, 64, 2042), (2, 256, 2038), (3, 128, 2038), (3, 256, 2036)])
def test_most_rays(dim, lanes, most):
    out = _evolved(dim, most, lanes, 0, 6)
    assert np.all(out["iters"][out["status"] == 0] == 6)
    assert _evolved(dim, most + 2, lanes, 0, 1) is None
