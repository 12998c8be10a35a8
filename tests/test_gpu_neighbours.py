"""Neighbour lists of the soft repulsion above the size whose items one workgroup places (8,192 contours).

Contours that lie outside the volume are not live, so adding them changes nothing for the others: the same
4,150 contours must evolve bit for bit alike alone and followed by 4,150 contours outside (which take the
other launch route), in 2D and 3D, in a crowd where lists are long.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch   # before the library: the process then has one HIP runtime
    assert torch.cuda.is_available(), "GPU tests need a GPU"


@pytest.mark.parametrize("dim,shape", [(3, (60, 120, 130)), (2, (1, 500, 520))])
def test_lists_do_not_depend_on_the_launch_route(dim, shape):
    from paper_1804_06304_amd import snk
    rng = np.random.default_rng(dim)
    n = 4150
    raw = rng.integers(0, 200, shape).astype(np.uint8)
    D = 64 if dim == 2 else 162
    p = synth.Params(dim=dim, r_max=12.0, r_init=5.0, n_dirs=D, n_rays=16, i_scale=1 / 160.0)
    inside = rng.uniform(0, 1, (n, 3)) * (np.array(shape[::-1]) - 1.0)
    inside[:, dim:] = 0.0
    out = []
    for seeds in (inside, np.concatenate([inside, inside - 1000.0 * np.array([1, 1, dim == 3])])):
        ctx = snk.Context(0)
        ctx.set_params(p)
        ctx.set_directions(synth.directions_for(dim, D))
        ctx.set_launch(64, 2, 0)
        ctx.set_tile(0)
        ctx.set_repulsion(0.05, 3)
        ctx.load_volume(raw)
        ctx.load_seeds(seeds)
        try:
            ctx.evolve(8)
        except snk.SnkError as e:           # a list longer than 64 is reported, and kept at its 64 lowest
            assert e.code == snk.SNK_ERANGE
        out.append(ctx.get_state())
        ctx.close()
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k][:n]), k
    assert np.all((out[1]["status"][n:] & 0x0F) == 3)
