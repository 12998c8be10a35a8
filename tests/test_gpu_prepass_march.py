"""The pre-pass of images with more rows of tiles than the chip holds workgroups, where a workgroup marches down several
of them, its next tile's loads in flight: odd sizes that no tile and no chunk divides, against the FP64 oracle and, for
the column pairs, the bits that evolve to. Quad records are not marched. Bound of |J - oracle| as in the test of the
tiles' edges: an axis of radius r rounds 2 r + 1 products and their taps, the intensity map twice.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch   # before the library: the process then has one HIP runtime
    assert torch.cuda.is_available(), "GPU tests need a GPU"


def _run(p, raw, layout, cen):
    from paper_1804_06304_amd import snk
    ctx = snk.Context(0)
    ctx.set_params(p)
    ctx.set_directions(synth.directions_for(2, 64))
    ctx.set_launch(64, 2, layout)
    ctx.load_volume(raw)
    ctx.prepass()
    J = ctx.read_volume(raw.shape)
    ctx.load_seeds(cen)
    ctx.evolve(3)
    st = ctx.get_state()
    ctx.close()
    return J, st


# tiles are 64 columns by 16 rows and the chip holds at most 2,048 workgroups: 65 x 257 tiles (9 rows a workgroup), 17 x
# 376, 3 x 2,050; radii 3 (its own kernel), 6, 9 (of the largest kernel), 1 and 0
@pytest.mark.parametrize("ny,nx,dtype,sigma", [(4099, 4111, np.uint8, 1.0), (6011, 1037, np.uint16, 2.0),
                                               (4099, 4111, np.float32, 0.3), (32797, 131, np.uint8, 3.0),
                                               (4100, 4090, np.uint16, 0.0)])
def test_marching(orc, ny, nx, dtype, sigma):
    rng = np.random.default_rng(ny + nx)
    raw = rng.uniform(0.0, 250.0, (1, ny, nx)).astype(dtype)
    p = synth.Params(dim=2, sigma_pre=sigma, dR=0.8, r_max=8.0, r_init=4.0, n_rays=16, n_dirs=64)
    cen = rng.uniform(0.0, 1.0, (400, 3)) * [nx - 1, ny - 1, 0]
    cen[:4] = [[nx - 1, ny - 1, 0], [0, 0, 0], [nx - 1, 0, 0], [0, ny - 1, 0]]
    ref = orc.prepass(raw, p)
    r = int(np.ceil(3.0 * sigma))
    bound = (3 * (2 * r + 2) + 2) * 2.0 ** -24 * raw.max()
    first = None
    for layout in (1, 4, 2):   # plain, pairs, quads
        print(ny, nx, np.dtype(dtype).name, sigma, "layout", layout, flush=True)
        J, st = _run(p, raw, layout, cen)
        assert np.max(np.abs(J - ref)) <= bound
        first = first or st
        for k in st:
            assert np.array_equal(st[k], first[k], equal_nan=True), k
