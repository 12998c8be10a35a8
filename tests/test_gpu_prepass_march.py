"""The pre-pass of images whose workgroups march down several rows of tiles, the next tile's loads in flight (up to six rows,
where there are more tiles than the chip holds workgroups): odd sizes that no tile and no chunk divides, against the FP64 oracle and, for
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


# tiles are 64 columns by 16 rows, and a workgroup takes up to 6 rows of them: 65 x 257 tiles, 17 x 376, 3 x 2,050; radii 3 (its own kernel), 6, 9 (of the largest kernel), 1 and 0
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


def test_more_rows_of_chunks_than_a_grid_has(orc):
    ny, nx = 7_000_003, 2
    raw = np.random.default_rng(1).uniform(0.0, 250.0, (1, ny, nx)).astype(np.uint8)
    p = synth.Params(dim=2, sigma_pre=1.0, dR=0.8, r_max=8.0, r_init=4.0, n_rays=16, n_dirs=64)
    J, _ = _run(p, raw, 0, np.array([[0.5, 3.5e6, 0.0]]))
    assert np.max(np.abs(J - orc.prepass(raw, p))) <= (3 * 8 + 2) * 2.0 ** -24 * raw.max()
