"""The pre-pass against the FP64 oracle at the edges of its tiles (64 columns, 63 with quad records; 16 rows, 8 with
more than 8 z planes to each side) and of its chunks of z, for every class of radii that has a kernel of its own,
and its second copies: contours evolve to the same bits over the plain volume, quad records and column pairs.

Bound of |J - oracle|: an axis of radius r adds 2 r + 1 products of positive taps that sum to one, each rounded
once, of taps rounded once; the intensity map rounds twice. So 3 (2 r + 2) + 2 half ulps of the largest intensity,
r the largest radius.
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
    ctx.set_directions(synth.directions_for(p.dim, p.n_dirs))
    ctx.set_launch(64, 1, layout)
    ctx.load_volume(raw)
    ctx.prepass()
    J = ctx.read_volume(raw.shape)
    ctx.load_seeds(cen)
    ctx.evolve(3)
    st = ctx.get_state()
    ctx.close()
    return J, st


# radii of x, y and z by sigma over spacing: 0; 3 3 2; 3 3 3; 3 2 1; 5 4 4, 8 8 5, 8 7 6; 8 6 8; 12 9 5, 9 9 0; 9 8 9, 16 16 16
CASES = [((5, 17, 65), np.uint8, 0.0, (1, 1, 1)), ((9, 33, 64), np.uint16, 1.0, (1, 1, 2)),
         ((31, 16, 63), np.uint8, 1.0, (1, 1, 1)), ((2, 15, 127), np.float32, 0.9, (1, 1.5, 3)),
         ((40, 18, 130), np.float32, 1.5, (1, 1.2, 1.2)), ((23, 47, 66), np.uint16, 2.6, (1, 1, 1.6)),
         ((18, 31, 70), np.uint8, 2.6, (1, 1.2, 1.4)), ((33, 9, 64), np.float32, 2.6, (1, 1.4, 1)),
         ((19, 34, 65), np.uint16, 3.9, (1, 1.3, 2.6)), ((21, 25, 129), np.float32, 3.0, (1, 1.2, 1)),
         ((12, 8, 30), np.uint8, 5.3, (1, 1, 1)), ((1, 65, 64), np.uint8, 1.0, (1, 1, 1)),
         ((1, 17, 200), np.float32, 2.0, (1, 1, 1)), ((1, 48, 63), np.uint16, 3.0, (1, 1, 1)),
         ((2, 2, 2), np.uint16, 1.6, (1, 1, 1))]


@pytest.mark.parametrize("shape,dtype,sigma,h", CASES)
def test_prepass_at_tile_edges(orc, shape, dtype, sigma, h):
    rng = np.random.default_rng(sum(shape))
    dim = 2 if shape[0] == 1 else 3
    raw = rng.uniform(0.0, 250.0, shape).astype(dtype)
    p = synth.Params(dim=dim, spacing=h, sigma_pre=sigma, dR=0.8, r_max=8.0, r_init=4.0, n_rays=16,
                     n_dirs=64 if dim == 2 else 162)
    top = (np.array(shape[::-1]) - 1.0) * h
    cen = rng.uniform(0.0, 1.0, (24, 3)) * top
    cen[:4] = [top, 0 * top, top * [1, 0, 1], top * [0, 1, 0.5]]
    cen[:, dim:] = 0.0
    ref = orc.prepass(raw, p)
    r = max(int(np.ceil(3.0 * sigma / s)) for s in h)
    bound = (3 * (2 * r + 2) + 2) * 2.0 ** -24 * raw.max()
    first = None
    for layout in (0, 1, 2):
        print(shape, np.dtype(dtype).name, sigma, h, "layout", layout, flush=True)
        J, st = _run(p, raw, layout, cen)
        assert np.max(np.abs(J - ref)) <= bound
        first = first or st
        for k in st:
            assert np.array_equal(st[k], first[k], equal_nan=True), k
