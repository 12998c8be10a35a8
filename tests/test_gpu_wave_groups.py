"""Whole-wave evolve kernels at the edges of their draw blocks, passes and launch shapes.

snk_evolve(n) must equal n calls of snk_trace_step bit for bit: the trace runs the general instances one
iteration per launch, so it shares neither the specialised sample loop nor the schedule of the draw blocks.
One iteration against the FP64 oracle is tested in test_gpu_parity.py.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch   # before the library: the process then has one HIP runtime
    assert torch.cuda.is_available(), "GPU tests need a GPU"


def _volume(dim, rng):
    shape = (1, 90, 101) if dim == 2 else (40, 44, 50)
    z, y, x = np.meshgrid(*(np.arange(s) for s in shape), indexing="ij")
    v = 20.0 + rng.normal(0, 8, shape)
    seeds = []
    for c in ((12, 11, 10), (31, 30, 24), (47, 20, 33), (3, 40, 20)):   # the last two near faces
        d2 = (x - c[0]) ** 2 + (y - c[1]) ** 2 + ((z - c[2]) * 1.5) ** 2 * (dim == 3)
        v += 160.0 / (1.0 + np.exp(np.sqrt(d2) - 5.5))
        seeds.append((c[0], c[1], c[2] * 1.5 * (dim == 3)))
    return np.clip(np.rint(v), 0, 255).astype(np.uint8), np.array(seeds) + rng.uniform(-0.5, 0.5, (4, 3)) * [1, 1, dim == 3]


def _context(dim, M, L, lanes, unroll, tile, layout=0):
    from paper_1804_06304_amd import snk
    rng = np.random.default_rng(M * 100 + L)
    raw, seeds = _volume(dim, rng)
    D = 64 if dim == 2 else 162
    p = synth.Params(dim=dim, spacing=(1.0, 1.0, 1.5 if dim == 3 else 1.0), i_offset=20.0, i_scale=1 / 160.0, r_init=6.5,
                     r_max=14.0, n_dirs=D, n_rays=M, n_radial=L)
    ctx = snk.Context(0)
    ctx.set_params(p)
    ctx.set_directions(synth.directions_for(dim, D))
    ctx.set_launch(lanes, unroll, layout)
    ctx.set_tile(tile)
    ctx.load_volume(raw)
    ctx.load_seeds(seeds)
    return ctx


def _same(a, b):
    for k in a:
        assert np.array_equal(a[k], b[k]), k


# pairs per iteration (M / 2): 1 and 5 (blocks of 16 iterations), 16 and 32 (whole passes), 17 and 33 (a ragged pass),
# 65 and 130 (blocks of more passes than a group has waves)
@pytest.mark.parametrize("lanes", [64, 128, 256])
@pytest.mark.parametrize("dim,M,L", [(3, 2, 16), (3, 10, 7), (3, 32, 16), (3, 34, 16), (3, 64, 16), (3, 66, 5),
                                     (3, 130, 16), (3, 260, 3), (2, 2, 16), (2, 16, 16), (2, 34, 9), (2, 130, 16)])
def test_evolve_equals_single_steps(dim, M, L, lanes):
    n = 40
    for unroll in (1, 2):
        one = _context(dim, M, L, lanes, unroll, 0)
        many = _context(dim, M, L, lanes, unroll, 0)
        one.evolve(n)
        for _ in range(n):
            many.trace_step()
        _same(one.get_state(), many.get_state())
        one.close()
        many.close()


@pytest.mark.parametrize("lanes,tile", [(64, 4096), (128, 2048), (128, 15500), (256, 14600)])
def test_box_at_the_lds_limit(lanes, tile):
    """Boxes that leave less of 64 KiB than the kernel's other LDS takes are still accepted."""
    a, b = _context(3, 64, 16, lanes, 2, tile), _context(3, 64, 16, lanes, 2, 0)
    for c in (a, b):
        c.evolve(80)
    assert a.get_timing()["tile_voxels"] == tile
    _same(a.get_state(), b.get_state())
    a.close()
    b.close()


# lanes by the rule of the sums' order: 128 up to 10 contours per CU (256 CUs) with M = 64, else 256; 64 up to 20
# with M = 32, else 128
@pytest.mark.parametrize("dim,n,M,lanes,tiled", [(3, 2049, 64, 128, True), (3, 2560, 64, 128, True),
                                                 (3, 2561, 64, 256, True), (3, 2561, 70, 256, True),
                                                 (3, 2600, 32, 64, True), (3, 5121, 32, 128, True),
                                                 (2, 1025, 16, 64, True), (2, 6200, 16, 64, True),
                                                 (2, 1024, 16, 64, False)])
def test_automatic_boxes_above_the_resident_contours(dim, n, M, lanes, tiled):
    """More contours than stay resident: the automatic shape stages boxes (256 lanes by two waves), in 2D over the
    plain layout, and gives the bits of the same lanes without a box."""
    from paper_1804_06304_amd import snk
    rng = np.random.default_rng(n)
    raw, seeds = _volume(dim, rng)
    top = np.array(raw.shape[::-1]) * [1.0, 1.0, 1.5 if dim == 3 else 1.0] - 1.0
    cen = rng.uniform(0, 1, (n, 3)) * top
    cen[:, dim:] = 0.0
    cen[: len(seeds)] = seeds
    D = 64 if dim == 2 else 162
    p = synth.Params(dim=dim, spacing=(1.0, 1.0, 1.5 if dim == 3 else 1.0), i_offset=20.0, i_scale=1 / 160.0, r_init=6.0,
                     r_max=14.0, n_dirs=D, n_rays=M)
    out = []
    for auto in (True, False):
        ctx = snk.Context(0)
        ctx.set_params(p)
        ctx.set_directions(synth.directions_for(dim, D))
        if not auto:
            ctx.set_launch(lanes, 2, 0)
            ctx.set_tile(0)
        ctx.load_volume(raw)
        ctx.load_seeds(cen)
        ctx.evolve(66)
        t = ctx.get_timing()
        assert t["lanes_per_contour"] == lanes and (t["tile_voxels"] > 0) == (auto and tiled)
        ctx.finalize()
        out.append(ctx.read())
        ctx.close()
    _same(*out)
