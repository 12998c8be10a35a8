"""Which copy of a 2D image an automatic evolve reads (3: column pairs, 1: plain), by what it does: boxes are staged
from the plain copy, gathers without a box read pairs with half the loads unless the pairs overflow the L2 by far. The
copy follows the evolve that comes, whatever the pre-pass wrote for another one, and the bits do not depend on it.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
SHAPE = (1, 500, 530)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch   # before the library: the process then has one HIP runtime
    assert torch.cuda.is_available(), "GPU tests need a GPU"


def _context(M, R, layout=0, lanes=0, flags=0, star=None, tile=-1):
    from paper_1804_06304_amd import snk
    y, x = np.meshgrid(np.arange(SHAPE[1]), np.arange(SHAPE[2]), indexing="ij")
    rng = np.random.default_rng(M)
    raw = np.clip(100 + 60 * np.sin(x / 9.0) * np.cos(y / 11.0) + rng.normal(0, 8, SHAPE[1:]), 0, 255).astype(np.uint8)[None]
    p = synth.Params(dim=2, i_offset=20.0, i_scale=1 / 160.0, r_init=R, r_max=2 * R, n_dirs=64, n_rays=M, flags=flags)
    ctx = snk.Context(0)
    ctx.set_params(p)
    ctx.set_directions(synth.directions_for(2, 64))
    ctx.set_launch(lanes, 0, layout)
    ctx.set_tile(tile)
    if star is not None:
        ctx.set_star(star)
    ctx.load_volume(raw)
    return ctx


def _evolve(ctx, n):
    rng = np.random.default_rng(n)
    ctx.load_seeds(rng.uniform(0, 1, (n, 3)) * (np.array(SHAPE[::-1]) - 1.0))
    ctx.evolve(9)
    ctx.finalize()
    t = ctx.get_timing()
    return ctx.read(), t["layout"], t["tile_voxels"] > 0


# 256 CUs: boxes from 1,025 contours. The pairs of 20 waves a CU with R 17 take 6.7 MiB of an XCD's L2, with R 18 7.4
@pytest.mark.parametrize("kw,n,layout,box", [
    (dict(M=16, R=9.0), 1025, 1, True), (dict(M=16, R=9.0), 1024, 3, False), (dict(M=8, R=9.0), 1100, 3, False),
    (dict(M=64, R=9.0), 1300, 3, False), (dict(M=64, R=40.0), 1300, 1, True), (dict(M=16, R=17.0), 5300, 3, False),
    (dict(M=16, R=18.0), 5300, 1, False), (dict(M=16, R=9.0, lanes=32), 1100, 3, False),
    (dict(M=16, R=9.0, star=0.3), 1100, 3, False), (dict(M=16, R=9.0, flags=2), 1100, 1, False),
    (dict(M=16, R=9.0, flags=4), 1100, 1, True), (dict(M=16, R=9.0, tile=0), 1100, 3, False)])
def test_copy_and_box(kw, n, layout, box):
    ctx = _context(**kw)
    out, *got = _evolve(ctx, n)
    ctx.close()
    assert got == [layout, box]
    lanes = kw.get("lanes") or (128 if "star" in kw else (256 if kw["M"] == 64 or kw.get("flags") == 2 else 64))
    ctx = _context(**{**kw, "layout": 1, "lanes": lanes, "tile": 0})   # plain, no box
    ref, *_ = _evolve(ctx, n)
    ctx.close()
    for k in out:
        assert np.array_equal(out[k], ref[k]), k


@pytest.mark.parametrize("then", ["fewer seeds", "box off", "star", "pre-pass first"])
def test_copy_follows_the_evolve(then):
    """Pairs for an evolve that reads them, after a pre-pass that had no use for them, and the other way round."""
    star = 0.3 if then == "star" else None
    fresh = _context(16, 9.0, star=star, tile=0 if then == "box off" else -1)
    n = 300 if then == "fewer seeds" else 1200
    want, *expect = _evolve(fresh, n)
    fresh.close()
    ctx = _context(16, 9.0)
    if then == "pre-pass first":
        ctx.prepass()                       # no contours yet: pairs
        out, *got = _evolve(ctx, n)
        assert got == expect == [1, True]
        small, *got = _evolve(ctx, 200)
        assert got == [3, False]
    else:
        _, *got = _evolve(ctx, 1200)
        assert got == [1, True]
        if then == "box off":
            ctx.set_tile(0)
        if then == "star":
            ctx.set_star(star)
        out, *got = _evolve(ctx, n)
        assert got == expect == [3, False]
        for layout in (2, 3, 0):            # quads, 64-bit plain, and back
            ctx.set_launch(0, 0, layout)
            again, *_ = _evolve(ctx, n)
            for k in out:
                assert np.array_equal(again[k], want[k]), (layout, k)
    ctx.close()
    for k in out:
        assert np.array_equal(out[k], want[k]), k
