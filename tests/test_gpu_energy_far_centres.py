"""Exact energy of contours whose centre is no place: seeds may be anywhere, and one outside the volume stops as OUT,
but the final energies are formed for every contour. Centres beyond the range of integers, infinite ones and ones that
are not numbers have no lattice point inside their ball: energy 0, and the others' results are what they are alone.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

FAR = [5e9, 1e12, 1e30, 1e300, np.inf, np.nan, -5e9, -1e30, -np.inf]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch   # before the library: the process then has one HIP runtime
    assert torch.cuda.is_available(), "GPU tests need a GPU"


def _case(dim):
    shape = (20, 30, 34) if dim == 3 else (1, 40, 44)
    raw = np.random.default_rng(dim).uniform(-1.0, 1.0, shape).astype(np.float32)
    p = synth.Params(dim=dim, sigma_pre=0.0, dR=0.75, r_max=12.0, r_init=6.0, n_dirs=64 if dim == 2 else 162, n_rays=16)
    mid = np.array([15.25, 14.5, 9.75 if dim == 3 else 0.0])
    cen = [mid]
    for a in range(dim):
        for v in FAR:
            c = mid.copy()
            c[a] = v
            cen.append(c)
    return raw, p, np.array(cen + [mid + [8.5, 3.0, 0.0]])


def _check(out, alone, n):
    assert np.all(out["status"][1:-1] == 3)     # OUT
    assert np.all(out["e_vox"][1:-1] == 0.0), out["e_vox"]
    assert np.all(out["keep"][1:-1] == 0)
    for k in ("radii", "centers", "e_mc", "e_vox", "iters", "status", "keep"):
        assert np.array_equal(out[k][[0, n - 1]], alone[k]), k


@pytest.mark.parametrize("dim", [2, 3])
def test_far_centres(orc, dim):
    from paper_1804_06304_amd import snk
    raw, p, cen = _case(dim)
    n = len(cen)
    res = []
    for sel in (slice(None), [0, n - 1]):
        ctx = snk.Context(0)
        ctx.set_params(p)
        ctx.set_directions(synth.directions_for(dim, p.n_dirs))
        ctx.load_volume(raw)
        ctx.load_seeds(cen[sel], ids=np.arange(n, dtype=np.uint32)[sel])
        ctx.evolve(5)
        ctx.finalize()
        res.append(ctx.read())
        ctx.close()
    _check(res[0], res[1], n)
    want, mag = orc.energy_vox(raw.astype(np.float64), p, res[1]["centers"], res[1]["radii"].astype(np.float64))
    # a centre is read back exactly; 2^-24: the readback; 1e-11: FP64 rounding of a few thousand terms
    assert np.all(np.abs(res[1]["e_vox"] - want) <= 2.0 ** -24 * np.abs(want) + 1e-11 * mag)


def test_far_centres_in_the_engine():
    from paper_1804_06304_amd import snk
    raw, p, cen = _case(3)
    n = len(cen)
    D = synth.directions_for(3, p.n_dirs)
    res = []
    for sel in (slice(None), [0, n - 1]):
        e = snk.Engine(0, None, 1 << 30)
        e.set_launch(64, 1, 0, 0)
        j = e.submit(p, D, raw, cen[sel], ids=np.arange(n, dtype=np.uint32)[sel], n_iter=5)
        e.run()
        res.append(e.read(j))
        e.close()
    _check(res[0], res[1], n)
