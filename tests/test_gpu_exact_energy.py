"""Exact energy of Eq. (5) against the FP64 oracle where its row walk can go wrong: balls across faces and far
beyond them, radii from the smallest to ones with more rows than a workgroup has lanes, anisotropic
spacing, centres on voxels and faces; and values that are not finite just outside the ball.

The image is the raw FP32 volume (no low-pass), so both sides sum the same FP64 terms: what is left is the
readback's FP32 rounding (2^-24 relative to the energy) and FP64 rounding of a few thousand terms (below 1e-11
of the sum of their magnitudes).
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch   # before the library: the process then has one HIP runtime
    assert torch.cuda.is_available(), "GPU tests need a GPU"


def _finalize(p, raw, cen, R):
    from paper_1804_06304_amd import snk
    ctx = snk.Context(0)
    ctx.set_params(p)
    ctx.set_directions(synth.directions_for(p.dim, p.n_dirs))
    ctx.load_volume(raw)
    ctx.load_seeds(cen)
    n = len(cen)
    ctx.set_state(cen, R, np.full(n, 1, np.int32), np.full(n, 2, np.uint8))
    ctx.prepass()
    ctx.finalize()
    out = ctx.read()
    ctx.close()
    return out["e_vox"]


def _params(dim, h):
    return synth.Params(dim=dim, spacing=h, sigma_pre=0.0, dR=0.8, r_max=40.0, r_init=5.0,
                        n_dirs=64 if dim == 2 else 162)


def _contours(dim, shape, h):
    top = (np.array(shape[::-1]) - 1.0) * h
    rng = np.random.default_rng(dim)
    cen = [top / 2, np.floor(top / (2 * np.array(h))) * h, 0 * top, top, top * [1, 0, 0.5]]
    cen += [rng.uniform(0, 1, 3) * top for _ in range(11)]
    cen = np.array(cen)
    cen[:, dim:] = 0.0
    lo = 0.8 * (1 + 2 ** (-1 / dim)) / (2 * (1 - 2 ** (-1 / dim)))
    R = np.concatenate([[lo, 5.0, 6.0, 7.0, 8.0, 25.0, 39.0], rng.uniform(lo, 20.0, 9)])
    return cen, R.astype(np.float32)


@pytest.mark.parametrize("dim,shape,h", [(3, (23, 37, 41), (1.0, 1.0, 2.0)), (3, (30, 20, 26), (1.0, 1.25, 0.8)),
                                         (2, (1, 53, 47), (1.0, 1.0, 1.0)), (2, (1, 64, 33), (1.0, 0.7, 1.0))])
def test_exact_energy_matches_oracle(orc, dim, shape, h):
    rng = np.random.default_rng(7)
    raw = rng.uniform(-1.0, 1.0, shape).astype(np.float32)
    p = _params(dim, h)
    cen, R = _contours(dim, shape, h)
    got = _finalize(p, raw, cen, R)
    want, mag = orc.energy_vox(raw.astype(np.float64), p, cen, R.astype(np.float64))
    # the device holds a centre as anchor + FP32 offset: 2^-25 voxel, times the steepest weight (2 / (rho dR), 3.6 a
    # unit) relative to the weights' magnitude
    tol = 2.0 ** -24 * np.abs(want) + (2.0 ** -25 * 3.6 * 2 + 1e-11) * mag
    assert np.all(np.abs(got - want) <= tol), np.max(np.abs(got - want) / tol)


def test_values_outside_the_ball_do_not_count(orc):
    """NaN and infinities everywhere beyond R + dR/2 leave the energy what it is with zeros there."""
    shape, p = (33, 33, 33), _params(3, (1.0, 1.0, 1.0))
    c, R = np.array([[16.3, 15.8, 16.1]]), np.array([9.0], np.float32)
    z, y, x = np.meshgrid(*(np.arange(s) for s in shape), indexing="ij")
    far = np.sqrt((x - c[0, 0]) ** 2 + (y - c[0, 1]) ** 2 + (z - c[0, 2]) ** 2) > 9.4 + 1e-4
    raw = np.random.default_rng(3).uniform(0.0, 1.0, shape).astype(np.float32)
    clean = np.where(far, 0.0, raw).astype(np.float32)
    bad = np.where(far, np.where((x + y) % 2 == 0, np.nan, np.inf), raw).astype(np.float32)
    a, b = _finalize(p, clean, c, R), _finalize(p, bad, c, R)
    assert np.isfinite(a[0]) and a[0] == b[0]
    inside = bad.copy()
    inside[16, 16, 16] = np.nan
    assert np.isnan(_finalize(p, inside, c, R)[0])
