"""Exact energy of radii below the smallest admissible one, where the inner ramp of the weight reaches into the outer
one: snk_set_state takes any radius in (0, r_max], and a larger dR set later leaves the loaded radii as they are.

Against the FP64 oracle, whose weight takes the four regions in order. Spacing, dR, radii and centres are binary
fractions, so both sides hold the same numbers and what differs is the readback's FP32 rounding (2^-24 relative)
and FP64 rounding of a few hundred terms (below 1e-11 of the sum of their magnitudes).
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch   # before the library: the process then has one HIP runtime
    assert torch.cuda.is_available(), "GPU tests need a GPU"


def _case(dim):
    shape = (24, 30, 36) if dim == 3 else (1, 40, 50)
    h = (1.0, 0.75, 1.25) if dim == 3 else (1.0, 0.75, 1.0)
    rng = np.random.default_rng(dim)
    raw = rng.uniform(-1.0, 1.0, shape).astype(np.float32)
    dR = 0.75
    least = dR * (1 + 2 ** (-1 / dim)) / (2 * (1 - 2 ** (-1 / dim)))
    cen = np.floor(rng.uniform(0, 1, (40, 3)) * (np.array(shape[::-1]) - 1.0) * 64) / 64   # voxels
    cen[:, dim:] = 0.0
    # as shares of the least radius: far below, where both ramps overlap, just below, at and above it
    share = np.tile([0.1, 0.3, 0.5, 0.7, 0.9, 0.99, 1.01, 2.0], 5)
    R = (np.floor(share * least * 4096) / 4096).astype(np.float32)
    return raw, h, dR, cen * np.array(h), R


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("how", ["set_state", "larger dR"])
def test_exact_energy_below_the_smallest_radius(orc, dim, how):
    from paper_1804_06304_amd import snk
    raw, h, dR, cen, R = _case(dim)
    n = len(R)
    D = 64 if dim == 2 else 162
    p = synth.Params(dim=dim, spacing=h, sigma_pre=0.0, dR=dR, r_max=40.0, r_init=8.0, n_dirs=D)
    ctx = snk.Context(0)
    ctx.set_params(p if how == "set_state" else p.replace(dR=0.03125))
    ctx.set_directions(synth.directions_for(dim, D))
    ctx.load_volume(raw)
    if how == "set_state":
        ctx.load_seeds(cen)
        ctx.set_state(cen, R, np.full(n, 1, np.int32), np.full(n, 2, np.uint8))
    else:
        R = np.maximum(R, np.float32(0.5))   # admissible with the small dR
        ctx.load_seeds(cen, r0=R)
        ctx.set_params(p)
    ctx.finalize()
    out = ctx.read()
    ctx.close()
    assert np.array_equal(out["radii"], R)
    want, mag = orc.energy_vox(raw.astype(np.float64), p, cen, R.astype(np.float64))
    tol = 2.0 ** -24 * np.abs(want) + 1e-11 * mag
    assert np.all(np.abs(out["e_vox"] - want) <= tol), np.max(np.abs(out["e_vox"] - want) / tol)
