"""How many bits the exact energy has: images made so that the energy's terms cancel.

The readback rounds the energy to FP32, 2^-24 relative; where the terms cancel to nothing it shows what the FP64 sum
left instead. With u = 2^-53 and correctly rounded operations, each point's distance r (three roundings of its square,
halved by the root, and the root's) errs by 0.76 u r (rms, a rounding's is u / sqrt 3), its weight by that times the
ramp's slope and by u / sqrt 3 for each of the difference, the quotient and 1/2 minus it. A lane's K terms add up in
K roundings of a partial sum that grows to the lane's share of the magnitude, m / lanes: K / 3 of its full size. 64
lanes add up in a tree, a level of n sums rounding n shares of m / n, and four such waves (3D) one after the other.
These are independent and centred: the tolerance is 4 times their rms, and u times the magnitude for the rounded ramp
width, a factor of every inner weight.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch   # before the library: the process then has one HIP runtime
    assert torch.cuda.is_available(), "GPU tests need a GPU"


def _points(dim, shape, cen, R, dR):
    """Distance, weight and slope of the weight of every voxel, in 80 bits (unit spacing)."""
    ld = np.longdouble
    axes = [np.arange(s, dtype=ld) for s in shape]
    z, y, x = np.meshgrid(*axes, indexing="ij")
    r = np.sqrt((x - ld(cen[0])) ** 2 + (y - ld(cen[1])) ** 2 + ((z - ld(cen[2])) ** 2 if dim == 3 else 0))
    rho = ld(2.0 ** (-1.0 / 3.0) if dim == 3 else np.sqrt(0.5))   # the constant as a double holds it
    R, dR = ld(R), ld(dR)
    a, dr = rho * R, rho * dR
    w = np.where(r < a - dr / 2, ld(-1), np.where(r < a + dr / 2, 2 * (r - a) / dr, np.where(
        r < R - dR / 2, ld(1), np.where(r < R + dR / 2, ld(0.5) - (r - R) / dR, ld(0)))))
    inner = (r >= a - dr / 2) & (r < a + dr / 2)
    outer = (r >= R - dR / 2) & (r < R + dR / 2)
    slope = np.where(inner, 2 / dr, np.where(outer, 1 / dR, 0))
    return r, w, slope


def _cancelled(rng, w):
    """An image whose weighted sum is as near nothing as voxels of FP32 allow."""
    J = rng.uniform(0.0, 1.0, w.shape).astype(np.float32)
    core = np.argwhere(w == -1)
    for at in core[rng.permutation(len(core))[:40]]:
        # a core voxel weighs exactly -1: it takes up what is left, as far as its 24 bits go
        t = tuple(at)
        J[t] = 0.0
        J[t] = np.float32((w * J).sum())
    return J, (w * J).sum()


@pytest.mark.parametrize("dim,R", [(3, 4.5), (3, 9.25), (3, 17.0), (2, 9.5), (2, 30.0)])
def test_cancelled_energy(dim, R):
    from paper_1804_06304_amd import snk
    dR = 0.75
    half = int(R) + 3
    shape = (2 * half,) * 3 if dim == 3 else (1, 2 * half, 2 * half)
    got, tol = [], []
    rng = np.random.default_rng(int(R * 4) + dim)
    for _ in range(6):
        cen = half + np.floor(rng.uniform(-0.5, 0.5, 3) * 4096) / 4096
        cen[dim:] = 0.0
        r, w, slope = _points(dim, shape, cen, R, dR)
        J, left = _cancelled(rng, w)
        p = synth.Params(dim=dim, sigma_pre=0.0, dR=dR, r_max=40.0, r_init=5.0, n_dirs=64 if dim == 2 else 162)
        ctx = snk.Context(0)
        ctx.set_params(p)
        ctx.set_directions(synth.directions_for(dim, p.n_dirs))
        ctx.load_volume(J)
        ctx.load_seeds(cen[None])
        ctx.set_state(cen[None], np.array([R], np.float32), np.array([1], np.int32), np.array([2], np.uint8))
        ctx.prepass()
        assert np.array_equal(ctx.read_volume(J.shape), J)
        ctx.finalize()
        e = ctx.read()["e_vox"].astype(np.float64)[0]
        ctx.close()
        norm = (2.0 * R) ** dim
        on = slope > 0
        per = np.where(on, np.hypot(0.76 * np.asarray(slope * r, float), 1.0), 0.0) * U * np.abs(J)
        mag = float(np.abs(w * J).sum())
        lanes, row = (256, 1) if dim == 3 else (64, 2)
        rows = (2 * half) ** (dim - 1)
        K = -(-rows * row // lanes) * (2 * half)   # terms of a lane, at most
        waves = lanes // 64
        tree = sum(1.0 / (waves * n) for n in (32, 16, 8, 4, 2, 1)) + sum((k / waves) ** 2 for k in range(2, waves + 1))
        sums = U / np.sqrt(3.0) * mag * np.sqrt(K / (3.0 * lanes) + tree)
        t = 4.0 * np.hypot(np.sqrt((per ** 2).sum()), sums) + U * mag + 2.0 ** -24 * abs(float(left))
        got.append((e * norm - float(left)) / t)
        tol.append(t / (U * mag))
    print("error over tolerance", np.round(got, 4), "tolerance over u mag", np.round(tol, 2), flush=True)
    assert np.all(np.abs(got) <= 1.0), got
