"""The engine's pre-pass takes volumes that agree in raw type and radii in one launch: a mix of types, radii, layouts
and odd shapes, in batched and served runs, gives every job the bits of the plain path on its volume alone.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

KEYS = ("radii", "centers", "e_mc", "e_vox", "iters", "status", "keep")


@pytest.fixture(scope="module")
def snk():
    import torch   # before the library: the process then has one HIP runtime
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1804_06304_amd import snk as mod
    return mod


def _jobs():
    rng = np.random.default_rng(3)
    out = []
    for k, (shape, dtype, sigma, hz) in enumerate([
            ((24, 31, 65), np.uint16, 1.0, 2.0), ((2, 16, 64), np.uint16, 1.0, 2.0), ((33, 70, 40), np.uint8, 1.0, 2.0),
            ((24, 31, 65), np.uint16, 1.0, 1.0), ((17, 17, 17), np.float32, 0.0, 2.0), ((50, 12, 129), np.uint16, 1.0, 2.0),
            ((20, 40, 30), np.uint8, 3.2, 1.0), ((21, 40, 30), np.uint8, 3.2, 1.0)]):
        raw = rng.uniform(0.0, 250.0, shape).astype(dtype)
        h = (1.0, 1.0, hz)
        p = synth.Params(dim=3, spacing=h, sigma_pre=sigma, dR=0.8, r_max=8.0, r_init=4.0, n_rays=16, n_dirs=162, seed=k)
        cen = rng.uniform(0.0, 1.0, (9 + k, 3)) * (np.array(shape[::-1]) - 1.0) * h
        out.append((p, synth.directions_for(3, 162), raw, cen))
    return out


def _plain(snk, p, dirs, raw, cen, layout):
    ctx = snk.Context(0)
    ctx.set_params(p)
    ctx.set_launch(64, 1, layout)
    ctx.set_directions(dirs)
    ctx.load_volume(raw)
    ctx.load_seeds(cen)
    ctx.evolve(30)
    ctx.finalize()
    out = ctx.read()
    ctx.close()
    return out


@pytest.mark.parametrize("served", [False, True])
@pytest.mark.parametrize("layout", [0, 2])
def test_mixed_volumes_equal_plain(snk, served, layout):
    jobs = _jobs()
    eng = snk.Engine(0, None, 1 << 30)
    eng.set_launch(64, 1, 0, layout)
    late = 3 if served else 0
    ids = [eng.submit(p, d, raw, cen, n_iter=30) for p, d, raw, cen in jobs[late:]]
    print("served" if served else "batched", "layout", layout, flush=True)
    if served:
        eng.step(10)
        ids = [eng.submit(p, d, raw, cen, n_iter=30) for p, d, raw, cen in jobs[:late]] + ids
        for _ in range(4):
            eng.step(10)
    else:
        eng.run()
        eng.run()
    for (p, d, raw, cen), j in zip(jobs, ids):
        got, ref = eng.read(j), _plain(snk, p, d, raw, cen, layout)
        for k in KEYS:
            assert np.array_equal(got[k], ref[k], equal_nan=True), (raw.shape, k)
    eng.close()


@pytest.mark.parametrize("served", [False, True])
def test_many_jobs_and_many_contours_equal_plain(snk, served):
    """Uploads and results beyond one staging copy: more jobs than the first table holds, and a job whose
    contours (nearly all outside its volume) are copied directly and read back in more than one part."""
    rng = np.random.default_rng(11)
    p = synth.Params(dim=3, sigma_pre=1.0, dR=0.8, r_max=8.0, r_init=4.0, n_rays=16, n_dirs=162)
    dirs = synth.directions_for(3, 162)
    jobs = []
    for k in range(70):
        raw = rng.integers(0, 250, (12, 14, 16)).astype(np.uint8)
        jobs.append((raw, rng.uniform(0.0, 11.0, (1 + k % 5, 3))))
    far = np.full((90001, 3), -50.0)
    far[::3000] = rng.uniform(0.0, 11.0, far[::3000].shape)
    jobs.insert(35, (jobs[0][0], far))
    print("served" if served else "batched", len(jobs), "jobs", flush=True)
    eng = snk.Engine(0, None, 1 << 30)
    eng.set_launch(64, 1, 0)
    ids = [eng.submit(p, dirs, raw, cen, n_iter=30) for raw, cen in jobs]
    if served:
        for _ in range(4):
            eng.step(10)
    else:
        eng.run()
    for (raw, cen), j in list(zip(jobs, ids))[::7]:
        got, ref = eng.read(j), _plain(snk, p, dirs, raw, cen, 0)
        for k in KEYS:
            assert np.array_equal(got[k], ref[k], equal_nan=True), (len(cen), k)
    eng.close()


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("served", [False, True])
def test_dense_competition_equals_plain(snk, dim, served):
    """Selection of a batch: jobs with none, one, a few and more contours than a job's workgroup takes at a time, so
    dense that a candidate has more overlapping rivals than its list holds."""
    rng = np.random.default_rng(17)
    shape = (24, 40, 44) if dim == 3 else (1, 150, 160)
    top = (np.array(shape[::-1]) - 1.0)
    p = synth.Params(dim=dim, sigma_pre=1.0, dR=0.8, r_max=8.0, r_init=5.0, n_rays=16, e0=10.0,
                     n_dirs=64 if dim == 2 else 162)
    dirs = synth.directions_for(dim, p.n_dirs)
    raw = rng.integers(0, 250, shape).astype(np.uint8)
    jobs = []
    for n in (0, 1, 31, 700, 4096, 9001):
        cen = rng.uniform(0.0, 1.0, (n, 3)) * top
        cen[:, dim:] = 0.0
        jobs.append(cen)
    print("served" if served else "batched", dim, flush=True)
    eng = snk.Engine(0, None, 1 << 30)
    eng.set_launch(64, 1, 0)
    ids = [eng.submit(p, dirs, raw, cen, n_iter=6) for cen in jobs]
    if served:
        eng.step(6)
    else:
        eng.run()
    for cen, j in zip(jobs, ids):
        got = eng.read(j)
        if len(cen) == 0:
            assert len(got["keep"]) == 0
            continue
        ctx = snk.Context(0)
        ctx.set_params(p)
        ctx.set_launch(64, 1, 0)
        ctx.set_directions(dirs)
        ctx.load_volume(raw)
        ctx.load_seeds(cen)
        ctx.evolve(6)
        ctx.finalize()
        ref = ctx.read()
        ctx.close()
        assert 0 < ref["keep"].sum() <= len(cen)
        for k in KEYS:
            assert np.array_equal(got[k], ref[k], equal_nan=True), (len(cen), k)
    eng.close()
