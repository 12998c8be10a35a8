"""Jobs released after a run or step that ended early, with their uploads still collected on the host: the call frees
them, and what they leave, memory and table rows, serves the next jobs, whose results are those of an engine alone.
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


def _job(k, rng):
    """Jobs of k rays differ in their launch class; 64 classes are the most that one run takes."""
    p = synth.Params(dim=3, sigma_pre=1.0, dR=0.8, r_max=8.0, r_init=4.0, n_rays=2 * k + 2, n_dirs=162, seed=k)
    raw = rng.integers(0, 255, (20, 24, 28)).astype(np.uint8)
    return p, synth.directions_for(3, 162), raw, rng.uniform(0.0, 19.0, (5 + k % 7, 3))


def _engine(snk):
    eng = snk.Engine(0, None, 1 << 30)
    eng.set_launch(64, 1, 0, 0)
    return eng


def _run(eng, served):
    if served:
        for _ in range(3):
            eng.step(10)
    else:
        eng.run()


@pytest.mark.parametrize("served", [False, True])
@pytest.mark.parametrize("which", ["first", "last", "all"])
def test_release_after_an_early_end(snk, served, which):
    rng = np.random.default_rng(2)
    jobs = [_job(k, rng) for k in range(70)]
    eng = _engine(snk)
    ids = [eng.submit(*j, n_iter=30) for j in jobs]
    with pytest.raises(snk.SnkError, match="classes"):
        _run(eng, served)
    drop = {"first": range(8), "last": range(62, 70), "all": range(70)}[which]
    for k in drop:
        eng.release(ids[k])
        with pytest.raises(snk.SnkError, match="unknown job"):
            eng.read(ids[k])
    kept = [k for k in range(70) if k not in drop]
    late = [_job(k, rng) for k in (3, 30)]   # into what the others left
    late_ids = [eng.submit(*j, n_iter=30) for j in late]
    print(which, "served" if served else "batched", flush=True)
    _run(eng, served)
    ref = _engine(snk)
    todo = [(jobs[k], ids[k]) for k in kept[::9]] + list(zip(late, late_ids))
    ref_ids = [ref.submit(*j, n_iter=30) for j, _ in todo]
    ref.run()
    for (_, i), r in zip(todo, ref_ids):
        got, want = eng.read(i), ref.read(r)
        for key in KEYS:
            assert np.array_equal(got[key], want[key], equal_nan=True), key
    stats = eng.get_stats()
    assert stats["pending"] == 0 and stats["running"] == 0
    for i in [ids[k] for k in kept] + late_ids:
        eng.release(i)
    assert eng.get_stats()["bytes_in_use"] == 0
    eng.close()
    ref.close()
