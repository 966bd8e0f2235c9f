"""Plans on two streams against the same plan held to one: the same
image bit for bit, the loss and the gradients within the rounding of sums in
another order, step after step into outputs filled with NaN.

* many small fans (more than one fan table, launched directly);
* large plans, from a graph and launched directly: more than 64 fans, and no image asked for (the
  forward that only records states then clears dL/dZ, and the second chain
  waits for it), with blur and without;
* long rays beside others, from a graph and launched directly, with FP32
  atomics and in the deterministic plan.
"""
import numpy as np
import pytest

from paper_2508_06768_amd import synth
from tests import helpers as H

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# fans, rays, samples, image
CASES = {"small_fans": (130, 6, 70, True), "small_fans_no_image": (130, 6, 70, False), "one_more": (65, 3, 300, True),
         "large_many_fans": (66, 100, 500, True), "large_no_image": (3, 540, 2000, False),
         "large_many_fans_no_image": (66, 100, 500, False)}


def _plan(n, rays, samples, effects, seed=61):
    from paper_2508_06768_amd.render import Geometry
    rng = np.random.default_rng(seed)
    Z = torch.from_numpy(rng.uniform(1.4, 1.8, size=(48, 40, 44)).astype(np.float32)).to(DEV)
    poses = np.zeros((n, 6), np.float32)
    poses[:, :3] = np.array([21.0, 19.0, 0.0]) + rng.uniform(-2.0, 2.0, (n, 3)) * [1.0, 1.0, 0.2]
    poses[:, 3:] = rng.uniform(-0.2, 0.2, (n, 3))
    # uneven fans of about rays x samples
    fans = [synth.FanSpec(rays + i % 3, samples - 7 * (i % 4), 1.2, 46.0 / samples, 0.5, i) for i in range(n)]
    ph = synth.PhysicsSpec(refl_mode=0, speckle_on=effects, blur_on=effects, seed=5)
    geom = Geometry(tuple(Z.shape), (1.0, 1.0, 1.0), (0.0, 0.0, 0.0), fans, ph)
    return geom, Z, torch.from_numpy(poses).to(DEV)


def _steps(step, geom, Z, poses, image, n=3):
    target = torch.full((geom.total,), 0.05, device=DEV)
    bm = torch.empty(geom.total, device=DEV) if image else None
    gZ, gp = torch.empty_like(Z), torch.empty((geom.n_poses, 6), device=DEV)
    loss = torch.zeros(1, dtype=torch.float64, device=DEV)
    runs = []
    for _ in range(n):
        for x in (bm, gZ, gp, loss):
            if x is not None:
                x.fill_(float("nan"))
        step.step(Z, poses, target, bmode=bm, loss=loss, grad_Z=gZ, grad_pose=gp)
        runs.append((bm.cpu().numpy() if image else np.zeros(0), loss.item(), gZ.cpu().numpy().astype(np.float64),
                     gp.cpu().numpy().astype(np.float64)))
    return runs


def _agree(runs, ref):
    for r in runs:
        np.testing.assert_array_equal(r[0], ref[0])
        assert r[1] == pytest.approx(ref[1], rel=1e-12)
        assert H.rel_l2(r[2], ref[2]) <= 1e-6
        np.testing.assert_allclose(r[3], ref[3], rtol=1e-6, atol=1e-6 * np.abs(ref[3]).max())


@pytest.mark.parametrize("which", sorted(CASES))
@pytest.mark.parametrize("effects", [False, True])
def test_two_chains_agree(which, effects):
    from paper_2508_06768_amd.render import FusedStep
    n, rays, samples, image = CASES[which]
    print("two chains", which, effects, flush=True)
    geom, Z, poses = _plan(n, rays, samples, effects)
    assert (geom.total >= 3 << 20) == which.startswith("large")
    ref = None
    for options in ({"one_stream": True}, {}, {"graph": False}):
        step = FusedStep(geom, **options)
        runs = _steps(step, geom, Z, poses, image)
        step.close()
        ref = ref or runs[0]
        _agree(runs, ref)


def test_schedule_changes_the_chains():
    """One plan through every form: few long rays on one chain; without spans
    two chains from a graph; with every ray in several wavefronts (whose
    launch then clears dL/dZ) one chain again.  Against a one-stream plan."""
    from paper_2508_06768_amd.render import FusedStep
    print("schedule changes", flush=True)
    geom, Z, poses = _plan(2, 250, 6500, True, seed=63)
    assert geom.total >= 3 << 20
    for image in (True, False):
        one = FusedStep(geom, one_stream=True, schedule={"fwd_chunk": 4})
        ref = _steps(one, geom, Z, poses, image, 1)[0]
        one.close()
        step = FusedStep(geom)
        for span in (0, -1, 1, -1, 0):
            step.set_schedule(fwd_chunk=4, span_samples=span)
            _agree(_steps(step, geom, Z, poses, image, 2), ref)
        step.close()


@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("image", [False, True])
def test_long_rays_beside_others(image, deterministic):
    """20 rays of 5000 samples take eight wavefronts each beside 600 of 300."""
    from paper_2508_06768_amd.render import FusedStep, Geometry
    print("long rays beside others", image, deterministic, flush=True)
    small, Z, poses = _plan(4, 200, 300, True, seed=65)
    fans = [synth.FanSpec(20, 5000, 0.5, 0.009, 0.5, 0)] + list(small.fans[1:])
    geom = Geometry(tuple(Z.shape), (1.0, 1.0, 1.0), (0.0, 0.0, 0.0), fans, small.phys)
    runs = {}
    for name, options in (("one", {"one_stream": True}), ("graph", {}), ("direct", {"graph": False})):
        step = FusedStep(geom, deterministic=deterministic, **options)
        runs[name] = _steps(step, geom, Z, poses, image)
        step.close()
    for r in runs.values():
        _agree(r, runs["one"][0])
        if deterministic:
            for x in r:
                np.testing.assert_array_equal(x[2], runs["one"][0][2])
