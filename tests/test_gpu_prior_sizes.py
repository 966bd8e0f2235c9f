"""The smoothness prior at rows of every length modulo the four voxels of a
thread and around the 1024 voxels of a block, and the pose gradients of
batches with and without empty fans.  Against the oracle: the prior's gradient
within 8 FP32 ulps of the sum of its six terms' sizes, its energy to 1e-6.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2508_06768_amd import synth
from tests import helpers as H
from tests.test_gpu_parity import _gpu, check_grad_pose

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("shape", [(2, 2, 2), (3, 2, 3), (5, 4, 4), (4, 7, 5), (3, 3, 8), (16, 8, 8), (17, 11, 31),
                                   (9, 13, 64), (33, 32, 36)])
def test_prior_sizes(shape):
    from paper_2508_06768_amd.render import Geometry, smoothness
    rng = np.random.default_rng(sum(shape))
    Z = rng.uniform(1.3, 7.8, shape).astype(np.float32)
    g0 = rng.standard_normal(shape).astype(np.float32)
    h, weight = (0.5, 1.25, 2.0), 0.25
    geom = Geometry(shape, h, (0.0,) * 3, [synth.FanSpec(2, 2, 1.0, 1.0)], synth.PhysicsSpec())
    print("prior", shape, flush=True)
    Zt, g = torch.from_numpy(Z).to(DEV), torch.from_numpy(g0).to(DEV)
    loss = torch.full((1,), 3.0, dtype=torch.float64, device=DEV)
    smoothness(Zt, geom, weight, g, loss)
    smoothness(Zt, geom, 0.0, g)                          # no weight, no loss: nothing added
    E, G = 0.0, np.zeros(shape)
    size = np.abs(g0).astype(np.float64)
    for axis, ha in ((2, h[0]), (1, h[1]), (0, h[2])):
        d = np.diff(Z.astype(np.float64), axis=axis)
        w = weight / ha ** 2
        E += w * (d * d).sum()
        lo, hi = [slice(None)] * 3, [slice(None)] * 3
        lo[axis], hi[axis] = slice(None, -1), slice(1, None)
        for part, sign in ((tuple(lo), -1.0), (tuple(hi), 1.0)):
            G[part] += sign * 2.0 * w * d
            size[part] += 2.0 * w * np.abs(d)
    err = np.abs(g.cpu().numpy() - (g0 + G))
    assert np.all(err <= 8 * 2.0 ** -23 * size)
    assert loss.item() == pytest.approx(3.0 + E, rel=1e-6)


@pytest.mark.parametrize("empty", [None, 0, 1, 2])
def test_pose_gradients_with_empty_fans(empty):
    """A batch whose poses all render gets its gradients from the pose sums;
    one with an empty fan through the accumulators, that pose's zero."""
    from paper_2508_06768_amd.render import FusedStep, render_backward
    Z = synth.brain_volume(7, 32, 1.0, semi_range=(3.0, 8.0))
    poses = np.array([[15.5, 15.0, 0.0, 0.1, -0.05, 0.2], [14.0, 16.5, 0.5, 0.0, 0.0, 0.0],
                      [16.0, 14.5, 1.0, 0.03, 0.2, -0.1]], dtype=np.float32)
    fans = [synth.FanSpec(n if p != empty else 0, S, 0.8, 25.0 / S, 0.0, p)
            for p, (n, S) in enumerate(((5, 300), (260, 70), (1, 500)))]
    case = synth.Case("empty", Z, (1.0,) * 3, (0.0,) * 3, poses, fans, synth.PhysicsSpec(refl_mode=1, blur_on=True, seed=7))
    print("poses, empty fan", empty, flush=True)
    geom, Zt, P = _gpu(case)
    w = np.random.default_rng(1).standard_normal(geom.total).astype(np.float32)
    _, gp = render_backward(Zt, P, geom, torch.from_numpy(w).to(DEV))
    _, rp = H.oracle_backward(case, w)
    check_grad_pose(gp.cpu().numpy(), rp, "direct")
    img = H.oracle_render(case)
    T = torch.from_numpy((img + np.abs(img).max() * w).astype(np.float32)).to(DEV)
    n = np.concatenate([np.full(f.n_rays * f.n_samples, f.n_rays * f.n_samples) for f in fans if f.n_rays])
    _, rp = H.oracle_backward(case, 2.0 * (img - T.cpu().numpy().astype(np.float64)) / n)
    out = torch.full((3, 6), 7.0, device=DEV)
    for pose_only in (False, True):
        step = FusedStep(geom, pose_only=pose_only)
        for _ in range(2):
            step.step(Zt, P, T, grad_Z=None if pose_only else torch.empty_like(Zt), grad_pose=out)
        torch.cuda.synchronize()
        step.close()
        check_grad_pose(out.cpu().numpy(), rp, f"step, pose only {pose_only}")
