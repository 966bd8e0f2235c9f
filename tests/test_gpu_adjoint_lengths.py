"""The adjoint at the ray lengths where its form changes: one wavefront per
256 samples up to 2048 (1, 2, 4, 8 wavefronts a ray), the forward's states in
the rows of dL/dZ beyond, and the fused step with and without a forward
before it.  Against the oracle at the suite's 1e-5 bars.
"""
import numpy as np
import pytest

from paper_2508_06768_amd import synth
from tests import helpers as H
from tests.test_gpu_parity import DEV, _check_images, _gpu, check_grad_pose, check_grad_volume

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def length_case(S, refl=0, atten=0, speckle=True, alpha=0.5, seed=3):
    """Three fans of S, S - 1 and about S / 3 samples (rows at every
    alignment), through and past a 32^3 volume."""
    Z = synth.brain_volume(seed, 32, 1.0, semi_range=(3.0, 8.0))
    poses = np.array([[15.5, 15.0, 0.0, 0.1, -0.05, 0.2], [14.0, 16.5, 0.5, -0.1, 0.06, 0.0],
                      [16.0, 14.5, 1.0, 0.03, 0.2, -0.1]], dtype=np.float32)
    fans = [synth.FanSpec(3, S, 0.9, 38.0 / S, 0.0, 0), synth.FanSpec(5, max(S - 1, 1), 0.7, 30.0 / S, 0.5, 1),
            synth.FanSpec(2, max(S // 3, 1), 0.4, 60.0 / S, 0.0, 2)]
    return synth.Case(f"length{S}", Z, (1.0,) * 3, (0.0,) * 3, poses, fans,
                      synth.PhysicsSpec(refl_mode=refl, atten_mode=atten, speckle_on=speckle, alpha=alpha, seed=seed))


LENGTHS = [1, 2, 3, 5, 255, 256, 257, 258, 511, 513, 1023, 1025, 2047, 2048, 2049, 2050, 2051, 4097]


@pytest.mark.parametrize("S", LENGTHS)
def test_adjoint_lengths(S):
    from paper_2508_06768_amd.render import render_backward
    case = length_case(S, refl=S % 2, atten=S % 3)
    print("adjoint, samples", S, flush=True)
    geom, Z, P = _gpu(case)
    w = np.random.default_rng(S).standard_normal(geom.total).astype(np.float32)
    gZ, gp = render_backward(Z, P, geom, torch.from_numpy(w).to(DEV))
    rV, rp = H.oracle_backward(case, w)
    check_grad_volume(gZ.cpu().numpy(), rV, case.name)
    check_grad_pose(gp.cpu().numpy(), rp, case.name)
    # one output at a time: the same numbers (dL/dZ up to its atomics)
    _, gp_only = render_backward(Z, P, geom, torch.from_numpy(w).to(DEV), want_Z=False)
    gZ_only, _ = render_backward(Z, P, geom, torch.from_numpy(w).to(DEV), want_pose=False)
    torch.testing.assert_close(gp_only, gp, rtol=0, atol=0)
    check_grad_volume(gZ_only.cpu().numpy(), rV, case.name)


@pytest.mark.parametrize("S", [1, 256, 257, 1025, 2048, 2049, 4097])
@pytest.mark.parametrize("image", [False, True])
def test_fused_step_without_blur(S, image):
    """Without blur the adjoint forms the loss itself: from its own states
    (no image wanted), or from the forward's."""
    from paper_2508_06768_amd.render import FusedStep
    case = length_case(S, refl=1, speckle=S % 2 == 0)
    print("fused step, samples", S, "image", image, flush=True)
    geom, Z, P = _gpu(case)
    img = H.oracle_render(case)
    rng = np.random.default_rng(S)
    target = (img + (np.abs(img).mean() + 1e-3) * rng.standard_normal(img.size)).astype(np.float32)
    T = torch.from_numpy(target).to(DEV)
    loss = torch.zeros(1, dtype=torch.float64, device=DEV)
    bm = torch.empty(geom.total, device=DEV) if image else None
    gZ, gp = torch.empty_like(Z), torch.empty((geom.n_poses, 6), device=DEV)
    step = FusedStep(geom)
    for _ in range(2):
        step.step(Z, P, T, bmode=bm, loss=loss, grad_Z=gZ, grad_pose=gp)
    torch.cuda.synchronize()
    step.close()
    n = np.concatenate([np.full(f.n_rays * f.n_samples, f.n_rays * f.n_samples) for f in case.fans])
    d = img - target.astype(np.float64)
    rV, rp = H.oracle_backward(case, 2.0 * d / n)
    assert loss.item() == pytest.approx(float((d * d / n).sum()), rel=1e-5)
    if image:
        _check_images(bm.cpu().numpy(), img, case.name, case.fans)
    check_grad_volume(gZ.cpu().numpy(), rV, case.name)
    check_grad_pose(gp.cpu().numpy(), rp, case.name)


@pytest.mark.parametrize("S", [200, 2100])
def test_adjoint_where_the_echo_underflows(S):
    """Attenuation so strong that the transmitted amplitude underflows in
    FP64 on the way down: finite gradients, the oracle's."""
    from paper_2508_06768_amd.render import render_backward
    case = length_case(S, refl=1, speckle=False, alpha=8000.0 / 38.0)
    print("underflow, samples", S, flush=True)
    geom, Z, P = _gpu(case)
    w = np.random.default_rng(S).standard_normal(geom.total).astype(np.float32)
    gZ, gp = render_backward(Z, P, geom, torch.from_numpy(w).to(DEV))
    assert torch.isfinite(gZ).all() and torch.isfinite(gp).all()
    rV, rp = H.oracle_backward(case, w)
    check_grad_volume(gZ.cpu().numpy(), rV, case.name)
    check_grad_pose(gp.cpu().numpy(), rp, case.name)
