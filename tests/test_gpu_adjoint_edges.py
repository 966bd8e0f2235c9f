"""The adjoint where its arithmetic could leave the finite numbers or lose
them: lanes past a ray's end under a steep speckle law, a negative or an
underflowing determinant.  Against the oracle, through the direct adjoint
(whole rays, and rays with a forward's states) and the fused step without an
image.
"""
import numpy as np
import pytest

from paper_2508_06768_amd import synth
from tests import helpers as H
from tests.test_gpu_parity import DEV, _gpu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _adjoints(case, w):
    """(dL/dZ, dL/dpose) of the direct adjoint of w, and of a fused step
    without an image whose residual is the image itself (target 0)."""
    from paper_2508_06768_amd.render import FusedStep, render_backward
    geom, Z, P = _gpu(case)
    gZ, gp = render_backward(Z, P, geom, torch.from_numpy(w).to(DEV))
    step = FusedStep(geom)
    loss = torch.zeros(1, dtype=torch.float64, device=DEV)
    sZ, sp = torch.empty_like(Z), torch.empty((geom.n_poses, 6), device=DEV)
    step.step(Z, P, torch.zeros(geom.total, device=DEV), loss=loss, grad_Z=sZ, grad_pose=sp)
    torch.cuda.synchronize()
    step.close()
    return [(a.cpu().numpy().astype(np.float64), b.cpu().numpy().astype(np.float64)) for a, b in ((gZ, gp), (sZ, sp))], \
        loss.item()


def _references(case, w):
    img = H.oracle_render(case)
    return (H.oracle_backward(case, w), H.oracle_backward(case, 2.0 * img / img.size)), float(np.mean(img ** 2))


# lengths that leave lanes past the end in tiles of whole rays (1 to 8
# wavefronts) and of rays with recorded states; the power of the depth
# fraction (up to 255 past a ray of two samples) overflows FP32 there
@pytest.mark.parametrize("samples,gamma", [(1, 20.0), (2, 30.0), (10, 40.0), (60, 80.0), (300, 400.0), (2100, 1000.0)])
def test_steep_speckle_past_the_end(samples, gamma):
    print("steep speckle", samples, gamma, flush=True)
    Z = synth.brain_volume(3, 32, 1.0, semi_range=(3.0, 9.0))
    ph = synth.PhysicsSpec(refl_mode=1, speckle_on=True, blur_on=False, gamma=gamma, seed=4)
    case = synth.Case("steep", Z, (1.0,) * 3, (0.0,) * 3, np.array([[15.0, 15.0, 1.0, 0.1, 0.0, 0.0]], np.float32),
                      [synth.FanSpec(5, samples, 0.6, 25.0 / max(samples, 2), 0.5, 0)], ph)
    w = np.random.default_rng(samples).standard_normal(5 * samples).astype(np.float32)
    got, loss = _adjoints(case, w)
    refs, ref_loss = _references(case, w)
    # the depth fraction is two FP32 roundings from k / (S - 1), and its power
    # magnifies them gamma times; the residual holds the gain twice
    tol = max(1e-5, 2.0 * gamma * 2.0 ** -23)
    for (gZ, gp), (rV, rp) in zip(got, refs):
        assert np.isfinite(gZ).all() and np.isfinite(gp).all()
        assert H.rel_l2(gZ, rV) <= tol
        assert np.abs(gp - rp).max() <= tol * np.linalg.norm(rp)
    assert loss == pytest.approx(ref_loss, rel=tol, abs=0.0)


# one tile, several wavefronts a ray, and rays with a forward's states
@pytest.mark.parametrize("samples", [60, 900, 3000])
def test_negative_impedance(samples):
    """Impedances of both signs (an optimiser's unclamped step): behind an
    interface with |R| > 1 the determinant is negative.  (The signed
    convention; |R| has no derivative that both sides agree on there.)"""
    print("negative impedance", samples, flush=True)
    Z = synth.brain_volume(5, 32, 1.0, semi_range=(3.0, 9.0))
    Z[12:14, 15, 15] = -0.2
    case = synth.Case("negative", Z, (1.0,) * 3, (0.0,) * 3, np.array([[15.0, 15.0, 1.0, 0.0, 0.0, 0.0]], np.float32),
                      [synth.FanSpec(3, samples, 0.05, 25.0 / samples, 0.5, 0)],
                      synth.PhysicsSpec(refl_mode=1, speckle_on=False, blur_on=False, seed=4))
    w = np.random.default_rng(samples).standard_normal(3 * samples).astype(np.float32)
    got, loss = _adjoints(case, w)
    refs, ref_loss = _references(case, w)
    for (gZ, gp), (rV, rp) in zip(got, refs):
        assert H.rel_l2(gZ, rV) <= 1e-5
        assert np.abs(gp - rp).max() <= 1e-5 * np.linalg.norm(rp)
    assert loss == pytest.approx(ref_loss, rel=1e-5)


def test_absorbed_ray():
    """A ray whose amplitude underflows on the way: finite gradients, and
    those of the part that is left agree with the oracle."""
    print("absorbed ray", flush=True)
    Z = synth.brain_volume(5, 32, 1.0, semi_range=(3.0, 9.0))
    case = synth.Case("absorbed", Z, (1.0,) * 3, (0.0,) * 3, np.array([[15.0, 15.0, 1.0, 0.0, 0.0, 0.0]], np.float32),
                      [synth.FanSpec(3, 1500, 0.05, 0.02, 0.5, 0)],
                      synth.PhysicsSpec(refl_mode=1, speckle_on=False, blur_on=False, seed=4, alpha=200.0, freq=7.0))
    w = np.random.default_rng(7).standard_normal(3 * 1500).astype(np.float32)
    got, _ = _adjoints(case, w)
    refs, _ = _references(case, w)
    for (gZ, gp), (rV, rp) in zip(got, refs):
        assert np.isfinite(gZ).all() and np.isfinite(gp).all()
        assert H.rel_l2(gZ, rV) <= 1e-5
        assert np.abs(gp - rp).max() <= 1e-5 * np.linalg.norm(rp)
