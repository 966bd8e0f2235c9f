"""Volumes around and past 2^30 voxels (4 GiB).

The gathers use 32-bit offsets from the volume's start, or in a larger volume
from the lowest slice a ray touches, or 64-bit ones for a ray that spans more.
Rays run through a small block of random voxels in the volume's far corner, or
through one column of it from end to end; the oracle renders that block alone
(its origin shifted, its far faces those of the volume).  Both with one
wavefront per ray and with several.
"""
import numpy as np
import pytest

from paper_2508_06768_amd import synth
from tests import helpers as H
from tests.test_gpu_parity import _check_images, check_grad_pose, check_grad_volume

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# nz of an nz x 1024 x 1024 volume, first slice of the block, fan:
#   the last voxel that 32-bit offsets reach from the start; one slice more; a
#   base of its own, rays ending inside and running out of the far face; more
#   than 4 GiB along one ray, up and (from behind the far face) down
CASES = {"end": (1024, 980, (40, 300, 0.9, 0.14, 1.0)), "one_more": (1025, 980, (40, 300, 0.9, 0.14, 1.0)),
         "base": (1200, 1150, (40, 290, 0.9, 0.15, 1.0)), "leaving": (1200, 1150, (40, 700, 0.3, 0.15, 1.0)),
         "whole": (1100, 0, (7, 2000, 0.006, 0.54, 5.0)), "down": (1100, 0, (7, 2000, 0.006, 0.54, 5.0))}


@pytest.mark.parametrize("which", sorted(CASES))
@pytest.mark.parametrize("span", [0, -1])
def test_large_volume(which, span):
    from paper_2508_06768_amd.render import FusedStep, Geometry, get_schedule, render, render_backward, set_schedule
    nz, z0, (n, S, aperture, ds, r0) = CASES[which]
    print("large volume", which, span, flush=True)
    rng = np.random.default_rng(nz + S)
    block = rng.uniform(1.4, 1.8, size=(nz - z0, 48, 48)).astype(np.float32)
    c0 = 1024 - 48
    pose = [c0 + 23.0, c0 + 24.0, z0 + 0.3, 0.02, -0.03, 0.1]
    if which == "whole":
        pose = [c0 + 23.0, c0 + 24.0, -3.0, 0.002, -0.003, 0.1]
    if which == "down":
        pose = [c0 + 23.0, c0 + 24.0, nz + 2.0, np.pi - 0.002, 0.001, 0.0]
    case = synth.Case(which, block, (1.0,) * 3, (float(c0), float(c0), float(z0)), np.array([pose], np.float32),
                      [synth.FanSpec(n, S, aperture, ds, r0, 0)],
                      synth.PhysicsSpec(refl_mode=1, speckle_on=True, blur_on=False, alpha=0.02, seed=3))
    Z = torch.full((nz, 1024, 1024), 1.6, device=DEV)
    Z[z0:, c0:, c0:] = torch.from_numpy(block).to(DEV)
    P = torch.from_numpy(case.poses).to(DEV)
    geom = Geometry(tuple(Z.shape), case.spacing, (0.0,) * 3, case.fans, case.phys)
    ref = H.oracle_render(case)
    w = rng.standard_normal(geom.total).astype(np.float32)
    rV, rp = H.oracle_backward(case, w)
    sV, sp = H.oracle_backward(case, 2.0 * ref / ref.size)
    old = get_schedule()
    try:
        set_schedule(**dict(old, span_samples=span))
        _check_images(render(Z, P, geom).cpu().numpy(), ref, which, case.fans)
        gZ, gp = render_backward(Z, P, geom, torch.from_numpy(w).to(DEV))
    finally:
        set_schedule(**old)
    check_grad_volume(gZ[z0:, c0:, c0:].cpu().numpy(), rV, which)
    check_grad_pose(gp.cpu().numpy(), rp, which)
    step = FusedStep(geom, schedule={"span_samples": span})
    T = torch.zeros(geom.total, device=DEV)
    for image in (True, False):
        gZ.fill_(float("nan"))
        bm = torch.empty(geom.total, device=DEV) if image else None
        step.step(Z, P, T, bmode=bm, grad_Z=gZ, grad_pose=gp)
        torch.cuda.synchronize()
        if image:
            _check_images(bm.cpu().numpy(), ref, which, case.fans)
        check_grad_volume(gZ[z0:, c0:, c0:].cpu().numpy(), sV, f"{which} step {image}")
        check_grad_pose(gp.cpu().numpy(), sp, f"{which} step {image}")
    # nothing outside the block
    gZ[z0:, c0:, c0:] = 0.0
    assert int(torch.count_nonzero(gZ)) == 0
    step.close()
    del Z, gZ
    torch.cuda.empty_cache()
