"""The scatter of small launches on both sides of the rule that gives sparse
fans four rays to a box and shorter depth segments: 7 and 8 rays (more than
two voxels apart or less), steps around 0.35 and 0.7 voxels of the widest
spacing (depths per lane and segment length), few and far rays inside the
volume and leaving it, and fans of both kinds in one table.  Against the
oracle, at the automatic number of rays per box.
"""
import numpy as np
import pytest

from paper_2508_06768_amd import synth
from tests import helpers as H
from tests.test_gpu_parity import DEV, _gpu, check_grad_pose, check_grad_volume

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (rays, samples, aperture, mm per sample) of each fan of a pose's table
CASES = {"seven": [(7, 90, 0.3, 0.5)], "eight_near": [(8, 90, 0.3, 0.5)], "eight_far": [(8, 90, 1.2, 0.5)],
         "two_far": [(2, 95, 1.9, 0.6)], "one": [(1, 130, 0.0, 0.4)], "step_0.35": [(12, 140, 1.5, 0.35)],
         "step_0.36": [(12, 140, 1.5, 0.36)], "step_0.7": [(12, 70, 1.5, 0.7)], "step_0.71": [(12, 70, 1.5, 0.71)],
         "coarse_far": [(9, 45, 1.6, 1.21)], "leaving": [(11, 100, 2.8, 0.6)],
         "mixed": [(40, 300, 0.3, 0.15), (3, 60, 1.5, 0.9)], "mostly_sparse": [(20, 30, 0.2, 0.2), (9, 120, 1.6, 0.45)]}


@pytest.mark.parametrize("spacing", [(1.0, 1.0, 1.0), (0.6, 1.0, 0.8)])
@pytest.mark.parametrize("which", sorted(CASES))
def test_sparse_fans(which, spacing):
    from paper_2508_06768_amd.render import render_backward
    print("sparse fans", which, spacing, flush=True)
    Z = synth.brain_volume(12, 64, 1.0, semi_range=(4.0, 15.0))
    ext = 63.0 * np.array(spacing)
    poses = np.array([[0.5 * ext[0], 0.48 * ext[1], 1.0 + p, 0.1, -0.1, 0.4 + p] for p in range(len(CASES[which]))],
                     np.float32)
    fans = [synth.FanSpec(n, S, a, ds, 0.0, i) for i, (n, S, a, ds) in enumerate(CASES[which])]
    case = synth.Case(which, Z, spacing, (0.0,) * 3, poses, fans,
                      synth.PhysicsSpec(refl_mode=1, speckle_on=False, blur_on=False, seed=12))
    geom, Zt, P = _gpu(case)
    w = np.random.default_rng(len(which)).standard_normal(geom.total).astype(np.float32)
    gZ, gp = render_backward(Zt, P, geom, torch.from_numpy(w).to(DEV))
    rV, rp = H.oracle_backward(case, w)
    check_grad_volume(gZ.cpu().numpy(), rV, which)
    check_grad_pose(gp.cpu().numpy(), rp, which)
