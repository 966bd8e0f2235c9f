"""The dL/dZ scatter where its LDS box changes form: rays too far apart for
one box (halves, quarters, single rays), depths too long for a box at steps
below and above 1.2 voxels, sixteen rays to a box, the volume's faces (clamped cells) and the segment and row ends.  Against the
oracle at the suite's 1e-5 bars, at every number of rays per wavefront.
"""
import numpy as np
import pytest

from paper_2508_06768_amd import synth
from tests import helpers as H
from tests.test_gpu_parity import DEV, _gpu, check_grad_pose, check_grad_volume

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# rays, samples, aperture, mm per sample (voxels of 1 mm): dense; 8 rays a
# half, a quarter and an eighth of a box apart; depths of 0.35, 0.7 and 6
# voxels per sample; rays that leave the volume sideways
FANS = {"dense": (19, 301, 0.3, 0.25), "half": (9, 600, 0.9, 0.1), "quarter": (10, 700, 2.0, 0.08),
        "single": (8, 3000, 3.0, 0.02), "two_per_lane": (13, 130, 0.8, 0.5), "one_per_lane": (11, 65, 1.2, 0.9),
        "no_box": (5, 40, 0.5, 6.0), "below_coarse": (21, 50, 1.5, 1.19), "coarse": (37, 49, 1.5, 1.22),
        "coarse_parts": (70, 25, 1.0, 2.6), "sixteen": (128, 41, 1.2, 0.23), "sixteen_part": (139, 33, 1.2, 1.7),
        "leaving": (33, 257, 2.8, 0.3)}


@pytest.mark.parametrize("rays_per_wave", [0, 2, 4, 8])
@pytest.mark.parametrize("which", sorted(FANS))
def test_scatter_boxes(which, rays_per_wave):
    from paper_2508_06768_amd.render import get_schedule, render_backward, set_schedule
    n, S, aperture, ds = FANS[which]
    Z = synth.brain_volume(11, 64, 1.0, semi_range=(4.0, 15.0))
    poses = np.array([[31.0, 30.5, 1.0, 0.3, -0.2, 0.4]], dtype=np.float32)
    case = synth.Case(which, Z, (1.0,) * 3, (0.0,) * 3, poses, [synth.FanSpec(n, S, aperture, ds, 0.0, 0)],
                      synth.PhysicsSpec(refl_mode=1, seed=11))
    print("scatter", which, "rays per wavefront", rays_per_wave, flush=True)
    geom, Zt, P = _gpu(case)
    w = np.random.default_rng(S).standard_normal(geom.total).astype(np.float32)
    old = get_schedule()
    try:
        set_schedule(**dict(old, scatter_rays=rays_per_wave))
        gZ, gp = render_backward(Zt, P, geom, torch.from_numpy(w).to(DEV))
    finally:
        set_schedule(**old)
    rV, rp = H.oracle_backward(case, w)
    check_grad_volume(gZ.cpu().numpy(), rV, which)
    check_grad_pose(gp.cpu().numpy(), rp, which)
