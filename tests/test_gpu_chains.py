"""One chain of launches or two.

A plan of at least 3 * 2^20 ray-samples runs its fans as two chains of launches
on two streams, replayed from a captured graph; smaller ones launch one chain
directly.  On both sides of the line a plan agrees with the same plan held to
one stream: the same image bit for bit, the loss and the gradients within the
rounding of sums in another order (FP64 loss and pose sums, FP32 atomics into
dL/dZ), step after step, with other buffers and after eager work in between.
"""
import numpy as np
import pytest

from paper_2508_06768_amd import synth
from tests import helpers as H

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("effects", [False, True])
@pytest.mark.parametrize("rays", [524, 525])        # 3 x rays x 2000: below and above 3 * 2^20
def test_chains_agree(rays, effects):
    from paper_2508_06768_amd.render import FusedStep, Geometry
    print("chains", rays, effects, flush=True)
    assert (3 * rays * 2000 >= 3 << 20) == (rays == 525)
    rng = np.random.default_rng(51)
    Z = torch.from_numpy(rng.uniform(1.4, 1.8, size=(48, 40, 44)).astype(np.float32)).to(DEV)
    poses = torch.tensor([[21.0, 19.0, 0.0, 0.0, 0.0, 0.0], [20.0, 20.0, 1.0, 0.1, 0.0, 0.1],
                          [22.0, 18.0, 2.0, 0.0, -0.1, 0.2]], device=DEV)
    fans = [synth.FanSpec(rays, 2000, 1.2, 0.025, 0.5, i) for i in range(3)]
    ph = synth.PhysicsSpec(refl_mode=0, speckle_on=effects, blur_on=effects, seed=5)
    geom = Geometry(tuple(Z.shape), (1.0, 1.0, 1.0), (0.0, 0.0, 0.0), fans, ph)
    target = torch.full((geom.total,), 0.05, device=DEV)
    out = {}
    for one in (True, False):
        step = FusedStep(geom, one_stream=one)
        loss = torch.zeros(1, dtype=torch.float64, device=DEV)
        runs = []
        for _ in range(2):              # a second set of buffers: a second capture
            bm = torch.empty(geom.total, device=DEV)
            gZ, gp = torch.empty_like(Z), torch.empty((3, 6), device=DEV)
            for _ in range(3):
                for x in (bm, gZ, gp, loss):
                    x.fill_(float("nan"))
                step.step(Z, poses, target, bmode=bm, loss=loss, grad_Z=gZ, grad_pose=gp)
                runs.append((bm.cpu().numpy(), loss.item(), gZ.cpu().numpy().astype(np.float64),
                             gp.cpu().numpy().astype(np.float64)))
        step.close()
        out[one] = runs
    ref = out[True][0]
    for r in out[True] + out[False]:
        np.testing.assert_array_equal(r[0], ref[0])
        assert r[1] == pytest.approx(ref[1], rel=1e-12)
        assert H.rel_l2(r[2], ref[2]) <= 1e-6
        np.testing.assert_allclose(r[3], ref[3], rtol=1e-6, atol=1e-6 * np.abs(ref[3]).max())
