"""Several wavefronts per ray where a launch has few rays.

At the default span length the forward and the fused step's adjoint give
each ray 2, 4 or 8 wavefronts when the rays are too few to fill the chip.
With ``span_samples = -1`` every ray has one.  The state and the adjoint
carried across tiles take the same operations either way, so images, loss and
the deterministic dL/dZ are the same bit for bit, and the pose gradients
differ only in the order of their FP64 sums; so with rays of 4096 samples and
more, which take eight up to 512 of them.  Lengths are the edges of one,
two, four and eight tiles of 256 samples and of 512; ray counts the ends of
the range.
"""
import numpy as np
import pytest

from paper_2508_06768_amd import synth
from tests import helpers as H
from tests.test_gpu_parity import _check_plan, _plan_reference
from tests.test_gpu_spans import _det_step, long_column_case

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def few_case(rays, samples, refl=0) -> synth.Case:
    """Fans of ``rays`` x ``samples``, 3 x 258 and 2 x 5 through one column of
    independent voxels, with speckle and blur."""
    case = long_column_case(refl, True, seed=samples)
    fans = [synth.FanSpec(rays, samples, 0.003, 1900.0 / samples, 0.5, 0),
            synth.FanSpec(3, min(258, samples), 0.02, 1.5, 0.2, 1), synth.FanSpec(2, 5, 0.03, 1.0, 0.0, 2)]
    return synth.Case("few_rays", case.Z, case.spacing, case.origin, case.poses, fans, case.phys)


@pytest.mark.parametrize("rays,samples", [(1, 256), (1, 257), (2, 511), (1, 513), (2, 1024), (1, 1025), (1, 2047),
                                          (2, 2049), (1, 4096), (1019, 300), (1020, 300), (507, 1000), (508, 1000),
                                          (507, 1100), (508, 1100), (512, 4100), (513, 4100)])
def test_few_rays_bit_identical(rays, samples):
    case = few_case(rays, samples, refl=rays % 2)
    print("few rays", rays, samples, flush=True)
    target = np.full(sum(f.n_rays * f.n_samples for f in case.fans), 0.05)
    a = _det_step(case, target, 0, fc=0)
    b = _det_step(case, target, -1, fc=0)
    np.testing.assert_array_equal(a[0], b[0])
    assert a[1] == b[1]
    np.testing.assert_array_equal(a[2], b[2])
    np.testing.assert_allclose(a[3], b[3], rtol=1e-10, atol=1e-12 * np.abs(b[3]).max())


@pytest.mark.parametrize("rays,samples", [(5, 260), (4, 770), (3, 1030)])
def test_few_rays_match_oracle(rays, samples):
    case = few_case(rays, samples)
    target = H.oracle_render(case, poses=case.poses + np.float32([[0.1, -0.1, 0.2, 0.0, 0.01, 0.0]]))
    _check_plan(case, _det_step(case, target, 0, fc=0), _plan_reference(case, target), f"few rays {rays} x {samples}")
