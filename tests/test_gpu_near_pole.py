"""The adjoint one step from a pole of the echo, against exact rational
arithmetic.

One-ray fans run along columns of the volume from voxel centre to voxel
centre, so their samples are the voxels themselves.  Three interfaces in the
|R| convention bring the recurrence to v1' / v1 = p, about 1e-9 (|R| a
rational function of FP32 voxels: p is exact here).  There a relative error
of the state before the interface is magnified 1 / p times in the pixel, and
twice that in its derivative.  The interfaces sit inside a chunk of four, or
across two (where the adjoint starts from a state at every fourth sample).
"""
from fractions import Fraction

import numpy as np
import pytest

from paper_2508_06768_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SAMPLES = 12


class Dual:
    """A rational number and its derivatives by the samples."""

    def __init__(self, v, d=None):
        self.v, self.d = Fraction(v), d or {}

    def _lin(self, v, a, o, b):
        d = {k: a * x for k, x in self.d.items()}
        for k, x in o.d.items():
            d[k] = d.get(k, 0) + b * x
        return Dual(v, d)

    def __add__(self, o):
        return self._lin(self.v + o.v, 1, o, 1)

    def __sub__(self, o):
        return self._lin(self.v - o.v, 1, o, -1)

    def __mul__(self, o):
        return self._lin(self.v * o.v, o.v, o, self.v)

    def __truediv__(self, o):
        return self._lin(self.v / o.v, 1 / o.v, o, -self.v / o.v ** 2)


def pixels(z):
    """Pixels of a ray of samples z without attenuation, and the ratios
    v1' / v1 of consecutive steps."""
    z = [Dual(x, {i: Fraction(1)}) for i, x in enumerate(z)]
    one, two = Dual(1), Dual(2)
    v0, v1, det = Dual(0), Dual(1), Dual(1)
    e, piv = [Dual(0)], [Fraction(1)]
    for a, b in zip(z, z[1:]):
        # (|R| has derivative 0 at R = 0)
        r = Dual(0) if a.v == b.v else ((b - a) if b.v > a.v else (a - b)) / (a + b)
        n1 = v0 * r + v1
        e.append(r * det / (v1 * n1))
        piv.append(n1.v / v1.v)
        v0, v1, det = v0 * (one - two * r * r) - v1 * r, n1, det * (one - r * r)
    return e, piv


def near_pole_ray(rng, first):
    """FP32 samples whose interfaces first, first + 1, first + 2 end p from a
    pole, 5e-10 <= |p| <= 2e-9, and that pixel's index."""
    for _ in range(4000):
        z = np.full(SAMPLES, np.float32(rng.uniform(1.0, 2.0)), np.float32)
        z[first:] = z[0] * np.float32(rng.uniform(6.0, 12.0))
        z[first + 1:] = z[first] / np.float32(rng.uniform(6.0, 12.0))
        a, b, c = (float(x) for x in (z[0], z[first], z[first + 1]))
        r1, r2 = (b - a) / (b + a), (b - c) / (b + c)
        v0, v1 = -r1 * (1 - 2 * r2 * r2) - r2, 1 - r1 * r2
        r3 = -v1 / v0
        if not 0.05 < r3 < 0.95:
            continue
        z[first + 2:] = np.float32(c * (1 + r3) / (1 - r3))
        z[first + 3:] = z[first + 2] * np.float32(rng.uniform(0.8, 0.9))     # behind it: one more interface
        d = float(z[first + 2])
        if 4e-10 <= abs(v0 * (d - c) / (d + c) + v1) / v1 <= 2.2e-9:
            _, piv = pixels([Fraction(float(x)) for x in z])
            if Fraction(5, 10 ** 10) <= abs(piv[first + 2]) <= Fraction(2, 10 ** 9):
                return z, first + 2, float(abs(piv[first + 2]))
    raise AssertionError("no ray found")


def test_near_pole():
    from paper_2508_06768_amd.render import FusedStep, Geometry, render_backward
    print("near pole", flush=True)
    rng = np.random.default_rng(101)
    rays = [near_pole_ray(rng, first) for first in (1, 2, 3, 5) for _ in range(48)]
    n = len(rays)
    Z = np.ones((SAMPLES + 2, 3, 2 * n + 2), np.float32)
    for i, (z, _, _) in enumerate(rays):
        Z[1:SAMPLES + 1, 1, 2 * i + 1] = z
    poses = torch.tensor([[2.0 * i + 1.0, 1.0, 1.0, 0.0, 0.0, 0.0] for i in range(n)], device=DEV)
    fans = [synth.FanSpec(1, SAMPLES, 0.0, 1.0, 0.0, i) for i in range(n)]
    ph = synth.PhysicsSpec(refl_mode=0, atten_mode=2, speckle_on=False, blur_on=False, seed=1)
    geom = Geometry(Z.shape, (1.0,) * 3, (0.0,) * 3, fans, ph)
    Zt = torch.from_numpy(Z).to(DEV)
    w = torch.zeros((n, SAMPLES), device=DEV)
    for i, (_, at, _) in enumerate(rays):
        w[i, at] = 1.0
    gZ, _ = render_backward(Zt, poses, geom, w.reshape(-1), want_pose=False)
    out = {"direct": gZ}
    for name, image in (("step", True), ("step without image", False)):
        step = FusedStep(geom)
        sZ = torch.empty_like(Zt)
        step.step(Zt, poses, torch.zeros(geom.total, device=DEV),
                  bmode=torch.empty(geom.total, device=DEV) if image else None, grad_Z=sZ)
        torch.cuda.synchronize()
        step.close()
        out[name] = sZ
    err = {name: [] for name in out}
    for i, (z, at, p) in enumerate(rays):
        e, _ = pixels([Fraction(float(x)) for x in z])
        one = np.array([float(e[at].d.get(k, 0)) for k in range(SAMPLES)])
        loss = np.array([float(sum((2 * x.v * x.d.get(k, 0) for x in e), Fraction(0)) / SAMPLES) for k in range(SAMPLES)])
        for name, g in out.items():
            ref = one if name == "direct" else loss
            g = g[1:SAMPLES + 1, 1, 2 * i + 1].cpu().numpy().astype(np.float64)
            d = np.abs(g - ref).max() / np.abs(ref).max()
            # past the FP32 output's own rounding, in units of 2^-53 / p
            err[name].append(max(d - 2.0 ** -24, 0.0) * p * 2.0 ** 53)
    for name, x in err.items():
        # p holds seven FP64 roundings (one in each of three reflections, two
        # in each component of the state before), each even over +-1: a root mean square
        # of sqrt(7 / 3); the pixel's derivative holds p twice, its square's thrice
        bar = (2 if name == "direct" else 3) * (7.0 / 3.0) ** 0.5
        rms = float(np.sqrt(np.mean(np.square(x))))
        print(name, f"rms {rms:.2f} bar {bar:.2f} worst {max(x):.2f}", flush=True)
        assert rms <= bar, name
