"""Precision of the diffraction-pressure term (second-order closures and their vector-Jacobian
products) at large optical depths and large eps / p^2, where the term is a fifth of the prediction
or more, against the FP64 oracle.

Forward: with Q = lap A / A the term is eps^2/4 lap-like of Q, so a relative error delta of every
A = sqrt(I) reaches the prediction as eps^2/4 times the stencil (D_x D_x + D_y D_y) applied twice.
That stencil is (four neighbours - 4 centre) / 4 two pixels apart; the sum of squares of its square
is 676 / 256, so the error is at most 1.625 eps^2/4 delta ||I||, plus three roundings of the
prediction itself.  delta is one unit in the last place (2^-23) for float32 exponentials, roots and
quotients that are exact to one unit; an exponential whose argument is rounded first is off by
depth x 2^-24 instead, ten units at the depths here.  One line at the reference energy: the
exponent a X is the float32 map itself."""

import numpy as np
import pytest

from oracle import epr_oracle as O
from tests.helpers import requires_gpu, to_dev, to_np

pytestmark = [pytest.mark.gpu, requires_gpu]

ULP = 2.0 ** -23


def case(depth, shape):
    from paper_2601_22793_amd import Geometry, Spectrum
    ny, nx = shape
    y, x = np.mgrid[:ny, :nx]
    noise = np.random.default_rng(3).standard_normal(shape)
    absorb = (depth + 0.25 * np.cos(0.9 * x + 0.3) * np.cos(0.7 * y) + 0.1 * np.sin(1.3 * x - 0.8 * y) +
              0.01 * noise).astype(np.float32)
    pixel, k = 1e-6, 2.0 * np.pi * 60e3 / O.HC_EV_M
    distance = 2.0 * np.sqrt(2.0) * k * pixel ** 2       # eps^2 / 4 = 2
    L = O.line_constants([60.0], [1.0], pixel, distance)
    assert L.absorb_scale[0] == 1.0
    return absorb, L, Geometry(ny, nx, pixel, distance), Spectrum([60.0], [1.0], 60.0, 2.0, 3.0)


def context():
    from paper_2601_22793_amd import Context
    return Context.get(0)


@pytest.mark.parametrize("model", ["local_l2", "nonlocal_l2"])
@pytest.mark.parametrize("depth", [2.0, 30.0, 70.0])
@pytest.mark.parametrize("shape", [(96, 120), (270, 1200)])
def test_forward_pressure_term(model, depth, shape):
    absorb, L, geom, spec = case(depth, shape)
    zero = np.zeros(shape, dtype=np.float32)
    ref = O.forward(zero, absorb, L, model)
    intensity = np.exp(-absorb.astype(np.float64))
    assert np.linalg.norm(ref - intensity) > 0.1 * np.linalg.norm(intensity)
    got = to_np(context().forward(to_dev(zero), to_dev(absorb), geom, spec, model))
    if model == "nonlocal_l2":  # the term alone: the transported part has an error of its own
        got -= to_np(context().forward(to_dev(zero), to_dev(absorb), geom, spec, "nonlocal"))
        got += O.forward(zero, absorb, L, O.NONLOCAL)
    q = 0.25 * L.eps_px[0] ** 2
    bound = ULP * (1.625 * q * np.linalg.norm(intensity) + 3.0 * np.linalg.norm(ref))
    err = np.linalg.norm(got - ref)
    print(f"pressure {model} depth={depth}: error / bound {err / bound:.3f}", flush=True)
    assert err <= bound


@pytest.mark.parametrize("model", ["local_l2", "nonlocal_l2"])
@pytest.mark.parametrize("depth", [2.0, 30.0, 70.0])
def test_vjp_pressure_term(model, depth):
    # dI = -q (D Q . k) + (lap^T t - t Q) / (2 A): the longest product chain (I k, its difference, the
    # quotient by A, the two second differences, the quotient by 2 A, then a I) is eight roundings of
    # one unit at most, each of random sign over the pixels: sqrt(8) units, and as much again for the
    # differences' own cancellation (the stencils above at most double the noise of random gradients)
    shape = (96, 120)
    absorb, L, geom, spec = case(depth, shape)
    zero = np.zeros(shape, dtype=np.float32)
    grad = np.random.default_rng(4).standard_normal(shape).astype(np.float32)
    _, ref = O.forward_vjp(zero, absorb, grad, L, model)
    _, plain = O.forward_vjp(zero, absorb, grad, L, O.NONLOCAL)
    assert np.linalg.norm(ref - plain) > 0.1 * np.linalg.norm(plain)
    _, ga = context().forward_vjp(to_dev(zero), to_dev(absorb), to_dev(grad), geom, spec, model)
    err = np.linalg.norm(to_np(ga) - ref) / np.linalg.norm(ref)
    print(f"vjp pressure {model} depth={depth}: rel L2 {err:.2e}", flush=True)
    assert err <= 2.0 * np.sqrt(8.0) * ULP


@pytest.mark.parametrize("model", ["local_l2", "nonlocal_l2"])
def test_opaque_regions_stay_finite(model):
    # depths at which exp(-a X) underflows: the term of such pixels is negligible, not NaN
    shape = (64, 128)
    absorb, L, geom, spec = case(1.0, shape)
    absorb[:, 64:] += np.linspace(0.0, 160.0, 64, dtype=np.float32)
    zero = np.zeros(shape, dtype=np.float32)
    grad = np.random.default_rng(5).standard_normal(shape).astype(np.float32)
    c = context()
    assert np.isfinite(to_np(c.forward(to_dev(zero), to_dev(absorb), geom, spec, model))).all()
    _, ga = c.forward_vjp(to_dev(zero), to_dev(absorb), to_dev(grad), geom, spec, model)
    assert np.isfinite(to_np(ga)).all()
