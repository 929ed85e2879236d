"""Vector-Jacobian products at the edges of their tiles and strips (62 x 30 and 56 x 8 pixels)
against the FP64 oracle: the smallest image, one tile or strip exactly filled, one pixel more,
line counts below, at and above the waves that share a strip, and displacements that leave the
image.  Each gradient is a sum of a few float32 products per line: 1e-5 as for the other gradients."""

import numpy as np
import pytest

from oracle import epr_oracle as O
from synthetic import workload
from tests.helpers import api_objects, oracle_lines, rel_l2, requires_gpu, to_dev, to_np

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("model", ["nonlocal", "nonlocal_l2", "local_l1", "local_l2"])
@pytest.mark.parametrize("shape", [(8, 8), (9, 54), (16, 60), (30, 64), (32, 120), (75, 128), (90, 250)])
@pytest.mark.parametrize("n_lines", [1, 3, 4, 6])
def test_vjp_edges_match_oracle(model, shape, n_lines):
    from paper_2601_22793_amd import Context
    print(f"vjp {model} {shape} lines={n_lines}", flush=True)
    w = workload("nonlocal-poly8-2048" if model == "nonlocal" else "local-mono-256", shape=shape)
    w.energies_kev = 60.0 + 100.0 * (np.arange(n_lines) + 0.5) / n_lines
    wt = np.linspace(1.0, 2.0, n_lines)
    w.weights = wt / wt.sum()
    rng = np.random.default_rng(11 + n_lines)
    y, x = np.mgrid[:shape[0], :shape[1]]
    wave = sum(np.cos(0.3 * k * y + rng.uniform(0, 6)) * np.cos(0.2 * k * x + rng.uniform(0, 6))
               for k in (1, 2, 3))
    absorb = 0.4 + 0.1 * np.roll(wave, 1, axis=0)
    if model == "nonlocal":
        wave = wave * 20.0
    # whole shapes of the float32 inputs enter the oracle: the map's cells are the same there
    phase, absorb = wave.astype(np.float32), absorb.astype(np.float32)
    grad = rng.standard_normal(shape).astype(np.float32)
    geom, spec, _ = api_objects(w)
    rp, ra = O.forward_vjp(phase, absorb, grad, oracle_lines(w), model)
    gp, ga = Context.get(0).forward_vjp(to_dev(phase), to_dev(absorb), to_dev(grad), geom, spec, model)
    assert rel_l2(to_np(ga), ra) <= 1e-5
    assert rel_l2(to_np(gp), rp) <= 1e-5


@pytest.mark.parametrize("shift", [0.4, 6.0, 19.5, 24.0, 70.0])
def test_vjp_window_sizes_match_oracle(shift):
    # displacements within, at the limit of and beyond the window of the gradient held in LDS
    # (phase smooth on the scale of the shift; tolerance as above)
    from paper_2601_22793_amd import Context
    shape = (150, 200)
    print(f"vjp window shift={shift}", flush=True)
    w = workload("nonlocal-poly8-2048", shape=shape)
    w.energies_kev, w.weights = w.energies_kev[:3], w.weights[:3] / w.weights[:3].sum()
    L = oracle_lines(w)
    y, x = np.mgrid[:shape[0], :shape[1]]
    phase = np.cos(0.06 * x + 0.5) * np.cos(0.05 * y) + 0.2 * np.sin(0.11 * x - 0.07 * y)
    gy, gx = np.gradient(phase)
    phase *= shift / (max(np.abs(gx).max(), np.abs(gy).max()) * np.max(L.eps_px * L.phase_scale))
    phase = phase.astype(np.float32)
    absorb = (0.5 + 0.2 * np.cos(0.1 * x)).astype(np.float32)
    grad = np.random.default_rng(5).standard_normal(shape).astype(np.float32)
    geom, spec, _ = api_objects(w)
    rp, ra = O.forward_vjp(phase, absorb, grad, L, O.NONLOCAL)
    gp, ga = Context.get(0).forward_vjp(to_dev(phase), to_dev(absorb), to_dev(grad), geom, spec, "nonlocal")
    assert rel_l2(to_np(ga), ra) <= 1e-5
    # dL/du is constant inside a cell and jumps between cells: a float32 shift that rounds across
    # a cell edge (one in 1e5 of the pixels and lines) takes the neighbouring cell's value
    assert rel_l2(to_np(gp), rp) <= 1e-2
