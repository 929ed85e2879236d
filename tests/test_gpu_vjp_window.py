"""Every pixel of the non-local phase gradient within, at the limit of and beyond the window of the
incoming gradient held in LDS, against the FP64 oracle.  dL/du jumps where a ray crosses from one
cell to the next, so pixels for which a shift of one of the lines lies within its float32 rounding
(4 units in the last place) of a whole number are left out, with the neighbours whose D^T reads them;
the rest are a few products a line: 1e-5 as for the other gradients,
in the norm, and 1e-4 of the largest value pixel by pixel, which one wrong tap exceeds."""

import numpy as np
import pytest

from oracle import epr_oracle as O
from synthetic import workload
from tests.helpers import api_objects, oracle_lines, rel_l2, requires_gpu, to_dev, to_np

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("shift", [0.4, 6.0, 12.5, 19.5, 21.0, 24.0, 70.0])
@pytest.mark.parametrize("shape", [(150, 200), (60, 128)])
@pytest.mark.parametrize("n_lines", [1, 3])
def test_every_unambiguous_pixel(shape, shift, n_lines):
    from paper_2601_22793_amd import Context
    print(f"vjp window {shape} shift={shift} lines={n_lines}", flush=True)
    w = workload("nonlocal-poly8-2048", shape=shape)
    w.energies_kev, w.weights = w.energies_kev[:n_lines], w.weights[:n_lines] / w.weights[:n_lines].sum()
    L = oracle_lines(w)
    y, x = np.mgrid[:shape[0], :shape[1]]
    phase = np.cos(0.06 * x + 0.5) * np.cos(0.05 * y) + 0.2 * np.sin(0.11 * x - 0.07 * y)
    gy, gx = np.gradient(phase)
    scale = L.eps_px * L.phase_scale
    phase *= shift / (max(np.abs(gx).max(), np.abs(gy).max()) * scale.max())
    phase = phase.astype(np.float32)
    absorb = (0.5 + 0.2 * np.cos(0.1 * x)).astype(np.float32)
    grad = np.random.default_rng(5).standard_normal(shape).astype(np.float32)
    geom, spec, _ = api_objects(w)
    rp, ra = O.forward_vjp(phase, absorb, grad, L, O.NONLOCAL)
    gp, ga = Context.get(0).forward_vjp(to_dev(phase), to_dev(absorb), to_dev(grad), geom, spec, "nonlocal")
    gp, ga = to_np(gp), to_np(ga)
    # (difference, product and line constant are off by half a unit each)
    gy, gx = np.gradient(phase.astype(np.float64))
    unsure = np.zeros(shape, dtype=bool)
    for s in range(n_lines):
        for g in (gx, gy):
            u = scale[s] * g
            unsure |= np.abs(u - np.round(u)) <= 4.0 * 2.0 ** -23 * np.maximum(np.abs(u), 1e-3)
    near = unsure.copy()
    near[1:] |= unsure[:-1]
    near[:-1] |= unsure[1:]
    near[:, 1:] |= unsure[:, :-1]
    near[:, :-1] |= unsure[:, 1:]
    assert near.mean() < 0.01
    keep = ~near
    assert rel_l2(ga, ra) <= 1e-5
    assert rel_l2(gp[keep], rp[keep]) <= 1e-5
    assert np.abs(gp - rp)[keep].max() <= 1e-4 * np.abs(rp).max()
