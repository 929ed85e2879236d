"""Splat instances by line count and tile: every line count from 1 to 16 (with an instance of its
own or in the next larger one) on images of the small and of the default tile, forward model and
one solve iteration, against the FP64 oracle at 1e-5 as for the other comparisons."""

import numpy as np
import pytest

from oracle import epr_oracle as O
from synthetic import workload
from tests.helpers import api_objects, oracle_lines, rel_l2, requires_gpu, to_dev, to_np

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("shape", [(48, 90), (512, 1024)])
@pytest.mark.parametrize("n_lines", range(1, 17))
def test_splat_every_line_count(shape, n_lines):
    from paper_2601_22793_amd import Context
    print(f"splat {shape} lines={n_lines}", flush=True)
    w = workload("nonlocal-poly8-2048", shape=shape)
    w.energies_kev = 60.0 + 100.0 * (np.arange(n_lines) + 0.5) / n_lines
    wt = np.linspace(1.0, 2.0, n_lines)
    w.weights = wt / wt.sum()
    L = oracle_lines(w)
    geom, spec, mat = api_objects(w)
    y, x = np.mgrid[:shape[0], :shape[1]]
    wave = np.cos(0.21 * x) * np.cos(0.17 * y) + 0.5 * np.cos(0.05 * x + 0.3 * y)
    c = Context.get(0)
    ref = O.forward(40.0 * wave, 0.5 + 0.2 * wave, L, O.NONLOCAL)
    out = c.forward(to_dev(40.0 * wave), to_dev(0.5 + 0.2 * wave), geom, spec, "nonlocal")
    assert rel_l2(to_np(out), ref) <= 1e-5
    tau0 = (1e-3 + 2e-4 * wave).astype(np.float32)
    sol = O.solve(ref.astype(np.float32), L, O.NONLOCAL, 1, 0.4, tau0=tau0)
    got = c.solve(to_dev(ref), geom, spec, mat, "nonlocal", 1, 0.4, thickness=to_dev(tau0))
    assert rel_l2(to_np(got), sol) <= 1e-5
