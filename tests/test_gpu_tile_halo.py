"""Per-tile halos of the splat: steep gradients in a few places and of both signs, displacements
around the distances at which the splat looks further than the segments next to a tile (16 rows,
32 columns), image widths and heights off the segment and band sizes.  Against the FP64 oracle; a
prediction is a sum of bilinear deposits rounded to 2^-22 of the brightest one or better, so 1e-5
as for the other forward comparisons."""

import numpy as np
import pytest

from oracle import epr_oracle as O
from synthetic import workload
from tests.helpers import api_objects, oracle_lines, rel_l2, requires_gpu, to_dev, to_np

pytestmark = [pytest.mark.gpu, requires_gpu]


def _maps(shape, w, shift, sign):
    """Phase with one hill and one edge whose largest displacement is `shift` pixels."""
    ny, nx = shape
    y, x = np.mgrid[:ny, :nx].astype(np.float64)
    s = max(2.0, shift)
    phase = np.exp(-(((y - 0.3 * ny) / s) ** 2 + ((x - 0.6 * nx) / s) ** 2))
    phase += 0.5 / (1.0 + np.exp(-(x - 0.25 * nx) / 2.0)) * (y > 0.5 * ny)
    phase += 1e-3 * np.cos(0.3 * x) * np.cos(0.2 * y)
    L = oracle_lines(w)
    gy, gx = np.gradient(phase)
    biggest = max(np.abs(gx).max(), np.abs(gy).max()) * np.max(L.eps_px * L.phase_scale)
    absorb = 0.5 + 0.3 * np.cos(0.05 * x) * np.sin(0.07 * y)
    return sign * phase * (shift / biggest), absorb


@pytest.mark.parametrize("shape", [(90, 96), (250, 250), (270, 324), (300, 450), (512, 160), (8, 600)])
@pytest.mark.parametrize("shift", [0.4, 6.0, 15.5, 16.5, 31.5, 33.0, 70.0])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_local_halo_covers_every_source(shape, shift, sign):
    from paper_2601_22793_amd import Context
    print(f"halo {shape} shift={shift} sign={sign}", flush=True)
    w = workload("nonlocal-poly8-2048", shape=shape)
    w.energies_kev, w.weights = w.energies_kev[:3], w.weights[:3] / w.weights[:3].sum()
    phase, absorb = _maps(shape, w, shift, sign)
    geom, spec, _ = api_objects(w)
    ref = O.forward(phase, absorb, oracle_lines(w), O.NONLOCAL)
    out = Context.get(0).forward(to_dev(phase), to_dev(absorb), geom, spec, "nonlocal")
    assert rel_l2(to_np(out), ref) <= 1e-5
