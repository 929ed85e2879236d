"""The form of the thickness update is chosen pixel by pixel.  With a relaxation of 1e-30 every update
is far below the thickness's rounding, and the difference form (a_s tau <= 8) then leaves the thickness
as it was, bit for bit, whatever the thickness of the pixels around it; the direct form beyond that
gives it back to a few roundings of the logarithm of a_s tau = 12."""

import numpy as np
import pytest

from synthetic import workload
from tests.helpers import api_objects, oracle_lines, requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("n_lines", [1, 2, 3, 8])
@pytest.mark.parametrize("shape", [(30, 256), (12, 1024), (9, 1080), (8, 2560)])
@pytest.mark.parametrize("kind", ["single", "batched", "xspec"])
def test_thin_pixels_next_to_thick_ones(kind, shape, n_lines):
    import torch
    from paper_2601_22793_amd import Context, SpectrumProfile
    w = workload("local-mono-256", shape=shape)
    w.energies_kev = 60.0 + 15.0 * np.arange(n_lines)
    w.weights = np.full(n_lines, 1.0 / n_lines)
    L = oracle_lines(w)
    geom, spec, mat = api_objects(w)
    a_tau = 0.5 + 0.4 * np.random.default_rng(7).random(shape)
    thick = np.zeros(shape, dtype=bool)
    thick[::3, 5::29] = True   # some in every wave
    a_tau[thick] = 12.0
    tau0 = to_dev(a_tau / L.mu.max())
    d = to_dev(np.full(shape, 0.5))
    c = Context.get(0)
    tau = tau0.clone()
    print(f"update form {kind} {shape} lines={n_lines}", flush=True)
    if kind == "single":
        c.solve(d, geom, spec, mat, "local_l1", 1, 1e-30, thickness=tau)
    elif kind == "batched":
        c.solve_batched([(d, tau, geom, spec, mat)], "local_l1", 1, 1e-30)
    else:
        e, wt = list(map(float, w.energies_kev)), list(map(float, w.weights))
        prof = SpectrumProfile([0.0, shape[1] - 1.0], [e, e], [wt, wt])
        c.solve_xspec(d, geom, spec, prof, mat, "local_l1", 1, 1e-30, thickness=tau)
    torch.cuda.synchronize()
    thin = torch.from_numpy(~thick).cuda()
    assert torch.equal(tau[thin], tau0[thin])
    assert torch.allclose(tau[~thin], tau0[~thin], rtol=2e-6, atol=0.0)
