"""Row inverse with several lines at once: line counts that do not fill the last round, images at
the widths where the groups change (512, 1024) and at the largest number of row blocks, thickness
and phase, with and without an x-dependent spectrum, against the FP64 oracle after two iterations
(1e-5 as for the other solves)."""

import numpy as np
import pytest

from oracle import epr_oracle as O
from synthetic import workload
from tests.helpers import api_objects, oracle_lines, rel_l2, requires_gpu, to_dev, to_np

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("shape", [(8, 8), (30, 96), (45, 512), (64, 540), (81, 1024), (1024, 64),
                                   (1080, 54), (48, 1080)])
@pytest.mark.parametrize("n_lines", [1, 2, 3, 5, 8, 9, 16])
def test_solve_line_groups(shape, n_lines):
    import torch
    from paper_2601_22793_amd import Context
    print(f"line groups {shape} lines={n_lines}", flush=True)
    w = workload("local-mono-256", shape=shape)
    w.energies_kev = 60.0 + 100.0 * (np.arange(n_lines) + 0.5) / n_lines
    wt = np.linspace(1.0, 2.0, n_lines)
    w.weights = wt / wt.sum()
    L = oracle_lines(w)
    geom, spec, mat = api_objects(w)
    y, x = np.mgrid[:shape[0], :shape[1]]
    d = (0.6 + 0.2 * np.cos(0.11 * x) * np.cos(0.07 * y)).astype(np.float32)
    ref = O.solve(d, L, O.LOCAL_L1, 2, 0.4)
    phase = torch.empty(shape, device="cuda")
    got = Context.get(0).solve(to_dev(d), geom, spec, mat, "local_l1", 2, 0.4, phase_out=phase)
    assert rel_l2(to_np(got), ref) <= 1e-5
    kref = 2.0 * np.pi * w.energy_ref_kev * 1e3 / 1.239841984e-6
    assert rel_l2(to_np(phase), -kref * w.delta_ref * ref) <= 1e-5


@pytest.mark.parametrize("n_lines", [2, 5, 8])
def test_nonfinite_update_is_flagged_by_every_group(n_lines):
    from paper_2601_22793_amd import Context
    shape = (64, 96)
    w = workload("local-mono-256", shape=shape)
    w.energies_kev = 60.0 + 10.0 * np.arange(n_lines)
    w.weights = np.full(n_lines, 1.0 / n_lines)
    geom, spec, mat = api_objects(w)
    d = np.full(shape, 0.6, dtype=np.float32)
    d[40, 50] = np.nan
    c = Context.get(0)
    c.solve(to_dev(d), geom, spec, mat, "local_l1", 1, 0.4)
    assert c.diagnostics()["nonfinite"] == 1
