"""Row inverse with several lines at once: the x-dependent spectrum and the preconditioner alone, at
the widths where the groups change (512, 1024), the largest number of row blocks, and line counts that
do not fill the last round, against the FP64 oracle (1e-4 as for the other x-dependent solves, 1e-5
as for the other preconditioner tests)."""

import numpy as np
import pytest

from oracle import epr_oracle as O
from synthetic import workload
from tests.helpers import api_objects, oracle_lines, rel_l2, requires_gpu, to_dev, to_np

pytestmark = [pytest.mark.gpu, requires_gpu]

SHAPES = [(8, 8), (45, 512), (30, 540), (18, 1024), (1024, 32), (1080, 30)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("n_lines", [1, 2, 3, 5, 9, 16])
def test_xspec_solve(shape, n_lines):
    from tests.test_gpu_xspec import BREF, DIST, DREF, PIX, api, ctx, profile
    bx, E, W = profile(shape[1], n_lines)
    cl = O.column_line_constants(bx, E, W, shape[1], PIX, DIST, DREF, BREF)
    y, x = np.mgrid[:shape[0], :shape[1]]
    d = (0.6 + 0.2 * np.cos(0.11 * x) * np.cos(0.07 * y)).astype(np.float32)
    ref = O.solve_columns(d, cl, "local_l1", 2, 0.4)
    geom, spec, prof, mat = api(shape, bx, E, W)
    got = to_np(ctx().solve_xspec(to_dev(d), geom, spec, prof, mat, "local_l1", 2, 0.4))
    print(f"x-dependent groups {shape} lines={n_lines}: {rel_l2(got, ref):.2e}", flush=True)
    assert rel_l2(got, ref) <= 1e-4


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("n_lines", [1, 2, 3, 5, 9, 16])
def test_precondition(shape, n_lines):
    from paper_2601_22793_amd import Context
    w = workload("local-mono-256", shape=shape)
    w.energies_kev = 60.0 + 100.0 * (np.arange(n_lines) + 0.5) / n_lines
    w.weights = np.full(n_lines, 1.0 / n_lines)
    geom, spec, mat = api_objects(w)
    r = np.random.default_rng(8).standard_normal((n_lines,) + shape).astype(np.float32)
    ref = O.precondition(r, oracle_lines(w))
    got = to_np(Context.get(0).precondition(to_dev(r), geom, spec, mat))
    print(f"preconditioner groups {shape} lines={n_lines}: {rel_l2(got, ref):.2e}", flush=True)
    assert rel_l2(got, ref) <= 1e-5
