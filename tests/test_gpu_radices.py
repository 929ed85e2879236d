"""Transform lengths whose radix sequences are chosen at run time, against the FP64 oracle: every
radix (2 ... 6, 8, 9, 10, 12, 15, 16) as a first, middle and last stage, both thread classes, and the lengths
at which radices 12 and 15 stop fitting one butterfly per thread.  A float32 transform of n points
is good to about 1e-7 log2(n); 1e-5 as for the other preconditioner comparisons."""

import numpy as np
import pytest

from oracle import epr_oracle as O
from synthetic import workload
from tests.helpers import api_objects, oracle_lines, rel_l2, requires_gpu, to_dev, to_np

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("shape", [(8, 8), (9, 10), (10, 12), (12, 18), (15, 20), (16, 30), (45, 60),
                                   (243, 486), (625, 250), (750, 90), (1080, 1200), (1215, 1500),
                                   (1250, 100), (1536, 72), (1620, 36), (1920, 48), (1944, 40),
                                   (2025, 54), (64, 1620), (72, 1944), (81, 2000), (2187, 36),
                                   (3000, 32), (3072, 48), (3125, 16), (3750, 64), (3840, 40),
                                   (4050, 24), (36, 4050), (40, 3888), (60, 3750)])
def test_precondition_run_time_lengths(shape):
    from paper_2601_22793_amd import Context
    print(f"precondition {shape}", flush=True)
    w = workload("nonlocal-poly8-2048", shape=shape)
    w.energies_kev, w.weights = w.energies_kev[:2], w.weights[:2] / w.weights[:2].sum()
    geom, spec, mat = api_objects(w)
    x = np.random.default_rng(3).standard_normal((2,) + shape).astype(np.float32) + 3.0
    ref = O.precondition(x, oracle_lines(w))
    out = Context.get(0).precondition(to_dev(x), geom, spec, mat)
    assert rel_l2(to_np(out), ref) <= 1e-5
