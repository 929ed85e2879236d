"""The thickness update over the whole range of a_s tau: one iteration from a ramp that starts at
zero and ends far beyond the thickness at which the update changes its form (a_s tau = 8), and
one from thin and slightly negative values, against the FP64 oracle.  The update is a few float32
operations on a thickness: 1e-5 as for the other solves, plus what a rounding of the filtered
residual (4e-7 of its largest value, a float32 transform) makes of the logarithm where its argument
is small."""

import numpy as np
import pytest

from oracle import epr_oracle as O
from synthetic import workload
from tests.helpers import api_objects, oracle_lines, rel_l2, requires_gpu, to_dev, to_np

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("n_lines", [1, 3])
@pytest.mark.parametrize("top", [-0.5, 1.0, 30.0, 50.0, 120.0])
def test_one_update_from_a_ramp(n_lines, top):
    from paper_2601_22793_amd import Context
    shape = (30, 512)
    w = workload("local-mono-256", shape=shape)
    w.energies_kev = 60.0 + 15.0 * np.arange(n_lines)
    w.weights = np.full(n_lines, 1.0 / n_lines)
    L = oracle_lines(w)
    geom, spec, mat = api_objects(w)
    tau0 = np.broadcast_to(np.linspace(0.0, top, shape[1]) / L.mu.max(), shape)
    tau0 = np.ascontiguousarray(tau0, dtype=np.float32)
    d = 0.5 + 0.3 * np.random.default_rng(2).random(shape)
    print(f"update lines={n_lines} top={top}", flush=True)
    ref = O.solve(d.astype(np.float32), L, O.LOCAL_L1, 1, 0.4, tau0=tau0)
    # the arguments r_s of the logarithms, and the thickness error that their rounding makes
    I = L.w[:, None, None] * np.exp(-L.mu[:, None, None] * tau0)
    P = O.forward_lines(I, -(L.k * L.delta)[:, None, None] * tau0, L, O.LOCAL_L1)
    total = np.maximum(P, 0.0).sum(axis=0)
    share = np.where(total > 1e-30, np.maximum(P, 0.0) / np.maximum(total, 1e-30), L.w[:, None, None])
    e = share * (d.astype(np.float32) - P.sum(axis=0))
    z = np.stack([0.4 / L.w[s] * O.paganin_filter(e[s], L.alpha_px[s]) for s in range(n_lines)])
    r = np.maximum(I / L.w[:, None, None] + z, 1e-6)
    dl = np.minimum(4e-7 * np.abs(z).max() / r, 14.0)
    wm = (L.w * L.mu)[:, None, None]
    bound = np.linalg.norm((wm * dl).sum(axis=0) / (L.w * L.mu ** 2).sum()) / np.linalg.norm(ref)
    got = Context.get(0).solve(to_dev(d), geom, spec, mat, "local_l1", 1, 0.4, thickness=to_dev(tau0))
    assert rel_l2(to_np(got), ref) <= 1e-5 + bound
