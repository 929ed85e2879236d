"""Single images run the launch choices that were tuned or cached, whatever their size."""

import json

import numpy as np
import pytest

from oracle import epr_oracle as O
from synthetic import workload
from tests.helpers import api_objects, oracle_lines, rel_l2, requires_gpu, to_dev, to_np

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("shape", [(90, 96), (256, 320), (512, 600)])
def test_cached_tile_is_the_one_a_small_image_runs(tmp_path, shape):
    # The splat's fixed-point unit follows from its tile, so other tiles round other bits: with one
    # line (where a single solve and a batch of one share every other kernel) the single solve gives
    # the bits of the batch, which takes the cached tile.
    import torch
    from paper_2601_22793_amd import Context
    w = workload("nonlocal-mono-2048", shape=shape, n_iter=4)
    obj = w.true_object()
    d = w.add_noise(O.forward(obj["phase"], obj["absorb"], oracle_lines(w), O.NONLOCAL))
    geom, spec, mat = api_objects(w)
    entry = (to_dev(d), torch.zeros(shape, dtype=torch.float32, device="cuda"), geom, spec, mat)
    for tile in ((64, 32), (32, 16)):
        c = Context(0)
        try:
            path = str(tmp_path / f"tile{tile[0]}.json")
            with open(path, "w") as fh:
                json.dump({"splat_tx": tile[0], "splat_ty": tile[1]}, fh)
            c.autotune([entry], "nonlocal", cache_json=path)
            entry[1].zero_()
            c.solve_batched([entry], "nonlocal", 4, 0.4)
            single = c.solve(entry[0], geom, spec, mat, "nonlocal", 4, 0.4)
            torch.cuda.synchronize()
            print(f"tile {tile} on {shape}: {int((single != entry[1]).sum())} pixels differ", flush=True)
            assert torch.equal(single, entry[1])
        finally:
            c.close()


@pytest.mark.parametrize("tile,n_lines", [((60, 64), 10), ((32, 84), 14), ((10, 211), 16)])
def test_largest_accepted_tiles_match_oracle(tmp_path, tile, n_lines):
    # tiles whose accumulators leave 64 to 320 bytes of a CU's 160 KB (tolerance of the solves)
    import torch
    from paper_2601_22793_amd import Context
    shape = (120, 250)
    w = workload("nonlocal-poly8-2048", shape=shape, n_iter=3)
    w.energies_kev = 60.0 + 100.0 * (np.arange(n_lines) + 0.5) / n_lines
    w.weights = np.full(n_lines, 1.0 / n_lines)
    obj = w.true_object()
    L = oracle_lines(w)
    d = w.add_noise(O.forward(obj["phase"], obj["absorb"], L, O.NONLOCAL))
    ref = O.solve(d, L, O.NONLOCAL, 3, 0.4)
    geom, spec, mat = api_objects(w)
    entry = (to_dev(d), torch.zeros(shape, dtype=torch.float32, device="cuda"), geom, spec, mat)
    c = Context(0)
    try:
        path = str(tmp_path / "tile.json")
        with open(path, "w") as fh:
            json.dump({"splat_tx": tile[0], "splat_ty": tile[1]}, fh)
        got = c.autotune([entry], "nonlocal", cache_json=path)
        assert (got["splat_tx"], got["splat_ty"]) == tile
        print(f"tile {tile} x {n_lines} lines", flush=True)
        assert rel_l2(to_np(c.solve(entry[0], geom, spec, mat, "nonlocal", 3, 0.4)), ref) <= 1e-4
        c.solve_batched([entry], "nonlocal", 3, 0.4)
        assert rel_l2(to_np(entry[1]), ref) <= 1e-4
    finally:
        c.close()


@pytest.mark.parametrize("lines", [0, 1, 2, 4])
@pytest.mark.parametrize("shape,n_lines", [((96, 128), 8), ((64, 250), 3), ((2048, 64), 8),
                                           ((60, 2560), 5)])
def test_xspec_solve_with_row_lines_matches_oracle(tmp_path, lines, shape, n_lines):
    # lines per row-pass workgroup as cached (0: untuned, which keeps the default two at 2048 rows),
    # a last group that is short, and rows of the 1024-thread class; the other x-dependent solves' tolerance
    import torch
    from paper_2601_22793_amd import Context
    from tests.test_gpu_xspec import BREF, DIST, DREF, PIX, api, profile, thickness
    bx, E, W = profile(shape[1], n_lines)
    cl = O.column_line_constants(bx, E, W, shape[1], PIX, DIST, DREF, BREF)
    d = O.forward_columns(thickness(shape, 7, 3.0, cl), cl, "nonlocal").astype(np.float32)
    ref = O.solve_columns(d, cl, "nonlocal", 3, 0.4)
    geom, spec, prof, mat = api(shape, bx, E, W)
    c = Context(0)
    try:
        if lines:
            path = str(tmp_path / "lines.json")
            with open(path, "w") as fh:
                json.dump({"row_lines": lines}, fh)
            entry = (to_dev(d), torch.zeros(shape, dtype=torch.float32, device="cuda"), geom, spec, mat)
            c.autotune([entry], "nonlocal", cache_json=path)
        got = to_np(c.solve_xspec(to_dev(d), geom, spec, prof, mat, "nonlocal", 3, 0.4))
    finally:
        c.close()
    print(f"xspec {shape} x {n_lines}, {lines} lines a workgroup: {rel_l2(got, ref):.2e}", flush=True)
    assert rel_l2(got, ref) <= 1e-4
