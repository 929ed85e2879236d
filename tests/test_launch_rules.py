"""Launch rules of the host code without a device: a tuned splat tile and a tuned number of lines per
row-pass workgroup hold for single images of every size, and only untuned ones go by the size.
The rules are inline functions of csrc/host.h, compiled into a small host program here."""

import os
import subprocess

import pytest

from paper_2601_22793_amd import build as B

PROGRAM = r"""
#include "host.h"
// args: tile_tuned tx ty lines_tuned lines ny nx n_lines single
int main(int, char** v) {
  epr_ctx h;
  int a[9];
  for (int i = 0; i < 9; ++i) a[i] = std::atoi(v[i + 1]);
  h.tile_tuned = a[0];
  h.splat_tx = a[1];
  h.splat_ty = a[2];
  h.lines_tuned = a[3];
  h.row_lines = a[4];
  epr::ProbDesc p;
  std::memset(&p, 0, sizeof p);
  p.ny = a[5];
  p.nx = a[6];
  p.lp.n = a[7];
  int tx = 0, ty = 0;
  epr::host::choose_tile(h, p.ny, p.nx, &tx, &ty);
  epr::host::apply_row_lines(&h, &p, a[8] != 0);
  std::printf("%d %d %d\n", tx, ty, p.rlpb);
  return 0;
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = str(d / "rules.cpp"), str(d / "rules")
    with open(src, "w") as fh:
        fh.write(PROGRAM)
    r = subprocess.run([B.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-I", B.CSRC, "-I",
                        os.path.join(B.ROOT, "include"), src, "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]

    def run(tuned_tile, tile, tuned_lines, lines, shape, n_lines, single=1):
        out = subprocess.run([exe] + [str(int(v)) for v in (tuned_tile, *tile, tuned_lines, lines,
                                                            *shape, n_lines, single)],
                             capture_output=True, text=True, check=True).stdout
        tx, ty, rl = map(int, out.split())
        return (tx, ty), rl
    return run


SHAPES = [(8, 8), (90, 96), (96, 128), (256, 2048), (1024, 1024), (2048, 2048), (4096, 4096)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("tile", [(64, 32), (32, 16), (128, 32)])
@pytest.mark.parametrize("lines", [1, 2, 4])
def test_tuned_choices_hold_for_every_size(rules, shape, tile, lines):
    assert rules(True, tile, True, lines, shape, 8) == (tile, lines)
    assert rules(True, tile, True, lines, shape, 8, single=0) == (tile, lines)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("n_lines", [1, 2, 8, 16])
def test_untuned_choices_go_by_the_size(rules, shape, n_lines):
    tile, lines = rules(False, (64, 32), False, 2, shape, n_lines)
    default_tiles = -(-shape[0] // 32) * -(-shape[1] // 64)
    assert tile == ((32, 16) if default_tiles < 256 else (64, 32))
    assert lines == (2 if -(-shape[0] // 4) * -(-n_lines // 2) >= 1024 else 1)
    assert rules(False, (64, 32), False, 2, shape, n_lines, single=0)[1] == 2
