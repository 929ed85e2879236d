"""The benchmark's kernel records without a device: the names it looks its counter records up by are
kernels of the built library, and a record goes stale with any header its kernel's source includes."""

import os
import re
import shutil

import pytest

import bench
from paper_2601_22793_amd import _lib as L

SINGLE = [(256, 256), (1024, 1024), (2048, 2048), (2160, 2560), (4096, 4096)]
BATCH = [(1024, 1024), (2048, 2048), (2160, 2560)]


def library_kernels():
    """Kernel template instances of the library as a profiler prints them."""
    blob = open(L.LIB_PATH, "rb").read()
    out = set()
    for m in re.finditer(rb"_ZN3epr\d+(k_[a-z_]+)I((?:L[bi]\d+E)+)E", blob):
        args = [("true" if v == b"1" else "false") if t == b"b" else v.decode()
                for t, v in re.findall(rb"L([bi])(\d+)E", m.group(2))]
        out.add(f"{m.group(1).decode()}<{', '.join(args)}>")
    return out


@pytest.mark.parametrize("stage", ["maxgrad", "splat", "local", "rowfft", "colfft", "rowinv"])
def test_kernel_names_are_kernels_of_the_library(stage):
    have = library_kernels()
    for n_lines in (1, 2, 3, 5, 8, 10, 16):
        for batched, shapes in [(False, [s]) for s in SINGLE] + [(True, BATCH[:2]), (True, BATCH[2:])]:
            cls = bench.size_class(*max(shapes))
            lines = bench.row_pass_lines(batched, shapes[0][0], n_lines, None)
            for model in ("local_l1", "local_l2", "nonlocal"):
                name = bench.kernel_instance(stage, cls, batched, n_lines, lines, shapes, model)
                assert name in have, (name, shapes, n_lines)


def test_untuned_row_lines_go_by_the_size():
    assert bench.row_pass_lines(False, 2048, 8, None) == 2
    assert bench.row_pass_lines(False, 256, 8, None) == 1
    assert bench.row_pass_lines(True, 256, 8, None) == 2
    assert bench.row_pass_lines(False, 256, 8, {"row_lines": 4}) == 4


@pytest.mark.parametrize("stage,header", [("splat", "split_bin.h"), ("local", "split_bin.h"),
                                          ("splat", "dev_common.h"), ("rowfft", "fft_lds.h"),
                                          ("colfft", "spectral.h"), ("rowinv", "epr_internal.h")])
def test_a_record_goes_stale_with_its_headers(tmp_path, monkeypatch, stage, header):
    csrc = os.path.join("paper_2601_22793_amd", "csrc")
    shutil.copytree(os.path.join(bench.ROOT, csrc), tmp_path / csrc)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    before = bench.source_digest(stage)
    assert bench.source_digest(stage) == before
    with open(tmp_path / csrc / header, "a") as fh:
        fh.write("// changed\n")
    assert bench.source_digest(stage) != before
