"""The splat's instances: every line count from 1 to 16 has one of its own, so that no count pays for
spare lines.  Read from the kernel names of the library that was built."""

import re

import pytest

from paper_2601_22793_amd import _lib as L


@pytest.mark.parametrize("kernel", ["7k_splat", "9k_splat_x"])
@pytest.mark.parametrize("batched", [0, 1])
def test_every_line_count_has_an_instance(kernel, batched):
    blob = open(L.LIB_PATH, "rb").read()
    pat = rb"_ZN3epr%sILb%dELi(\d+)EEEv" % (kernel.encode(), batched)
    have = sorted({int(n) for n in re.findall(pat, blob)})
    assert have == list(range(1, L.EPR_MAX_LINES + 1))
