"""Forms the device code must not use, checked in its source (no GPU, no compiler)."""

import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1503_07659_amd", "csrc")


@pytest.mark.parametrize("name", ["dgvol_adjoint.hpp", "dgvol_forward_direct.hpp", "dgvol_gradd.hpp"])
def test_column_counts_of_buffer_ranges(name):
    """The column count of a buffer range comes from cols_left, never from a guarded subtraction:
    `cond ? min(most, n - c0) : 0` evaluated twice in a function was folded to `most` by the
    compiler, and the range then ran past the arrays (dgvol_device.hpp, cols_left)."""
    with open(os.path.join(CSRC, name)) as fh:
        code = re.sub(r"//[^\n]*", "", fh.read())
    guarded = re.findall(r"\?\s*min\((?:\([^()]*\)|[^(),])+,[^;:]*?-[^;:]*\)\s*:\s*0", code)
    assert not guarded, guarded
