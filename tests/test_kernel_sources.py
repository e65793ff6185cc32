"""Checks of the kernels' text, on the CPU."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2105_14088_amd", "csrc")
SOURCES = sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h")))


def code_of(path):
    text = open(path).read()
    return re.sub(r"//[^\n]*|/\*.*?\*/", "", text, flags=re.S)


@pytest.mark.parametrize("path", SOURCES, ids=os.path.basename)
def test_no_workgroup_reduction_of_the_library(path):
    """__syncthreads_and and its kin reduce over the whole workgroup and promise nothing once wavefronts of it have
    returned, as they have in the searches whose spare wavefronts only make the partner lists."""
    assert not re.search(r"__syncthreads_(and|or|count)\s*\(", code_of(path))
