"""Checks of the kernels' text, on the CPU."""
import glob
import os
import re

import pytest

from paper_2105_14088_amd.build import DYNAMIC_LDS_AT_0, check_dynamic_lds

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


def _listing(folder, kernel, lds):
    name = f"_ZN2cc{len(kernel)}{kernel}ILi10ELb0EEEvPKi"
    (folder / "cc_batch-hip-amdgcn-amd-amdhsa-gfx950.s").write_text(
        f"\t.amdhsa_kernel {name}\n\t\t.amdhsa_group_segment_fixed_size {lds}\n\t\t.amdhsa_next_free_vgpr 64\n\t.end_amdhsa_kernel\n")


@pytest.mark.parametrize("kernel", DYNAMIC_LDS_AT_0)
def test_a_build_with_lds_before_what_a_kernel_addresses_from_0_is_refused(kernel, tmp_path):
    _listing(tmp_path, kernel, 0)
    check_dynamic_lds(str(tmp_path))
    _listing(tmp_path, kernel, 4)
    with pytest.raises(RuntimeError, match=kernel):
        check_dynamic_lds(str(tmp_path))
    _listing(tmp_path, "some_other_kernel", 0)
    with pytest.raises(RuntimeError, match=kernel):
        check_dynamic_lds(str(tmp_path))


def test_kernels_that_address_lds_from_an_integer_are_looked_at_by_the_build():
    for path in SOURCES:
        for at in re.finditer(r"address_space\(3\)\)\)[^;]*\(uintptr_t\)", code_of(path)):
            before = re.findall(r"__global__[^{;]*?\b(\w+)\s*\(\s*const", code_of(path)[: at.start()])
            assert before[-1] in DYNAMIC_LDS_AT_0
