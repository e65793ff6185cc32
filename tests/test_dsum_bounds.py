"""The directed ring sum's bounds at the ends of their range, on the CPU: as constant expressions, in which an overflow of a signed sum
is an error of the compiler."""
import os
import subprocess

import pytest

from paper_2105_14088_amd.build import HIPCC_FLAGS

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2105_14088_amd", "csrc")
MAX = (1 << 21) - 1


def _terms(n, i, j, forward, backward, least):
    """Constants of a move i .. j on an order whose hops all cost `forward` as walked and `backward` the other way."""
    step = backward - forward
    upto_i, upto_j, turned = step * (i + 1), step * (j + 1), step * n
    inner = upto_j - upto_i
    kept, other = 2 * least - 2 * forward + inner, 2 * least - 2 * backward + turned - inner
    first = f"cc::dsum::term_of_first({least}, {least}, {forward}, {backward}, {upto_i})"
    last = f"cc::dsum::term_of_last({least}, {least}, {forward}, {backward}, {upto_j}, {turned})"
    return [f"static_assert(cc::dsum::together({first}.{way}, {last}.{way}) == {want});" for way, want in (("kept", kept), ("other", other))]


@pytest.mark.parametrize("forward,backward,least", [(MAX, 0, 0), (0, MAX, 0), (MAX, MAX, MAX), (MAX - 1, 1, 1)])
def test_bounds_of_the_largest_costs(forward, backward, least, tmp_path):
    lines = []
    for n in (2, 64, 1023, 1024):
        for i, j in {(1, n - 1), (1, 2), (n - 2, n - 1), (n // 2, n - 1), (1, n - 2)}:
            if 1 <= i < j < n:
                lines += _terms(n, i, j, forward, backward, least)
    source = tmp_path / "bounds.hip"
    source.write_text('#include "cc_dsum_bounds.h"\n' + "\n".join(lines) + "\n")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    run = subprocess.run([hipcc, *HIPCC_FLAGS, "-I", CSRC, "--cuda-host-only", "-fsyntax-only", str(source)], capture_output=True, text=True)
    assert run.returncode == 0, run.stderr
