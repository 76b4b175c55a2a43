"""What the compiler makes of a kernel, read in its assembly: no GPU."""
import os
import re
import subprocess

import pytest

from paper_2512_15742_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
def test_searches_keep_their_arrays_in_registers(tmp_path):
    """An array that a lane indexes by a value of its own goes to scratch or to LDS, and its address there is read from the
    launch's packet in host memory: 9 to 12 us of a search that takes 8."""
    src, out = os.path.join(build.CSRC, "kan_assign.hip"), str(tmp_path / "kan_assign.s")
    subprocess.run([build.HIPCC, *build.COMMON, "--offload-device-only", "-S", src, "-o", out], check=True, capture_output=True, timeout=600)
    with open(out) as f:
        kernels = re.findall(r"\.amdhsa_kernel (\S+)(.*?)\.end_amdhsa_kernel", f.read(), re.S)
    names = " ".join(name for name, _ in kernels)
    for part in ("kan_assign_own_kernelItLi2ELb1E", "kan_assign_own_kernelIjLi4ELb0E", "kan_assign_whole_kernel", "kan_assign_bounded_kernel"):
        assert part in names
    for name, head in kernels:
        assert re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", head).group(1) == "0", name
        assert "amdhsa_user_sgpr_dispatch_ptr 1" not in head, name
