"""What the compiler makes of the kernels, read from the assembly of this repository's own sources (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_1802_06058_amd import build


def _assembly(source, tmp_path):
    out = str(tmp_path / "k.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "-S", "--offload-device-only", os.path.join(build.CSRC, source), "-o", out],
                   check=True, capture_output=True)
    with open(out) as f:
        return f.read()


@pytest.mark.parametrize("source", ["vgc_unpack.hip", "vgc_sqgrad_fc.hip", "vgc_sqgrad_conv_f32.hip"])
def test_buffer_loads_are_bounded_by_their_whole_offset(source, tmp_path):
    """Kernels that ask for rows or rounds past an array's end rely on the range of the buffer resource to answer them with
    zeros.  The offset in the vector register and the instruction's own are documented to be held against it, the scalar
    one is not, so no load may carry any part of its place there."""
    loads = re.findall(r"buffer_load_\w+\s+(?:v\S+),\s+(?:v\S+|off),\s+s\[\d+:\d+\],\s+(\S+)", _assembly(source, tmp_path))
    assert loads
    assert set(loads) == {"0"}
