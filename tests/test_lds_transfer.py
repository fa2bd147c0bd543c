"""The transfer from memory into LDS is inline assembly, which the compiler's hazard pass does not look into: the wait
states of the hardware have to be inside the block."""
import os
import re
import subprocess

import pytest

from paper_2306_15799_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.parametrize("opt", ["-O1", "-O3"])
def test_wait_states_inside_the_block(opt):
    res = subprocess.run([build.find_hipcc(), "-x", "hip", "--offload-arch=gfx950", "--offload-device-only", "-S", "-std=c++17", opt,
                          "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, os.path.join(HERE, "host", "lds_transfer.hip"),
                          "-o", "-"], check=True, capture_output=True, text=True)
    blocks = re.findall(r"#ASMSTART\n(.*?);*#ASMEND", res.stdout, re.S)
    blocks = [b for b in blocks if " lds" in b]
    assert len(blocks) == 1, res.stdout
    lines = [x.strip() for x in blocks[0].strip().splitlines()]
    assert lines[-1].startswith("buffer_load_dwordx4") and lines[-1].endswith("lds")
    # a scalar register written by a vector instruction just before the block is read by the load
    states = sum(int(x.split()[1]) + 1 if x.startswith("s_nop") else 1 for x in lines[:-1])
    assert states >= 5, lines
    # m0 and the load that uses it
    m0 = max(i for i, x in enumerate(lines) if re.match(r"s_\w+ m0,", x))
    assert m0 < len(lines) - 2, lines
