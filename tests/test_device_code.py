"""The gfx950 code the compiler makes of the kernels (no GPU): properties that
no output shows."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2609_20186_amd import build as B

pytestmark = pytest.mark.skipif(shutil.which(B.HIPCC) is None, reason="no hipcc")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Assembly of every kernel of the product library, by (mangled) name."""
    out = str(tmp_path_factory.mktemp("asm") / "kernels.s")
    subprocess.run([B.HIPCC] + B.COMMON + B.DEVICE +
                   ["-x", "hip", "--cuda-device-only", "-S",
                    os.path.join(B.CSRC, "switchsd_kernels.hip"), "-o", out],
                   check=True, capture_output=True, text=True, timeout=600)
    text = open(out).read()
    bodies = dict(re.findall(r"^(\w+):\s*; @\1\n(.*?)^\.Lfunc_end", text, re.M | re.S))
    names = re.findall(r"^\s*\.amdhsa_kernel (\w+)", text, re.M)
    return {n: bodies[n] for n in names}


def test_buffer_reads_are_bounded(kernels):
    """The row draw reads past a row's end by design and relies on the buffer's
    record count, which bounds the lane's offset and the instruction's
    constant but not the scalar offset: that one is 0 in every buffer load."""
    loads = {n: re.findall(r"buffer_load_\w+ \S+ \S+ s\[\d+:\d+\], (\S+) offen", t)
             for n, t in kernels.items()}
    rows = [n for n in kernels if "k_row_draw" in n]
    assert rows and all(loads[n] for n in rows)
    assert sum(map(len, loads.values())) == sum(t.count("buffer_load_") for t in kernels.values())
    assert {n: sorted(set(o)) for n, o in loads.items() if set(o) - {"0"}} == {}
