"""The gfx950 code the compiler makes of the kernels (no GPU): properties that
no output shows."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2609_20186_amd import build as B

pytestmark = pytest.mark.skipif(shutil.which(B.HIPCC) is None, reason="no hipcc")


class Kernels(dict):
    """Bodies by name; ``meta``: their descriptors."""

    def __init__(self, bodies, meta):
        super().__init__(bodies)
        self.meta = meta


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
    meta = dict(re.findall(r"^\s*\.amdhsa_kernel (\w+)\n(.*?)\.end_amdhsa_kernel", text,
                           re.M | re.S))
    return Kernels({n: bodies[n] for n in meta}, meta)


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


def test_no_scratch(kernels):
    """Scratch reads in a loop that streams rows wait behind the next row's
    loads."""
    used = {n: int(re.search(r"private_segment_fixed_size (\d+)", kernels.meta[n]).group(1))
            for n in kernels}
    assert len([n for n in used if "k_row_draw" in n]) == 10
    assert {n: u for n, u in used.items() if u} == {}


def test_no_select_reads_a_wide_carry(kernels):
    """A condition kept in the scalar condition bit must not be overwritten
    before it is used: no select or branch takes the carry of the upper half of
    a 64-bit sum or difference (a loop over the draw's blocks was once compiled
    like that, ran past its end and read out of bounds)."""
    bad = []
    for n, t in kernels.items():
        last = ""
        for line in t.splitlines():
            op = line.split()[0] if line.startswith("\ts_") else ""
            if op.startswith(("s_cselect", "s_cbranch_scc", "s_cmov")):
                if last.startswith(("s_addc", "s_subb")):
                    bad.append((n, line.strip()))
            elif op and not op.startswith(("s_mov", "s_mul_", "s_nop", "s_waitcnt", "s_load",
                                           "s_cbranch", "s_branch", "s_barrier", "s_ff", "s_flbit")):
                last = op
    assert not bad, bad
