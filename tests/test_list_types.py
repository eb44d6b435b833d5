"""The lists of 16-bit entries that a wave of the adjoint fills and walks without a barrier between: what is read
or written wider than an entry must be allowed to alias the entries.  Read from the compiler's own output before
any optimisation: an access at the address of a 16-bit element is of that type or tagged as one that may alias."""
import os
import re
import subprocess

import pytest

from paper_2404_01133_amd import build

HIPCC = None
try:
    HIPCC = build.hipcc()
except RuntimeError:
    pass


def _front_end_ir(source, out):
    subprocess.run([HIPCC] + build.flags() + ["-S", "-emit-llvm", "-Xclang", "-disable-llvm-passes",
                                              "--cuda-device-only", source, "-o", out],
                   check=True, capture_output=True)
    with open(out) as f:
        return f.read()


@pytest.mark.skipif(HIPCC is None, reason="needs hipcc")
def test_wide_accesses_to_the_adjoints_lists_may_alias(tmp_path):
    ir = _front_end_ir(os.path.join(build.CSRC, "raster_bwd.hip"), str(tmp_path / "bwd.ll"))
    access = r"(?:load|store) (?P<type>\S+|<\d+ x \S+)>?(?: [^,\n]*)?, ptr (?:addrspace\(\d+\) )?%(?P<at>\S+), align \d+, !tbaa (?P<tag>!\d+)"
    wide = []
    pointers = set()
    for line in ir.splitlines():
        if line.startswith("define"):
            pointers = set()
        g = re.match(r"\s*%(\S+) = getelementptr inbounds (i16|<4 x i32>),", line)
        if g:
            pointers.add(g.group(1))
        a = re.search(access, line)
        if a and a.group("at") in pointers and a.group("type") != "i16":
            wide.append(a.group("tag"))
    assert len(wide) >= 40  # the fill and the walk of each of the twenty kernels
    for tag in set(wide):
        # (scalar access type, base type, offset); the type that may alias anything is "omnipotent char"
        kind = re.search(r"^%s = !\{(!\d+), \1, i64 0\}" % re.escape(tag), ir, re.M).group(1)
        assert re.search(r'^%s = !\{!"omnipotent char",' % re.escape(kind), ir, re.M), tag
