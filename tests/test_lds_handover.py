"""Data that lanes of one wavefront hand to others through LDS is fenced.

The hardware keeps a wavefront's LDS operations in order; the compiler does
only where a fence says so, or where it cannot tell two addresses apart, on
which nothing may rest.  Results show a missing fence only once a compiler
uses its freedom, so this reads the kernels' own intermediate code instead:
each of the Gram kernels writes a tile as 8-element vectors and reads it back
as 4-element ones, and needs a wavefront fence between the last store and the
first load, and another after the last load, before the next tile's stores.
"""
import os
import re
import subprocess

import pytest

from paper_2311_18715_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
def test_gram_tiles_are_fenced(tmp_path):
    out = tmp_path / "gram.ll"
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", "-emit-llvm", "-o", str(out), os.path.join(build.CSRC, "gram.hip")],
                   check=True, stderr=subprocess.DEVNULL)
    text = out.read_text()
    kernels = [f for f in re.split(r"^(?=define )", text, flags=re.M) if f.startswith("define") and "k_gram" in f.split("(")[0]]
    assert len(kernels) == 2
    for f in kernels:
        f = f[:f.index("\n}")]
        seen = [m.group() for m in re.finditer(r'store <8 x i16>[^\n]*addrspace\(3\)|load <4 x i16>, ptr addrspace\(3\)|fence syncscope\("wavefront"\) (?:release|acquire)', f)]
        word = "".join({"s": "S", "l": "L"}.get(x[0], "R" if "release" in x else "A") for x in seen)
        assert re.fullmatch(r"S+RAL+RA", word), word
