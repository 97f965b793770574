"""Transforms of up to 64 lanes exchange without workgroup barriers: what the
variant text's "barriers" counts for them are points of one wave's order."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2603_27569_amd as sf
from paper_2603_27569_amd import build

SHAPES = [(256, 4, 4, "4, 4, 4, 4"), (512, 8, 4, "8, 8, 8"), (1024, 16, 2, "16, 16, 4"), (1024, 8, 2, "8, 8, 8, 2"),
          (2048, 8, 1, "8, 8, 8, 4")]


@pytest.mark.skipif(not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)), reason="needs hipcc")
def test_barriers_of_the_compiled_kernels(tmp_path):
    src = tmp_path / "k.hip"
    src.write_text('#include "kernels.hpp"\nnamespace stockfft {\n' + "".join(
        f"template __global__ void k_stockham<Shape<{n}, {e}, {b}, 4, {r}>, false>(const c32*, c32*, const c32*, int64_t);\n"
        for n, e, b, r in SHAPES) + "}\n")
    asm = tmp_path / "k.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, "-S", "--cuda-device-only", str(src), "-o", str(asm)],
                   check=True, capture_output=True)
    bodies = re.split(r"^(_Z\w*k_stockham\w*):", asm.read_text(), flags=re.M)[1:]
    counted = dict(zip(bodies[::2], (len(re.findall(r"^\s+s_barrier\b", b.split("s_endpgm")[0], re.M)) for b in bodies[1::2])))
    by_shape = {(v["n"], v["values_per_lane"], v["radices"].__len__()): v for v in sf.variants() if v["kind"] == "single"}
    for n, e, b, r in SHAPES:
        (barriers,) = [c for name, c in counted.items() if f"Li{n}ELi{e}ELi{b}E" in name]
        v = by_shape[n, e, r.count(",") + 1]
        assert v["lanes_per_transform"] == n // e
        assert barriers == (0 if v["lanes_per_transform"] <= 64 else v["barriers"]), (n, e)
