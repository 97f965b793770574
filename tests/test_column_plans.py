"""What column splits report about themselves, and the tables they run on."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2603_27569_amd as sf

CSRC = os.path.join(os.path.dirname(os.path.abspath(sf.__file__)), "csrc")
# N, then the radices of the N2-point first and the N1-point second columns
SPLITS = [(1 << 15, (16, 16), (16, 8)), (1 << 16, (16, 16), (16, 16)), (1 << 17, (32, 16), (16, 16)),
          (1 << 18, (32, 16), (32, 16)), (1 << 19, (32, 16), (32, 32)), (1 << 20, (32, 32), (32, 32))]


def _entries(first, second):
    n2, n1 = first[0] * first[1], second[0] * second[1]
    return n2 + n1 + n2 * (second[0] + second[1])


@pytest.mark.gpu
@pytest.mark.parametrize("n,first,second", SPLITS)
def test_plan_describes_the_kernels_it_runs(n, first, second):
    p = sf.Plan(n, 3)
    d = p.describe()
    p.close()
    v = d["variant"]
    assert v["kind"] == "columns" and v["name"] == d["four_step"]["name"] and v["n"] == n
    assert tuple(v["first_radices"]) == first and tuple(v["second_radices"]) == second
    assert v["twiddle_entries"] == _entries(first, second)
    for key, (r0, r1) in (("variant_resources", first), ("second_resources", second)):
        tile = 32 if r1 == 8 else 16
        r = d[key]
        # one padded column tile, in halves where a lane holds 32 values
        assert r["lds_bytes"] == r0 * tile * (r1 + 1) * (4 if r0 == 32 else 8)
        assert r["max_threads"] >= tile * r1 and 0 < r["vgprs"] <= 128 and r["scratch_bytes_per_lane"] == 0


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_column_tables_rounded_once_from_fp64(tmp_path):
    """Every entry of the tables on the device is the root it stands for, rounded
    once: within half an ulp of the exact one (plus FP64 evaluation slack)."""
    src = tmp_path / "t.cpp"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include "twiddles.hpp"\n'
                   "int main(int, char** a) {\n"
                   "  stockfft::ColumnShape c{atoi(a[1]), atoi(a[2]), atoi(a[3]), atoi(a[4]), atoi(a[5])};\n"
                   "  std::vector<float> t;\n  stockfft::column_twiddles(c, t);\n"
                   "  if ((int64_t)t.size() != 2 * stockfft::column_twiddle_entries(c)) return 1;\n"
                   "  return fwrite(t.data(), 4, t.size(), stdout) != t.size();\n}\n")
    exe = str(tmp_path / "t")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", exe], check=True)
    for n, (a0, a1), (b0, b1) in SPLITS:
        tile = 32 if b1 == 8 else 16
        got = np.frombuffer(subprocess.run([exe, *map(str, (a0, a1, b0, b1, tile))], check=True,
                                           capture_output=True).stdout, np.float32)
        n2, n1 = a0 * a1, b0 * b1
        outer = np.multiply.outer
        k2 = np.arange(n2).reshape(-1, 1, tile)  # tiles of adjacent k2
        exps = [(outer(np.arange(a0), np.arange(a1)), n2), (outer(np.arange(b0), np.arange(b1)), n1),
                (k2 * np.arange(b1)[None, :, None], n), (k2 * np.arange(b0)[None, :, None], n // b1)]
        angle = np.concatenate([2 * np.pi * (m % L).ravel() / L for m, L in exps])
        want = np.stack([np.cos(angle), -np.sin(angle)], -1).ravel()
        assert got.shape == want.shape
        half_ulp = 0.5 * np.spacing(np.abs(want).astype(np.float32)).astype(np.float64)
        assert (np.abs(got - want) <= half_ulp * (1 + 1e-6) + 1e-15).all(), n
