"""The loss total of the fused energy kernels: every row published before the
workgroups' counters let the last one add them, in one fixed order of FP32
additions, so the total is compared bit for bit with the same additions of the
returned rows."""
import numpy as np
import pytest

import paper_2603_27569_amd as sf

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _total(rows):
    """1024 lanes add rows v, v + 1024, ... in turn, then a halving tree."""
    v = np.zeros(1024, dtype=np.float32)
    for i in range(0, len(rows), 1024):
        part = rows[i:i + 1024]
        v[:len(part)] += part
    h = 512
    while h:
        v[:h] += v[h:2 * h]
        h //= 2
    return v[0]


# Batches around the 16 first-level counters, the 1024 lanes of the sum and the
# 4096 / 8192 / 16384 rows of one round of its loads; lengths with several
# transforms per workgroup, one, and registers full.
@pytest.mark.parametrize("want_grad", [True, False], ids=["grad", "loss"])
@pytest.mark.parametrize("n,batches", [(256, (1, 15, 17, 1025, 4097, 16385, 16390)), (1024, (16, 33, 1023, 8193)),
                                       (4096, (1, 31, 255, 513, 1030)), (16384, (2, 17, 100, 500))])
def test_total_is_the_ordered_sum(n, batches, want_grad):
    gen = torch.Generator(device=DEV).manual_seed(n)
    w = torch.rand(n, device=DEV, generator=gen)
    for b in batches:
        x = torch.randn(b, n, dtype=torch.complex64, device=DEV, generator=gen)
        for _ in range(3):  # the counters are left zeroed
            total, rows = sf.spectral_energy(x, w, want_grad=want_grad)[:2]
            assert float(total) == float(_total(rows.cpu().numpy())), (n, b)
