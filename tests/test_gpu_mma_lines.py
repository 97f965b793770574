"""The matrix-core kernels on both sides of the lines between two and four
blocks of 32 butterflies per wave at 2048 and 4096 points (12288 and 16384
blocks of a launch): rows at the ends against the FP64 oracle, the rest the same
bits as a launch with one block per wave."""
import numpy as np
import pytest

import oracle
import paper_2603_27569_amd as sf
from paper_2603_27569_amd import metrics, workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("inverse", [False, True], ids=["forward", "backward"])
@pytest.mark.parametrize("n,batch", [(n, line * 512 // n + extra) for n, line in
                                     [(2048, 12288), (2048, 16384), (4096, 12288), (4096, 16384)]
                                     for extra in (0, 1)])
def test_blocks_per_wave(n, batch, inverse, fmt):
    dtype = torch.float16 if fmt == "f16" else torch.bfloat16
    g = torch.Generator(device="cuda:0")
    g.manual_seed(n + batch)
    x = torch.randn(batch, n, 2, device="cuda:0", generator=g).to(dtype)
    out = torch.full((batch + 1, n, 2), 7.0, dtype=dtype, device="cuda:0")
    sf.fft_lowp(x, inverse=inverse, out=out[:batch], mma=True)
    assert torch.all(out[batch] == 7.0)  # nothing stored past the last row
    rows = [0, 1, batch // 2, batch - 2, batch - 1]
    xv = torch.view_as_complex(x[rows].float()).cpu().numpy().astype(np.complex128)
    got = torch.view_as_complex(out[rows].float()).cpu().numpy()
    ok, worst, _, ab = metrics.gate_storage(got, oracle.fft(xv, inverse=inverse), xv, fmt, mma=True)
    assert ok, (worst, ab)
    small = 8 * 4096 // n
    for lo in range(0, batch, max(small, batch // 3)):
        part = x[lo:lo + small].contiguous()
        assert torch.equal(sf.fft_lowp(part, inverse=inverse, mma=True), out[lo:lo + len(part)])
    sf.clear_plan_cache()
