"""The matrix-core kernels on both sides of each line between one, two and
four blocks of 32 butterflies per wave, with ragged last workgroups, against
the FP64 oracle on the stored values."""
import numpy as np
import pytest

import oracle
import paper_2603_27569_amd as sf
from paper_2603_27569_amd import metrics, workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# Blocks of a transform: n / 512.  The lines lie at 4096 and 8192 blocks.
EDGES = [(n, max(1, lines * 512 // n) + extra)
         for n, lines in [(512, 4096), (512, 8192), (1024, 4096), (1024, 8192),
                          (2048, 4096), (4096, 4096), (8192, 4096)]
         for extra in (0, 1)] + [(512, 8195), (16384, 131)]


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("n,batch", EDGES)
def test_blocks_per_wave(fmt, n, batch):
    gen = np.random.default_rng(n + batch)
    x = (gen.standard_normal((batch, n)) + 1j * gen.standard_normal((batch, n))).astype(np.complex64)
    stored, xv = workloads.to_storage(x, fmt)
    t = torch.from_numpy(np.ascontiguousarray(stored))
    if fmt == "bf16":
        t = t.view(torch.int16).view(torch.bfloat16)
    guarded = torch.full((batch + 1, n, 2), 7.0, dtype=t.dtype, device="cuda:0")
    rows = sorted({0, 1, 2, 3, batch // 2, batch - 3, batch - 2, batch - 1})
    p = {inv: sf.Plan(n, batch, sf.FFT_BACKWARD if inv else sf.FFT_FORWARD, sf.FFT_ALGO_SINGLE_PASS)
         for inv in (False, True)}
    io = sf.FFT_IO_C16_MMA if fmt == "f16" else sf.FFT_IO_BC16_MMA
    xt = t.to("cuda:0")
    for inv in (False, True):
        guarded[:batch] = 0
        sf.fft_exec_io(p[inv].handle, xt.data_ptr(), guarded.data_ptr(), io,
                       torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        p[inv].close()
        assert torch.all(guarded[batch] == 7.0)  # nothing stored past the last row
        a = guarded[rows].cpu()
        if fmt == "bf16":
            v = workloads.bf16_value(a.view(torch.int16).numpy().view(np.uint16)).astype(np.float64)
        else:
            v = a.numpy().astype(np.float64)
        ok, worst, _, ab = metrics.gate_storage(v[..., 0] + 1j * v[..., 1],
                                                oracle.fft(xv[rows], inverse=inv), xv[rows], fmt, mma=True)
        assert ok, (inv, worst, ab)
