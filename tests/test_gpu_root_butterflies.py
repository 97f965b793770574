"""Impulses through every root of the in-register DFTs: a 1 at element p gives
e^{-+2 pi i p k / n} at every bin k, one product chain per bin.  The ragged, the
plain complex64 and the column kernels correct the roots that round most, the
16-bit kernels take them as FP32 rounds them."""
import numpy as np
import pytest

import paper_2603_27569_amd as sf

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"
U = 2.0 ** -24


def _case(n, inverse):
    gen = np.random.default_rng(n)
    p = np.unique(np.concatenate([n // 32 * np.arange(32), gen.integers(0, n, 33)]))
    x = np.zeros((len(p), n), dtype=np.complex64)
    x[np.arange(len(p)), p] = 1.0
    k = (p[:, None] * np.arange(n)[None, :]) % n
    return x, np.exp((2j if inverse else -2j) * np.pi * k / n)


# One bin is a chain of one root per radix-2 stage (two rounded constants and
# two fused operations, or a constant, a product, a sum) and one twiddle per
# pass (a rounded table entry and a product): at most 6 U per stage and per
# pass, and there are no more passes than stages.
def _bound(n):
    return 12 * U * np.log2(n)


@pytest.mark.parametrize("inverse", [False, True], ids=["forward", "backward"])
@pytest.mark.parametrize("n", [256, 512, 1024, 2048, 4096, 8192, 16384])
def test_impulses(n, inverse):
    x, want = _case(n, inverse)
    direction = sf.FFT_BACKWARD if inverse else sf.FFT_FORWARD
    xt = torch.from_numpy(x).to(DEV)
    plan = sf.RaggedPlan([n] * len(x), direction)
    got = {"ragged": sf.ragged_fft(xt.reshape(-1), plan, graph=False).reshape(xt.shape),
           "plain": sf.fft(xt, inverse=inverse)}
    for name, y in got.items():
        assert np.abs(y.cpu().numpy() - want).max() <= _bound(n), name
    half = torch.view_as_real(xt).to(torch.float16)
    y = torch.view_as_complex(sf.fft_lowp(half, inverse=inverse).float().contiguous()).cpu().numpy()
    assert np.abs(y - want).max() <= _bound(n) + 2.0 ** -11 * np.sqrt(2), "binary16"  # the result's rounding


@pytest.mark.parametrize("inverse", [False, True], ids=["forward", "backward"])
@pytest.mark.parametrize("n", [1 << 15, 1 << 17])
def test_impulses_columns(n, inverse):
    x, want = _case(n, inverse)
    y = sf.fft(torch.from_numpy(x).to(DEV), inverse=inverse).cpu().numpy()
    assert np.abs(y - want).max() <= _bound(n)
