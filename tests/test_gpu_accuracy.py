"""The tuned choices and the column splits are as accurate as the plans they
compete with: a radix-16 or radix-32 plan has fewer passes than the radix-8
one and may not lose more for it."""
import numpy as np
import pytest

import oracle
import paper_2603_27569_amd as sf
from paper_2603_27569_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"
RADIX8 = {256: "n256_e8_b8_p4_r8.8.4_pt", 512: "n512_e8_b4_p4_r8.8.8_pt", 1024: "n1024_e8_b2_p4_r8.8.8.2_pt",
          2048: "n2048_e8_b1_p4_r8.8.8.4_pt", 4096: "n4096_e8_b1_p4_r8.8.8.8_pt",
          8192: "n8192_e8_b1_p4_r8.8.8.8.2_pt", 16384: "n16384_e16_c2_b1_p4_r8.8.8.8.4_pt"}
# Errors are independent from value to value but for the few constants of a
# plan, so an RMS over 2^18 values is good to about 1 / sqrt(2^18) = 0.2%, and
# shapes of the same radices differ by no more than 1% (the order of the
# passes).  A plan may exceed the radix-8 one by the sum of both sides.
SLACK = 1.02


def _rms(y, want):
    y = y.cpu().numpy().astype(np.complex128)
    return float(np.sqrt((np.abs(y - want) ** 2).sum() / (np.abs(want) ** 2).sum()))


def _rows(n):
    x = workloads.plain_normal(n, max(1, (1 << 18) // n), seed=n)
    return x, torch.from_numpy(x).to(DEV)


@pytest.mark.parametrize("n", sorted(RADIX8))
def test_plain_and_ragged(n):
    x, xt = _rows(n)
    want = oracle.fft(x)
    limit = SLACK * _rms(sf.fft(xt, algorithm=sf.FFT_ALGO_SINGLE_PASS, variant=RADIX8[n]), want)
    names = {sf.fft_tune_query(n, b) for b in (1, 100, 200, 300, 400, 600, 900, 1200, 1800, 2500, 3500, 5000, 7000, 9000)}
    for name in sorted(nm for nm in names if nm.startswith("n")):
        assert _rms(sf.fft(xt, algorithm=sf.FFT_ALGO_SINGLE_PASS, variant=name), want) <= limit, name
    plan = sf.RaggedPlan([n] * len(x))
    assert _rms(sf.ragged_fft(xt.reshape(-1), plan, graph=False).reshape(xt.shape), want) <= limit
    plan.close()
    sf.clear_plan_cache()


@pytest.mark.parametrize("n", sorted(RADIX8))
def test_filter_and_gradient(n):
    x, xt = _rows(n)
    batch = len(x)
    h = workloads.plain_normal(n, 1, seed=3)[0]
    ht = torch.from_numpy(h).to(DEV)
    w = np.random.default_rng(4).random(n).astype(np.float32)
    wt = torch.from_numpy(w).to(DEV)
    rows = torch.empty(batch, dtype=torch.float32, device=DEV)
    filtered = oracle.matched_filter(x, h)
    grad = oracle.spectral_energy(x, w)[1]

    def errors(f, e):
        y, g = torch.empty_like(xt), torch.empty_like(xt)
        st = torch.cuda.current_stream().cuda_stream
        pf = sf.Plan(n, batch, sf.FFT_FORWARD, sf.FFT_ALGO_SINGLE_PASS, f)
        pe = sf.Plan(n, batch, sf.FFT_FORWARD, sf.FFT_ALGO_SINGLE_PASS, e)
        sf.fft_exec_matched_filter(pf.handle, xt.data_ptr(), ht.data_ptr(), y.data_ptr(), st)
        sf.fft_exec_spectral_energy(pe.handle, xt.data_ptr(), wt.data_ptr(), 0, g.data_ptr(), rows.data_ptr(), 0, st)
        torch.cuda.synchronize()
        pf.close()
        pe.close()
        return _rms(y, filtered), _rms(g, grad)

    limit = [SLACK * e for e in errors(RADIX8[n], RADIX8[n])]
    batches = (1, 200, 300, 400, 600, 900, 1800, 3500, 5000, 9000)
    for f, e in sorted({(sf.fft_tune_query_filter(n, b), sf.fft_tune_query_fused(n, b)) for b in batches}):
        got = errors(f, e)
        assert got[0] <= limit[0], f
        assert got[1] <= limit[1], e


# rel-RMS of the tiled splits and N1 x 16384 splits that the column kernels
# took the place of.
@pytest.mark.parametrize("n,limit", [(1 << 16, 1.48e-7), (1 << 20, 1.70e-7)])
def test_columns(n, limit):
    x, xt = _rows(n)
    assert _rms(sf.fft(xt), oracle.fft(x)) <= limit
    sf.clear_plan_cache()
