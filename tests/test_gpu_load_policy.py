"""The row loads' cache policy changes nothing but time: batches on either side
of the sizes where a launcher switches between streaming and ordinary loads
give the same bits for the rows they share."""
import pytest

import oracle
import paper_2603_27569_amd as sf
from paper_2603_27569_amd import metrics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
BELOW, ABOVE = 24 << 20, 192 << 20  # bytes of rows in and out between which loads are ordinary


@pytest.mark.parametrize("edge", [BELOW, ABOVE])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_matrix_core_rows_same_bits_either_policy(edge, dtype):
    n = 2048
    batch = edge // (2 * n * 4)
    g = torch.Generator(device=DEV)
    g.manual_seed(edge)
    x = torch.randn(batch + 1, n, 2, device=DEV, generator=g).to(dtype)
    want = sf.fft_lowp(x[:batch - 1].contiguous(), mma=True)
    for rows in (batch, batch + 1):
        assert torch.equal(sf.fft_lowp(x[:rows].contiguous(), mma=True)[:batch - 1], want)
    sf.clear_plan_cache()


@pytest.mark.parametrize("edge", [BELOW, ABOVE])
def test_ragged_same_bits_either_policy(edge):
    n = 16384
    count = edge // (16 * n)
    g = torch.Generator(device=DEV)
    g.manual_seed(edge + 1)
    x = torch.randn((count + 1) * n, dtype=torch.complex64, device=DEV, generator=g)
    ys = []
    for k in (count - 1, count, count + 1):
        p = sf.RaggedPlan([n] * k)
        ys.append(sf.ragged_fft(x[:k * n].contiguous(), p, graph=False))
        torch.cuda.synchronize()
        p.close()
    short = (count - 1) * n
    assert torch.equal(ys[0], ys[1][:short]) and torch.equal(ys[0], ys[2][:short])
    xs = x[short - n:short].cpu().numpy().reshape(1, n)
    ok, worst, _, ab = metrics.gate(ys[1][short - n:short].cpu().numpy().reshape(1, n), oracle.fft(xs), xs)
    assert ok, (worst, ab)
