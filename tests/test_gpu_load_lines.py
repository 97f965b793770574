"""Bits do not depend on the loads' cache policy: batches on either side of each
line where the matrix-core and the ragged launcher switch between streaming and
ordinary loads agree on the rows they share."""
import pytest

import paper_2603_27569_amd as sf

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MIB = 1 << 20


@pytest.mark.parametrize("n", [512, 4096, 16384])
@pytest.mark.parametrize("edge", [44 * MIB, 192 * MIB])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_matrix_core(n, edge, dtype):
    batch = edge // (8 * n)
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    x = torch.randn(batch + 1, n, 2, device=DEV, generator=g).to(dtype)
    at, over = (sf.fft_lowp(x[:rows].contiguous(), mma=True) for rows in (batch, batch + 1))
    assert torch.equal(at, over[:batch])
    sf.clear_plan_cache()


@pytest.mark.parametrize("edge", [128 * MIB, 160 * MIB])
def test_ragged(edge):
    n = 4096
    count = edge // (16 * n)
    g = torch.Generator(device=DEV)
    g.manual_seed(edge)
    x = torch.randn((count + 1) * n, dtype=torch.complex64, device=DEV, generator=g)
    ys = []
    for k in (count, count + 1):
        p = sf.RaggedPlan([n] * k)
        ys.append(sf.ragged_fft(x[:k * n].contiguous(), p, graph=False))
        torch.cuda.synchronize()
        p.close()
    assert torch.equal(ys[0], ys[1][:count * n])
