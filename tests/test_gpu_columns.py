"""Column splits of the long transforms (N = N1 x N2, 2^15 .. 2^20) against the
oracle: every split in both directions, with the ordinary and the streaming
cache policy (batches on either side of the size where the launcher switches),
in place, and with a launch limit that cuts the batch into single rows.

The gates are those of the other lengths (metrics.gate: rel-RMS <= 5e-6 per
row), far above what an FP32 transform of this depth loses (about 2e-7)."""
import pytest

import oracle
import paper_2603_27569_amd as sf
from paper_2603_27569_amd import metrics, workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SPLITS = [(1 << 15, "fs32768_tile128x256"), (1 << 16, "fs65536_tile256x256"), (1 << 17, "fs131072_tile256x512"),
          (1 << 18, "fs262144_tile512x512"), (1 << 19, "fs524288_tile1024x512"),
          (1 << 20, "fs1048576_tile1024x1024")]
SWITCH = (256 << 20) // 24  # elements above which the launcher streams


@pytest.mark.parametrize("n,name", SPLITS, ids=[s[1] for s in SPLITS])
@pytest.mark.parametrize("inverse", [False, True], ids=["fwd", "bwd"])
def test_column_split_rows_both_policies_in_place(n, name, inverse):
    edge = SWITCH // n
    for batch in (1, 3, edge, edge + 1):
        g = torch.Generator(device=DEV)
        g.manual_seed(n + batch)
        x = torch.randn(batch, n, dtype=torch.complex64, device=DEV, generator=g)
        rows = sorted({0, batch // 2, batch - 1})
        xs = x[rows].cpu().numpy()
        y = sf.fft(x, inverse=inverse, algorithm=sf.FFT_ALGO_FOUR_STEP, variant=name)
        ref = oracle.fft(xs, inverse=inverse)
        ok, worst, _, ab = metrics.gate(y[rows].cpu().numpy(), ref, xs)
        assert ok, (batch, worst, ab)
        z = x.clone()
        sf.fft(z, inverse=inverse, out=z, algorithm=sf.FFT_ALGO_FOUR_STEP, variant=name)
        assert torch.equal(z, y), batch
    sf.clear_plan_cache()


def test_column_split_single_row_launches():
    n = 1 << 16
    x = torch.from_numpy(workloads.plain_normal(n, 5, seed=17)).to(DEV)
    want = sf.fft(x)
    try:
        sf.fft_set_launch_limit(16)  # one row of 16 tiles per launch
        assert torch.equal(sf.fft(x), want)
        sf.fft_set_launch_limit(1)  # below one row: still whole rows
        assert torch.equal(sf.fft(x), want)
    finally:
        sf.fft_set_launch_limit(0)


def test_retired_split_names_are_accepted():
    for n, old in ((1 << 18, "fs262144_tile512x512_c2"), (1 << 20, "fs1048576_tile1024x1024_c2")):
        p = sf.Plan(n, 1, variant=old)
        assert p.describe()["four_step"]["name"] == old[:-3]
        p.close()
        x = torch.from_numpy(workloads.plain_normal(n, 1, seed=n)).to(DEV)
        assert torch.equal(sf.fft(x, algorithm=sf.FFT_ALGO_FOUR_STEP, variant=old), sf.fft(x))
    sf.clear_plan_cache()
