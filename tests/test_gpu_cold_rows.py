"""Calls whose rows come from HBM keep up with the calls they compete with."""
import statistics

import pytest

import paper_2603_27569_amd as sf
from paper_2603_27569_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _us(launch, k, repeats=5):
    """Median device time of one launch, us: a graph of k launches on k different
    buffers, replayed."""
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for i in range(3):
            launch(i, stream.cuda_stream)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        for i in range(k):
            launch(i, stream.cuda_stream)
    times = []
    for _ in range(repeats + 1):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        with torch.cuda.stream(stream):
            a.record(stream)
            for _ in range(4):
                graph.replay()
            b.record(stream)
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / (4 * k))
    return statistics.median(times[1:])


def test_matrix_cores_keep_up_with_the_vector_units():
    """binary16 4096 x 1800 from HBM: the same bytes, and the DFTs off the vector
    units, so the matrix-core form has no reason to take longer.  (It takes 1.2
    times as long with 256 lanes per transform and 0.93 with 128; the line lies
    halfway.)"""
    n, batch, k = 4096, 1800, 18
    x = torch.randn(k, batch, n, 2, device=DEV, dtype=torch.float16)
    y = torch.empty_like(x)
    p = sf.Plan(n, batch, sf.FFT_FORWARD, sf.FFT_ALGO_SINGLE_PASS)
    vector, matrix = (_us(lambda i, st, io=io: sf.fft_exec_io(p.handle, x[i % k].data_ptr(), y[i % k].data_ptr(), io, st), k)
                      for io in (sf.FFT_IO_C16, sf.FFT_IO_C16_MMA))
    p.close()
    assert matrix <= 1.06 * vector, (matrix, vector)


@pytest.mark.parametrize("count", [1200, 1500])
def test_ragged_plan_takes_the_grain_that_fits(count):
    """8192-point transforms go one or two to a task; which is better depends on
    how the batch divides over the chip (1200 lengths 22.2 / 24.5 us, 1500 31.0 /
    27.0).  A plan left to itself is as good as the better of the two; 4% is
    well under what the other grain costs and above what two runs differ by."""
    sizes = [int(s) for s in workloads.ragged_sizes(count, 1005)]
    total, k = sum(sizes), 12
    x = torch.randn(k, total, dtype=torch.complex64, device=DEV)
    y = torch.empty_like(x)

    def us(shape):
        sf.fft_tune_clear_ragged()
        if shape:
            sf.fft_tune_set_ragged(8192, shape)
        p = sf.RaggedPlan(sizes)
        t = _us(lambda i, st: p.exec_direct(x[i % k].data_ptr(), y[i % k].data_ptr(), st), k)
        p.close()
        return t

    try:
        named = [us(shape) for shape in sf.fft_ragged_shapes(8192)]
        assert us(None) <= 1.04 * min(named), named
    finally:
        sf.fft_tune_clear_ragged()
