"""Workloads of this library at the sizes a program calls it with.

``listed()`` gives the fixed cases, ``draw(rng)`` another one of the same
ranges, ``prepare(case, seed)`` what a program has on the GPU before the call,
``run(state)`` one pass through the public entry points, ``work(case)`` the
bytes and operations the pass cannot do without, and ``exact(case, seed)`` the
same outputs in FP64 from torch's own FFT.

Kinds of pass:

  fft      the unscaled transform of contiguous complex64 rows, either
           direction; 256 .. 16384 points in one dispatch, up to 2^20 by the
           four-step (``fft``)
  grad     the transform as a differentiable layer: forward, then the gradient
           of its input for a given upstream gradient (``FFTFunction``)
  energy   the fused forward -> weight -> adjoint kernel: total and per-row
           weighted spectral energy and the gradient (``spectral_energy``)
  train    the same loss as an autograd function: loss-only forward, then the
           gradient scaled by the upstream one (``SpectralEnergyFunction``)
  filter   range compression, F^{-1}(conj(h) F x) (``matched_filter``)
  lowp     16-bit storage, binary16 or bfloat16, with FP32 arithmetic or with
           the DFTs on the matrix cores (``fft_lowp``)
  ragged   transforms of mixed lengths packed in one buffer (``RaggedPlan``,
           ``ragged_fft``)
"""
import math

import torch

import paper_2603_27569_amd as sf
from paper_2603_27569_amd import workloads

DEVICE = "cuda"
MAX_ELEMENTS = 1 << 24  # complex values of the largest pass


def listed():
    return [
        # A handful of short lines, one call at a time: launch and call
        # latency are what the caller sees.
        {"name": "fft_256x64", "kind": "fft", "n": 256, "batch": 64, "inverse": False},
        # The paper's headline batch: one row per compute unit.
        {"name": "fft_4096x256", "kind": "fft", "n": 4096, "batch": 256, "inverse": False},
        # Back-transforming an ordinary batch whose row count is no round number.
        {"name": "ifft_1024x1000", "kind": "fft", "n": 1024, "batch": 1000, "inverse": True},
        # A block of long range lines, the longest that fit one dispatch.
        {"name": "fft_16384x1024", "kind": "fft", "n": 16384, "batch": 1024, "inverse": False},
        # Lines longer than one dispatch holds, an odd number of them.
        {"name": "fft_65536x101", "kind": "fft", "n": 65536, "batch": 101, "inverse": False},
        # The longest supported transform, a few rows: azimuth apertures and
        # spectrum analysis.
        {"name": "fft_1048576x16", "kind": "fft", "n": 1 << 20, "batch": 16, "inverse": False},
        # A spectral layer inside a training step: forward and backward.
        {"name": "grad_2048x777", "kind": "grad", "n": 2048, "batch": 777, "inverse": False},
        # The weighted spectral energy with its gradient in one call.
        {"name": "energy_4096x512", "kind": "energy", "n": 4096, "batch": 512},
        # Range compression of a block of radar lines.
        {"name": "filter_8192x300", "kind": "filter", "n": 8192, "batch": 300},
        # Half-precision storage of a large block, FP32 arithmetic.
        {"name": "f16_4096x2048", "kind": "lowp", "n": 4096, "batch": 2048, "inverse": False,
         "dtype": "float16", "mma": False},
        # bfloat16 storage with the DFTs on the matrix cores.
        {"name": "bf16_mma_2048x3000", "kind": "lowp", "n": 2048, "batch": 3000, "inverse": True,
         "dtype": "bfloat16", "mma": True},
        # One submission of 2000 lines of mixed length.
        {"name": "ragged_2000", "kind": "ragged", "count": 2000, "sizes_seed": 1005, "inverse": False},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fft", "fft", "fft", "grad", "energy", "train", "filter", "lowp", "lowp", "ragged"])
    if kind == "ragged":
        return {"kind": kind, "count": _log_uniform(rng, 16, 2000), "sizes_seed": rng.randrange(1 << 20),
                "inverse": rng.random() < 0.5}
    top = 20 if kind in ("fft", "grad") else 14
    mma = kind == "lowp" and rng.random() < 0.4
    n = 1 << rng.randint(9 if mma else 8, top)
    # two transforms of device memory in a gradient pass, one elsewhere
    most = MAX_ELEMENTS // 2 if kind in ("grad", "train") else MAX_ELEMENTS
    batch = max(1, _log_uniform(rng, max(1.0, 8192 / n), most / n))
    if batch > 2 and rng.random() < 0.7:
        batch -= 1 - batch % 2  # mostly odd row counts
    case = {"kind": kind, "n": n, "batch": batch}
    if kind in ("fft", "grad", "lowp"):
        case["inverse"] = rng.random() < 0.5
    if kind == "lowp":
        case["dtype"] = rng.choice(["float16", "bfloat16"])
        case["mma"] = mma
    return case


def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    return g


def _normal(shape, g):
    return torch.view_as_complex(torch.randn(*shape, 2, device=DEVICE, generator=g))


def _chirps(n, batch, g):
    """Linear-FM chirps of n / 4 samples at random offsets and bandwidths, in
    noise 10 dB below them (the recipe of ``workloads.chirp_noise``)."""
    length = n // 4
    x = _normal((batch, n), g) * math.sqrt(0.05)
    off = (torch.rand(batch, 1, device=DEVICE, generator=g) * (n - length + 1)).long().clamp_(max=n - length)
    beta = 0.2 + 0.6 * torch.rand(batch, 1, device=DEVICE, generator=g, dtype=torch.float64)
    m = torch.arange(length, device=DEVICE)[None, :]
    t = m.double()
    phase = torch.remainder(-0.5 * beta * t + beta / (2.0 * length) * t * t, 1.0).float() * (2 * math.pi)
    x.scatter_add_(1, off + m, torch.polar(torch.ones_like(phase), phase))
    return x


def _filter_spectrum(n, beta=0.5):
    """The stationary-phase spectrum of a chirp (``workloads.range_compression_inputs``)."""
    k = torch.arange(n, dtype=torch.float64)
    f = torch.where(k < n / 2, k, k - n) / n
    phase = math.pi * (n // 4) * f * f / beta
    band = (f.abs() < beta / 2).double()
    return torch.complex(band * torch.cos(phase), band * torch.sin(phase)).to(torch.complex64).to(DEVICE)


def _inputs(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    if kind == "ragged":
        sizes = workloads.ragged_sizes(case["count"], case["sizes_seed"])
        return {"sizes": [int(s) for s in sizes], "x": _normal((int(sizes.sum()),), g)}
    n, batch = case["n"], case["batch"]
    if kind == "lowp":
        return {"x": torch.randn(batch, n, 2, device=DEVICE, generator=g).to(getattr(torch, case["dtype"]))}
    radar = kind == "filter" or (kind == "fft" and n in (8192, 16384))
    d = {"x": _chirps(n, batch, g) if radar else _normal((batch, n), g)}
    if kind == "grad":
        d["upstream"] = _normal((batch, n), g)
    elif kind in ("energy", "train"):
        d["w"] = torch.rand(n, device=DEVICE, generator=g)
        if kind == "train":
            d["upstream"] = 0.5 + torch.rand((), device=DEVICE, generator=g)
    elif kind == "filter":
        d["h"] = _filter_spectrum(n)
    return d


def prepare(case, seed):
    state = _inputs(case, seed)
    state["case"] = case
    if case["kind"] == "ragged":
        state["plan"] = sf.RaggedPlan(state["sizes"], sf.FFT_BACKWARD if case["inverse"] else sf.FFT_FORWARD)
    elif case["kind"] in ("grad", "train"):
        state["x"].requires_grad_(True)
    return state


def run(state):
    case, x = state["case"], state["x"]
    kind = case["kind"]
    if kind == "fft":
        return sf.fft(x, inverse=case["inverse"])
    if kind == "grad":
        y = sf.FFTFunction.apply(x, case["inverse"])
        (gx,) = torch.autograd.grad(y, x, state["upstream"])
        return {"y": y.detach(), "grad": gx}
    if kind == "energy":
        total, rows, grad = sf.spectral_energy(x, state["w"])
        return {"total": total, "rows": rows, "grad": grad}
    if kind == "train":
        loss = sf.SpectralEnergyFunction.apply(x, state["w"])
        (gx,) = torch.autograd.grad(loss, x, state["upstream"])
        return {"loss": loss.detach(), "grad": gx}
    if kind == "filter":
        return sf.matched_filter(x, state["h"])
    if kind == "lowp":
        return sf.fft_lowp(x, inverse=case["inverse"], mma=case["mma"])
    return sf.ragged_fft(x, state["plan"])


def work(case):
    if case["kind"] == "ragged":
        sizes = [int(s) for s in workloads.ragged_sizes(case["count"], case["sizes_seed"])]
        return {"bytes": 16 * sum(sizes), "flops": sum(5 * s * (s.bit_length() - 1) for s in sizes)}
    n, batch, kind = case["n"], case["batch"], case["kind"]
    points = n * batch
    one = 5 * points * (n.bit_length() - 1)  # the usual 5 N log2 N of a transform
    if kind == "grad":  # x and the upstream gradient in, y and the gradient out
        return {"bytes": 32 * points, "flops": 2 * one}
    if kind == "energy":
        return {"bytes": 16 * points + 4 * (n + batch), "flops": 2 * one + 8 * points}
    if kind == "train":  # the loss comes back before its upstream gradient exists: x is read twice
        return {"bytes": 24 * points + 4 * n, "flops": 3 * one + 12 * points}
    if kind == "filter":
        return {"bytes": 16 * points + 8 * n, "flops": 2 * one + 6 * points}
    if kind == "lowp":
        return {"bytes": 8 * points, "flops": one}
    return {"bytes": 16 * points, "flops": one}


def _dft64(x, inverse):
    """The unscaled transform of the last axis in complex128."""
    return torch.fft.ifft(x, norm="forward") if inverse else torch.fft.fft(x)


def exact(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "lowp":
        x = torch.view_as_complex(d["x"].cpu().double())
        return torch.view_as_real(_dft64(x, case["inverse"]))
    x = d["x"].cpu().to(torch.complex128)
    if kind == "ragged":
        parts = torch.split(x, d["sizes"])
        return torch.cat([_dft64(p, case["inverse"]) for p in parts])
    if kind == "fft":
        return _dft64(x, case["inverse"])
    if kind == "grad":
        up = d["upstream"].cpu().to(torch.complex128)
        return {"y": _dft64(x, case["inverse"]), "grad": _dft64(up, not case["inverse"])}
    y = _dft64(x, False)
    if kind == "filter":
        return torch.fft.ifft(torch.conj(d["h"].cpu().to(torch.complex128)) * y)
    w2 = d["w"].cpu().double() ** 2
    rows = (w2 * (y.real ** 2 + y.imag ** 2)).sum(-1)
    grad = _dft64(2.0 * w2 * y, True)
    if kind == "energy":
        return {"total": rows.sum().reshape(1), "rows": rows, "grad": grad}
    return {"loss": rows.sum(), "grad": grad * float(d["upstream"])}
