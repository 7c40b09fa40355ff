"""Timed cases: the work that programs using this library have it do.

listed() names the cases, draw() makes more of the same ranges, prepare()
builds what a program holds before the call (plans, signals), run() is one
pass through the public entry points, exact() the same results in 64 bits by
full-length FFTs, work() the bytes and operations a pass cannot do without.
Sizes are those of workloads.py, the tests and the benchmark, or generic.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_1910_01972_amd.ols as ols

STENCILS = {
    "difference": ols.DIFFERENCE_STENCIL,
    "midpoint": ols.MIDPOINT_CUBIC_STENCIL,
}

# Largest number of output samples of a case (2^23 samples, 32 filters).
MAX_OUTPUTS = 1 << 28


def _case(kind, name=None, **kw):
    c = {"kind": kind}
    if name:
        c["name"] = name
    c.update(kw)
    return c


def _forward(name, Ns, K, M, N=0, real=False, derivative=False, power=False, stencil=""):
    return _case("forward", name, Ns=Ns, K=K, M=M, N=N, real=real, derivative=derivative, power=power,
                 stencil=stencil)


def listed():
    return [
        # one short block of a stream through a small bank: latency and launches
        _forward("short_block", 8192, 4, 64),
        # matched filtering of one signal with one template (single_filter_2p20)
        _forward("single_filter_2p20", 1 << 20, 1, 64, N=1024),
        # an ordinary signal of no particular length, rows off every alignment grid
        _forward("ragged_signal", 1000003, 7, 100),
        # the benchmark: a long signal through a filter bank (filter_bank_2p23_k32_m256)
        _forward("filter_bank_2p23", 1 << 23, 32, 256, N=2048),
        # filters that fill much of the longest transforms (M = 2048 of the sweep)
        _forward("long_filters", 1 << 24, 8, 2048),
        # a search that keeps only the power of each output
        _forward("power_bank", 1 << 23, 32, 256, N=2048, power=True),
        # real data, real filters (filter_bank_real_2p23_k32_m256)
        _forward("real_bank", 1 << 23, 32, 256, N=2048, real=True),
        # the non-local stage: difference of neighbouring outputs
        _forward("stage_difference", 1 << 23, 32, 256, N=2048, stencil="difference"),
        # one training step of learnable filters (grad_2p22_k16_m512): new
        # filter values, forward, gradients of the signal and the filters
        _case("train", "train_2p22", Ns=1 << 22, K=16, M=512, N=4096),
        # the adjoint alone on a short signal: launches and reductions
        _case("backward", "backward_short", Ns=50000, K=4, M=64, N=1024),
        # many signals of uneven length, each with its own filters, planned once
        _case("batch", "batch_uneven", n=64, items_seed=4, min_log2=14.0, max_log2=22.0, max_k=16),
        # the single-call batched path: items and filters read anew on every call
        _case("batched", "batched_call", n=24, items_seed=11, min_log2=10.0, max_log2=16.0, max_k=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(2.0 ** rng.uniform(math.log2(lo), math.log2(hi))))


def _length(rng, lo, hi):
    """A length in [lo, hi]: as drawn (odd ones among them), on a 16-sample grid, or a power of two."""
    n = _log_int(rng, lo, hi)
    form = rng.choice(("any", "any", "odd", "grid", "pow2"))
    if form == "odd":
        n |= 1
    elif form == "grid":
        n = n // 16 * 16
    elif form == "pow2":
        n = 1 << int(math.log2(n))
    return max(lo, min(hi, n))


def _fft_length(rng, M, lo=256):
    """0 (the library's choice), mostly, or a power of two that keeps at least half of each segment."""
    lengths = [n for n in (256, 512, 1024, 2048, 4096, 8192) if n >= 2 * M and n >= lo]
    if not lengths or rng.random() < 0.6:
        return 0
    return rng.choice(lengths)


def draw(rng):
    kind = rng.choice(("forward",) * 5 + ("train", "backward", "batch", "batched"))
    if kind == "batch":
        return _case("batch", n=rng.randint(4, 64), items_seed=rng.randrange(1 << 20), min_log2=14.0,
                     max_log2=rng.uniform(17.0, 22.0), max_k=rng.randint(2, 16))
    if kind == "batched":
        return _case("batched", n=rng.randint(2, 64), items_seed=rng.randrange(1 << 20), min_log2=10.0,
                     max_log2=rng.uniform(13.0, 18.0), max_k=rng.randint(2, 16))
    if kind == "train":
        K, M = _log_int(rng, 1, 32), _log_int(rng, 16, 1024)
        return _case("train", Ns=_length(rng, 1 << 14, min(1 << 22, (1 << 26) // K)), K=K, M=M,
                     N=_fft_length(rng, M))
    if kind == "backward":
        K, M = _log_int(rng, 1, 16), _log_int(rng, 16, 1024)
        return _case("backward", Ns=_length(rng, 1 << 12, min(1 << 22, (1 << 26) // K)), K=K, M=M,
                     N=_fft_length(rng, M))
    form = rng.choice(("plain",) * 4 + ("power", "real", "derivative", "stencil"))
    K, M = _log_int(rng, 1, 64), _log_int(rng, 8, 2048)
    stencil = rng.choice(sorted(STENCILS)) if form == "stencil" else ""
    J = len(STENCILS[stencil][0]) if stencil else 1
    return _forward(None, _length(rng, 1 << 12, min(1 << 25, MAX_OUTPUTS // (K * J))), K, M,
                    N=_fft_length(rng, M + 8), real=form == "real", derivative=form == "derivative",
                    power=form == "power" or (form == "stencil" and rng.random() < 0.3), stencil=stencil)


# ---------------------------------------------------------------------------
# Inputs: signals i.i.d. uniform[-1, 1], filters i.i.d. N(0, 1) / sqrt(M),
# upstream gradients i.i.d. N(0, 1), as in workloads.py.
# ---------------------------------------------------------------------------
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _signal(g, Ns, real=False):
    s = torch.empty(Ns if real else 2 * Ns, dtype=torch.float32, device="cuda").uniform_(-1.0, 1.0, generator=g)
    return s if real else torch.view_as_complex(s.view(Ns, 2))


def _normal(g, rows, cols, scale, real=False):
    h = torch.empty(rows * cols * (1 if real else 2), dtype=torch.float32, device="cuda")
    h = h.normal_(0.0, 1.0, generator=g) * scale
    return h.view(rows, cols) if real else torch.view_as_complex(h.view(rows, cols, 2))


def _batch_shapes(case):
    """(N_s, K, M) of every signal, lengths log-uniform, M of 16 .. 1024 taps."""
    r = np.random.default_rng(case["items_seed"])
    out = []
    for _ in range(case["n"]):
        Ns = int(round(2.0 ** r.uniform(case["min_log2"], case["max_log2"])))
        K = int(r.integers(1, case["max_k"] + 1))
        M = int(round(2.0 ** r.uniform(4.0, 10.0)))
        out.append((Ns, K, M))
    return out


def _inputs(case, seed):
    g = _generator(seed)
    if case["kind"] in ("batch", "batched"):
        return [(_signal(g, Ns), _normal(g, K, M, 1.0 / math.sqrt(M))) for Ns, K, M in _batch_shapes(case)]
    real = bool(case.get("real", False))
    s = _signal(g, case["Ns"], real)
    h = _normal(g, case["K"], case["M"], 1.0 / math.sqrt(case["M"]), real)
    if case["kind"] in ("train", "backward"):
        return s, h, _normal(g, case["K"], case["Ns"], 1.0)
    return s, h


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return {"kind": kind, "batch": ols.OLSBatch(_inputs(case, seed))}
    if kind == "batched":
        return {"kind": kind, "batch": ols.OLSBatched(_inputs(case, seed))}
    if kind == "forward":
        s, h = _inputs(case, seed)
        plan = ols.OLSPlan(h, N=case["N"], derivative=case["derivative"], power=case["power"],
                           stencil=STENCILS[case["stencil"]] if case["stencil"] else None)
        return {"kind": kind, "plan": plan, "s": s}
    s, h, gy = _inputs(case, seed)
    if kind == "backward":
        return {"kind": kind, "plan": ols.OLSPlan(h, N=case["N"]), "s": s, "gy": gy}
    return {"kind": kind, "conv": ols.OLSConv(h, N=case["N"]), "h": h, "s": s.requires_grad_(), "gy": gy}


def run(state):
    kind = state["kind"]
    if kind == "forward":
        return state["plan"].forward(state["s"])
    if kind == "backward":
        return state["plan"].backward(state["s"], state["gy"])
    if kind == "train":
        conv, s = state["conv"], state["s"]
        with torch.no_grad():
            conv.h.copy_(state["h"])  # the optimizer's write of this step's filters
        y = conv(s)
        ds, dh = torch.autograd.grad(y, (s, conv.h), state["gy"])
        return y.detach(), ds, dh
    return state["batch"].run()


# ---------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------
def _conv64(s, h, outputs):
    """Rows of the full linear convolution, samples 0 .. outputs - 1, float64."""
    L = 1 << max(1, (s.numel() + h.shape[1] - 1).bit_length())
    rdt = not s.is_complex()
    S = torch.fft.fft(s.to(torch.complex128), L)
    out = torch.empty((h.shape[0], outputs), dtype=torch.float64 if rdt else torch.complex128, device=s.device)
    for r in range(h.shape[0]):
        y = torch.fft.ifft(S * torch.fft.fft(h[r].to(torch.complex128), L))[:outputs]
        out[r] = y.real if rdt else y
    return out


def _adjoint64(s, h, gy):
    Ns, M = s.numel(), h.shape[1]
    L = 1 << (Ns + M - 1).bit_length()
    S = torch.fft.fft(s.to(torch.complex128), L).conj()
    E = torch.zeros(L, dtype=torch.complex128, device=s.device)
    dh = torch.empty(h.shape, dtype=torch.complex128, device=s.device)
    for r in range(h.shape[0]):
        G = torch.fft.fft(gy[r].to(torch.complex128), L)
        E += G * torch.fft.fft(h[r].to(torch.complex128), L).conj()
        dh[r] = torch.fft.ifft(S * G)[:M]
    return torch.fft.ifft(E)[:Ns], dh


def _forward64(case, s, h):
    Ns = s.numel()
    w, left = STENCILS[case["stencil"]] if case["stencil"] else ([[1.0]], 0)
    T = len(w[0])
    right = T - 1 - left
    y = _conv64(s, h, Ns + right)
    if case["derivative"]:
        y[:, 1:] -= y[:, :-1].clone()
    if case["stencil"]:
        y = torch.cat((torch.zeros((y.shape[0], left), dtype=y.dtype, device=y.device), y), dim=1)
        z = torch.zeros((y.shape[0], Ns, len(w)), dtype=y.dtype, device=y.device)
        for j, row in enumerate(w):
            for d, wd in enumerate(row):
                if wd != 0.0:
                    z[:, :, j] += wd * y[:, d:d + Ns]
        y = z.reshape(y.shape[0], Ns * len(w))
    if case["power"]:
        y = y * y if not y.is_complex() else y.real * y.real + y.imag * y.imag
    return y


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch", "batched"):
        return [_conv64(s, h, s.numel()) for s, h in _inputs(case, seed)]
    if kind == "forward":
        return _forward64(case, *_inputs(case, seed))
    s, h, gy = _inputs(case, seed)
    ds, dh = _adjoint64(s, h, gy)
    if kind == "backward":
        return ds, dh
    return _conv64(s, h, s.numel()), ds, dh


# ---------------------------------------------------------------------------
# Bytes and operations of one pass
# ---------------------------------------------------------------------------
def _segment(case, M):
    """(N, H): the case's FFT length, or a power of two of about four filter lengths."""
    N = case.get("N", 0) or min(8192, max(1024, 1 << (4 * M - 1).bit_length()))
    return N, max(1, N - M + 1)


def _transform_flops(Ns, M, N, H, transforms, products):
    segments = -(-Ns // H)
    return segments * N * (transforms * 5 * math.log2(N) + products * 6)


def work(case):
    kind = case["kind"]
    if kind in ("batch", "batched"):
        b = f = 0.0
        for Ns, K, M in _batch_shapes(case):
            N, H = _segment({}, M)
            b += 8 * (K + 1) * Ns + 8 * K * M
            f += _transform_flops(Ns, M, N, H, K + 1, K)
        return {"bytes": b, "flops": f}
    Ns, K, M = case["Ns"], case["K"], case["M"]
    N, H = _segment(case, M)
    if kind == "forward":
        J = len(STENCILS[case["stencil"]][0]) if case["stencil"] else 1
        el_in = 4 if case["real"] else 8
        el_out = 4 if case["real"] or case["power"] else 8
        f = _transform_flops(Ns, M, N, H, K + 1, K) * (0.5 if case["real"] else 1.0)
        return {"bytes": el_in * (Ns + K * M) + el_out * J * K * Ns, "flops": f}
    # adjoint: gradient and signal in, ds and dh out; every gradient window
    # transformed once, one transform back per segment and per filter
    b = 8 * K * Ns + 16 * Ns + 16 * K * M
    f = _transform_flops(Ns, M, N, H, K + 2, 2 * K)
    if kind == "train":
        b += 8 * (K + 1) * Ns + 8 * K * M
        f += _transform_flops(Ns, M, N, H, K + 1, K)
    return {"bytes": b, "flops": f}
