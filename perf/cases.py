"""The framework's measured work: single calls of its public entry points.

Each case is one call (or the two or three calls that a program makes together)
of ``Plan``, ``PencilPlan``, ``SlabPlan`` or ``BatchPlan`` on tensors that are on
the GPU already, with the plan and the output tensors that a program keeps from
call to call.  ``listed`` gives the fixed cases, ``draw`` more of the same
ranges, ``prepare`` / ``run`` one of them, ``work`` its unavoidable bytes and
operations, and ``exact`` its result in 64 bits from torch.
"""
import math

import torch

from paper_1506_07933_amd import BatchPlan, PencilPlan, Plan, SlabPlan
from paper_1506_07933_amd import synth

DEV = "cuda:0"
_C = {"fp32": torch.complex64, "fp64": torch.complex128}
_R = {"fp32": torch.float32, "fp64": torch.float64}
_OPS = ("poisson", "laplacian", "helmholtz", "dx", "dy", "dz")
_ALPHA = 1.5


def listed():
    return [
        # the smallest grid in use: a forward and the inverse that follows it,
        # where launches and their latency are what counts
        {"name": "c2c_32_fp64_pair", "op": "pair", "shape": "32x32x32", "prec": "fp64"},
        # the smallest grid of the served Poisson solves
        {"name": "poisson_64_fp32", "op": "poisson", "shape": "64x64x64", "prec": "fp32"},
        # an ordinary grid whose axes are all different and none a power of two
        {"name": "c2c_100x120x144_fp32", "op": "forward", "shape": "100x120x144", "prec": "fp32"},
        # real fields of ordinary size, each direction, each precision
        {"name": "r2c_256_fp32", "op": "r2c", "shape": "256x256x256", "prec": "fp32"},
        {"name": "c2r_256_fp64", "op": "c2r", "shape": "256x256x256", "prec": "fp64"},
        # three derivatives of a real field
        {"name": "gradient_256_fp64", "op": "gradient", "shape": "256x256x256", "prec": "fp64"},
        # the headline transform
        {"name": "c2c_512_fp32", "op": "forward", "shape": "512x512x512", "prec": "fp32"},
        # the largest grid of the served Poisson solves
        {"name": "poisson_512_fp32", "op": "poisson", "shape": "512x512x512", "prec": "fp32"},
        # 64 transforms of uneven sizes at once
        {"name": "batch_64_uneven_fp32", "op": "batch", "shape": "64x0", "prec": "fp32", "mode": "persistent"},
        # one rank's share of a 1024^3 grid on 4 x 4 ranks: z, pack, unpack, y
        {"name": "pencil_1024_4x4_fp32", "op": "pencil", "shape": "1024x1024x1024", "prec": "fp32", "p0": 4, "p1": 4},
        # one task's share of a 512^3 grid over 4 tasks, forward
        {"name": "slab_512_p4_fp32", "op": "slab_forward", "shape": "512x512x512", "prec": "fp32", "p": 4, "kind": "c2c"},
        # the largest array: four axes, 8 GiB
        {"name": "c2c_512x256x128x64_fp32", "op": "forward", "shape": "512x256x128x64", "prec": "fp32"},
    ]


# ------------------------------------------------------------------ draws

def _smooth(n):
    for p in (2, 3, 5):
        while n % p == 0:
            n //= p
    return n == 1


_ANY = [n for n in range(2, 1025) if _smooth(n)]
# lengths that programs choose most: 2^k and 3 2^k
_COMMON = [n for n in _ANY if n >= 8 and (n & (n - 1) == 0 or (n % 3 == 0 and (n // 3) & (n // 3 - 1) == 0))]


def _length(rng, want, lo, hi, even=False, div=1):
    menu = [n for n in (_COMMON if rng.random() < 0.5 else _ANY) if lo <= n <= hi and not (even and n % 2)]
    menu = [n for n in menu if n % div == 0] or [n for n in _ANY if lo <= n <= hi and n % div == 0 and not (even and n % 2)]
    return min(menu, key=lambda n: abs(math.log(n / want)))


def _grid(rng, log2_lo, log2_hi, even=False):
    """Three axis lengths whose product is spread over the logarithm."""
    v = rng.uniform(log2_lo, log2_hi)
    a, b = rng.uniform(-0.6, 0.6), rng.uniform(-0.6, 0.6)
    w = [2 ** (v / 3 + e) for e in (a, b, -a - b)]
    return [_length(rng, x, 8, 1024, even and i == 2) for i, x in enumerate(w)]


def draw(rng):
    prec = "fp32" if rng.random() < 0.65 else "fp64"
    top = 27 if prec == "fp32" else 26
    op = rng.choice(["forward", "inverse", "forward", "r2c", "c2r", "r2c", "c2r", "spectral", "spectral", "gradient",
                     "divergence", "batch", "pencil", "slab_forward", "slab_inverse", "nd"])
    if op == "batch":
        return {"op": "batch", "shape": "%dx%d" % (rng.randrange(8, 97), rng.randrange(1, 1000)), "prec": prec,
                "mode": rng.choice(["persistent", "grouped"])}
    if op == "pencil":
        p0, p1 = rng.choice([2, 4]), rng.choice([2, 4, 5])
        n0, n1, n2 = (_length(rng, 2 ** rng.uniform(6, 10), 32, 1024, div=p) for p in (p0, p1, p1))
        return {"op": op, "shape": "%dx%dx%d" % (n0, n1, n2), "prec": prec, "p0": p0, "p1": p1}
    if op.startswith("slab"):
        p, kind = rng.choice([2, 3, 4, 8]), rng.choice(["c2c", "r2c"])
        n0, n1 = (_length(rng, 2 ** rng.uniform(5.5, 9), 32, 512, div=p) for _ in range(2))
        n2 = _length(rng, 2 ** rng.uniform(5.5, 9), 32, 512, even=True)
        return {"op": op, "shape": "%dx%dx%d" % (n0, n1, n2), "prec": prec, "p": p, "kind": kind}
    if op == "nd":
        v = rng.uniform(16, top - 1) / 4
        dims = [_length(rng, 2 ** (v + rng.uniform(-0.7, 0.7)), 4, 256) for _ in range(4)]
        return {"op": rng.choice(["forward", "inverse"]), "shape": "x".join(map(str, dims)), "prec": prec}
    if op == "spectral":
        op = rng.choice(_OPS)
    real = op not in ("forward", "inverse")
    shape = "%dx%dx%d" % tuple(_grid(rng, 15, top - (1 if op in ("gradient", "divergence") else 0), even=real))
    return {"op": op, "shape": shape, "prec": prec}


# ---------------------------------------------------------- inputs, plans

def _dims(case):
    return tuple(int(v) for v in case["shape"].split("x"))


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _real(shape, prec, g):
    return torch.randn(shape, dtype=_R[prec], device=DEV, generator=g)


def _complex(shape, prec, g):
    """re, im ~ U[-1, 1)."""
    x = torch.rand(tuple(shape) + (2,), dtype=_R[prec], device=DEV, generator=g)
    return torch.view_as_complex(x.mul_(2).sub_(1))


def _half(shape):
    return tuple(shape[:-1]) + (shape[-1] // 2 + 1,)


def _batch_shapes(case):
    import numpy as np
    count, pick = _dims(case)
    idx = np.random.default_rng(pick).choice(len(synth.UNEVEN_SHAPES), size=count)
    return [tuple(synth.UNEVEN_SHAPES[i]) for i in idx]


def _slab_shapes(case):
    n0, n1, n2 = _dims(case)
    p = case["p"]
    nc = n2 // 2 + 1 if case["kind"] == "r2c" else n2
    return {"slab": (n0 // p, n1, n2), "mid": (n0 // p, n1, nc), "share": (n0, n1 // p, nc),
            "send": (p, n0 // p, n1 // p, nc)}


def _inputs(case, seed):
    op, prec, d, g = case["op"], case["prec"], _dims(case), _gen(seed)
    if op in ("pair", "forward", "inverse"):
        return [_complex(d, prec, g)]
    if op == "c2r":  # an evolved spectrum
        return [torch.view_as_complex(torch.randn(_half(d) + (2,), dtype=_R[prec], device=DEV, generator=g))]
    if op == "divergence":
        return [_real(d, prec, g) for _ in range(3)]
    if op == "batch":
        return [_complex(s, prec, g) for s in _batch_shapes(case)]
    if op == "pencil":
        return [_complex((d[0] // case["p0"], d[1] // case["p1"], d[2]), prec, g)]
    if op == "slab_forward":
        s = _slab_shapes(case)["slab"]
        return [_real(s, prec, g) if case["kind"] == "r2c" else _complex(s, prec, g)]
    if op == "slab_inverse":  # the share, and the blocks received after the exchange
        s = _slab_shapes(case)
        return [_complex(s["share"], prec, g), _complex(s["send"], prec, g)]
    return [_real(d, prec, g)]  # r2c, gradient, the operators


def prepare(case, seed):
    op, prec, d = case["op"], case["prec"], _dims(case)
    x = _inputs(case, seed)
    c, r = _C[prec], _R[prec]
    new = lambda shape, dt: torch.empty(shape, dtype=dt, device=DEV)  # noqa: E731
    if op in ("pair", "forward", "inverse"):
        out = [new(d, c) for _ in range(2 if op == "pair" else 1)]
        return {"case": case, "plan": Plan(d, "c2c", prec), "x": x, "out": out}
    if op == "batch":
        plan = BatchPlan(_batch_shapes(case), prec, mode=case["mode"])
        return {"case": case, "plan": plan, "x": x, "out": [torch.empty_like(t) for t in x]}
    if op == "pencil":
        plan = PencilPlan(d, (case["p0"], case["p1"]), prec)
        return {"case": case, "plan": plan, "x": x, "out": [new(plan.send_shape, c), new(plan.out_shape, c)]}
    if op.startswith("slab"):
        plan, s = SlabPlan(d, case["p"], case["kind"], prec), _slab_shapes(case)
        if op == "slab_forward":
            out = [new(s["send"], c), new(s["share"], c), new(s["mid"], c)]
        else:
            out = [new(s["send"], c), new(s["slab"], r if case["kind"] == "r2c" else c), new(s["send"], c)]
        return {"case": case, "plan": plan, "x": x, "out": out}
    plan = Plan(d, "r2c", prec)
    if op == "r2c":
        out = [new(_half(d), c)]
    else:
        out = [new(d, r) for _ in range(3 if op == "gradient" else 1)]
    return {"case": case, "plan": plan, "x": x, "out": out}


def run(state):
    case, p, x, out = state["case"], state["plan"], state["x"], state["out"]
    op = case["op"]
    if op in ("forward", "r2c"):
        return p.forward(x[0], out=out[0])
    if op in ("inverse", "c2r"):
        return p.inverse(x[0], out=out[0])
    if op == "pair":
        p.forward(x[0], out=out[0])
        p.inverse(out[0], out=out[1])
        return out
    if op == "poisson":
        return p.poisson(x[0], out=out[0])
    if op == "gradient":
        return p.gradient(x[0], outs=out)
    if op == "divergence":
        return p.divergence(x, out=out[0])
    if op == "batch":
        return p.forward(x, outs=out)
    if op == "pencil":
        p.forward_share(x[0], out[0], out[1])
        return out
    if op == "slab_forward":  # the send buffer stands in for the receive buffer
        p.forward_local(x[0], out[0], out[2])
        p.forward_x(out[0], out[1])
        return out[:2]
    if op == "slab_inverse":
        p.inverse_x(x[0], out[0])
        p.inverse_local(x[1], out[2], out[1])
        return out[:2]
    return p.spectral(_OPS.index(op), x[0], out=out[0], alpha=_ALPHA)


# ------------------------------------------------------------------- work

def _c2c_flops(dims):
    n = math.prod(dims)
    return 5.0 * n * math.log2(max(2, n))


def work(case):
    op, d = case["op"], _dims(case)
    r = 4 if case["prec"] == "fp32" else 8
    c = 2 * r
    n = math.prod(d)
    if op == "pair":
        return {"bytes": 4 * c * n, "flops": 2 * _c2c_flops(d)}
    if op in ("forward", "inverse"):
        return {"bytes": 2 * c * n, "flops": _c2c_flops(d)}
    if op in ("r2c", "c2r"):
        return {"bytes": r * n + c * math.prod(_half(d)), "flops": _c2c_flops(d) / 2}
    if op in ("gradient", "divergence"):
        return {"bytes": 4 * r * n, "flops": 4 * _c2c_flops(d) / 2}
    if op == "batch":
        shapes = _batch_shapes(case)
        return {"bytes": sum(2 * c * math.prod(s) for s in shapes), "flops": sum(_c2c_flops(s) for s in shapes)}
    if op == "pencil":  # z of the share, its blocks written; the blocks read, y
        m = n // (case["p0"] * case["p1"])
        return {"bytes": 4 * c * m, "flops": 5.0 * m * math.log2(d[1] * d[2])}
    if op.startswith("slab"):
        s = _slab_shapes(case)
        m, e = math.prod(s["send"]), (r if case["kind"] == "r2c" else c)
        return {"bytes": 3 * c * m + e * math.prod(s["slab"]), "flops": _c2c_flops(d) / case["p"] * e / c}
    return {"bytes": 2 * r * n, "flops": 2 * _c2c_flops(d) / 2}


# ------------------------------------------------------------------ exact

def _wave(n, half=False):
    k = torch.arange(n // 2 + 1 if half else n, device=DEV)
    return k if half else torch.where(2 * k < n, k, k - n)


def _k(d, j):
    """The wavenumbers along axis j, with the Nyquist mode of an even axis set to 0."""
    k = _wave(d[j], half=j == 2).to(torch.float64)
    if d[j] % 2 == 0:
        k[d[j] // 2] = 0
    return k.reshape([-1 if i == j else 1 for i in range(3)])


def _fft(x, sign, axes):
    """Unscaled transform, one axis after the other."""
    for a in axes:
        x = torch.fft.fft(x, dim=a) if sign < 0 else torch.fft.ifft(x, dim=a, norm="forward")
    return x


def _c2r(y, n):
    """Unscaled z-inverse of a half line; the imaginary parts of its ends do not count."""
    y = y.clone()
    y.imag[..., 0] = 0
    y.imag[..., -1] = 0
    full = torch.cat([y, y[..., 1:-1].flip(-1).conj()], dim=-1)
    return _fft(full, +1, (-1,)).real.contiguous()


def _operator(op, d):
    kk = sum(_wave(n, half=j == 2).to(torch.float64).reshape([-1 if i == j else 1 for i in range(3)]) ** 2
             for j, n in enumerate(d))
    if op == "laplacian":
        return -kk
    if op == "poisson":
        return torch.where(kk > 0, -1.0 / torch.where(kk > 0, kk, torch.ones_like(kk)), torch.zeros_like(kk))
    return 1.0 / (_ALPHA + kk)


def exact(case, seed):
    op, d = case["op"], _dims(case)
    x = [t.to(torch.complex128 if t.is_complex() else torch.float64) for t in _inputs(case, seed)]
    if math.prod(d) > 1 << 28 and op != "pencil":
        return None  # a 16 GiB array in 64 bits
    if op == "pair":
        y = _fft(x[0], -1, (2, 1, 0))
        return [y, x[0] * math.prod(d)]
    if op in ("forward", "inverse"):
        return _fft(x[0], -1 if op == "forward" else +1, range(len(d) - 1, -1, -1))
    if op == "batch":
        return [_fft(t, -1, (2, 1, 0)) for t in x]
    if op == "pencil":
        n0l, n1l, m = d[0] // case["p0"], d[1] // case["p1"], d[2] // case["p1"]
        send = _fft(x[0], -1, (2,)).reshape(n0l, n1l, case["p1"], m).permute(2, 0, 1, 3).contiguous()
        return [send, _fft(send.permute(1, 0, 2, 3).reshape(n0l, d[1], m), -1, (1,))]
    if op == "slab_forward":
        s, p = _slab_shapes(case), case["p"]
        y = _fft(x[0].to(torch.complex128), -1, (2,))[..., : s["mid"][2]]
        y = _fft(y, -1, (1,)).reshape(d[0] // p, p, d[1] // p, -1).permute(1, 0, 2, 3).contiguous()
        return [y, _fft(y.reshape(s["share"]), -1, (0,))]
    if op == "slab_inverse":
        s, p = _slab_shapes(case), case["p"]
        send = _fft(x[0], +1, (0,)).reshape(s["send"])
        y = _fft(x[1].permute(1, 0, 2, 3).reshape(s["mid"]), +1, (1,))
        return [send, _c2r(y, d[2]) if case["kind"] == "r2c" else _fft(y, +1, (2,))]
    if op == "c2r":
        return _c2r(_fft(x[0], +1, (0, 1)), d[2])
    h = [_fft(_fft(t.to(torch.complex128), -1, (2,))[..., : d[2] // 2 + 1], -1, (1, 0)) for t in x]
    if op == "r2c":
        return h[0]
    back = lambda y: _c2r(_fft(y, +1, (0, 1)), d[2]) / math.prod(d)  # noqa: E731
    if op == "gradient":
        return [back(1j * _k(d, j) * h[0]) for j in range(3)]
    if op == "divergence":
        return back(sum(1j * _k(d, j) * h[j] for j in range(3)))
    if op in ("dx", "dy", "dz"):
        return back(1j * _k(d, ("dx", "dy", "dz").index(op)) * h[0])
    return back(_operator(op, d) * h[0])
