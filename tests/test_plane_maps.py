"""The plane and split schedules on the CPU (MIFFT_PLAN_ONLY): the index maps
of their passes, followed with a library FFT per line, compose to the 3-D DFT
for every split, with and without the workspace, in both directions and for
real data; every plan over a range of shapes keeps its passes inside its
buffers (the library checks each at plan time)."""
import ctypes

import numpy as np
import pytest

from paper_1506_07933_amd._lib import MIFFT_PLAN_ONLY, lib
from paper_1506_07933_amd.fft import plan_describe, plan_destroy


def _lists(shape, kind, prec):
    h = ctypes.c_void_p()
    assert lib.mifft_plan_create(ctypes.byref(h), *shape, kind, prec, MIFFT_PLAN_ONLY) == 0, lib.mifft_last_error()
    text = plan_describe(h.value)
    ws = lib.mifft_workspace_bytes(h.value)
    plan_destroy(h.value)
    out = {}
    for line in text.splitlines():
        d = dict(kv.split("=") for kv in line.split()[1:])
        for k, v in d.items():
            if "/" in v:
                d[k] = tuple(int(x) for x in v.split("/"))
            elif v.lstrip("-").isdigit():
                d[k] = int(v)
        out.setdefault(line.split()[0], []).append(d)
    return out, ws // (16 if prec else 8)


def _dft(x, sgn, axis):
    return np.fft.fft(x, axis=axis) if sgn > 0 else np.fft.ifft(x, axis=axis) * x.shape[axis]


def _plane(p, src, dst, n1):
    """Rows (x, b, r) of L points (pairs of reals on a real side)."""
    A, nb, L, kind = p["rows"], p["nb"], p["L"], p["kind"]
    c_in, c_out = L + (kind == "plane_c2r"), L + (kind == "plane_r2c")
    sgn = -1 if kind == "plane_c2r" else (1 if kind == "plane_r2c" else p["sgn"])
    for t in range(p["tiles"]):
        x, b = divmod(t, nb)
        rows = [src[x * p["is"][0] + b * p["sb"][0] + r * p["is"][1]:][:c_in] for r in range(A)]
        v = np.array(rows)
        if kind == "plane_r2c":
            v = np.fft.rfft(np.stack([v.real, v.imag], -1).reshape(A, 2 * L), axis=1)
        elif kind == "plane":
            v = _dft(v, sgn, 1)
        v = _dft(v, sgn, 0)
        if kind == "plane_c2r":
            v = np.fft.irfft(v, 2 * L, axis=1) * (2 * L)
            v = v[:, 0::2] + 1j * v[:, 1::2]
        if p["tw"]:
            v = v * np.exp(-2j * np.pi * sgn * b * np.arange(A) / n1)[:, None]
        for k in range(A):
            o = x * p["os"][0] + b * p["sb"][1] + k * p["os"][1]
            dst[o:o + c_out] = v[k]


def _cols(p, src, dst, n1):
    L, B = p["rows"], p["nb"]
    out = []
    for g in range(p["groups"]):
        at = lambda i: [[g * p["gs"][i] + x * p["es"][i] + y * p["ys"][i] for y in range(B)] for x in range(L)]  # noqa: E731
        idx = np.array(at(0))[:, :, None] + np.arange(p["cols"])
        v = _dft(_dft(src[idx], p["sgn"], 1), p["sgn"], 0)
        if p["tw"]:
            v = v * np.exp(-2j * np.pi * p["sgn"] * np.arange(B) * g / n1)[None, :, None]
        out.append((np.array(at(1))[:, :, None] + np.arange(p["cols"]), v))
    for idx, v in out:
        dst[idx] = v


def _strided(p, src, dst):
    for g in range(p["groups"]):
        idx = lambda i: g * p["gs"][i] + np.arange(p["L"])[:, None] * p["es"][i] + np.arange(p["cols"])  # noqa: E731
        dst[idx(1)] = _dft(src[idx(0)], p["sgn"], 0)


def _run(passes, bufs, order, n1):
    for p, (s, d) in zip(passes, order):
        if p["kind"] == "cols":
            _cols(p, bufs[s], bufs[d], n1)
        elif p["kind"] == "strided":
            _strided(p, bufs[s], bufs[d])
        else:
            _plane(p, bufs[s], bufs[d], n1)


SPLITS = [("2,16", (6, 8, 12)), ("3,16", (5, 12, 16)), ("4,8", (4, 8, 20)), ("5,8", (3, 20, 10)), ("6,16", (9, 24, 8)),
          ("8,8", (5, 32, 6)), ("4,8", (3, 256, 128)), ("8,4", (2, 512, 64))]


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("split,shape", SPLITS)
def test_split_maps_compose_to_the_3d_dft(monkeypatch, split, shape, kind):
    monkeypatch.setenv("MIFFT_SPLIT", split)
    n0, n1, n2 = shape
    nc = n2 // 2 + 1 if kind else n2
    lists, ws = _lists(shape, kind, 1)
    fwd, inv = lists.get("plane_forward"), lists.get("plane_inverse")
    assert fwd and inv
    rng = np.random.default_rng(3)
    size = max(n0 * n1 * n2, n0 * n1 * nc)
    via = "ws" if fwd[0]["os"][1] > nc else "out"  # ka n0 B rows apart in the workspace, adjacent in the output
    x = rng.standard_normal(shape) if kind else rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    flat = (x.reshape(-1, 2) @ [1, 1j]) if kind else x.reshape(-1)
    bufs = {"in": flat.astype(complex), "out": np.zeros(size, complex), "ws": np.zeros(max(ws, size), complex)}
    order = [("in", via), (via, "out")]
    _run(fwd, bufs, order, n1)
    ref = np.fft.rfftn(x) if kind else np.fft.fftn(x)
    got = bufs["out"][:n0 * n1 * nc].reshape(n0, n1, nc)
    assert np.linalg.norm(got - ref) <= 1e-12 * np.linalg.norm(ref)
    bufs = {"in": ref.reshape(-1).copy(), "out": np.zeros(size, complex), "ws": np.zeros(max(ws, size), complex)}
    _run(inv, bufs, [("in", "ws"), ("ws", "out")] if kind else order, n1)
    got = bufs["out"][:n0 * n1 * n2 // (2 if kind else 1)]
    want = flat * (n0 * n1 * n2)
    assert np.linalg.norm(got - want) <= 1e-12 * np.linalg.norm(want)


def test_every_plan_stays_inside_its_buffers():
    """Lengths of every kind on each axis (the library rejects a pass that
    reaches past a buffer)."""
    lens = (2, 3, 8, 15, 25, 48, 64, 90, 100, 125, 128, 162, 200, 243, 256, 300, 384, 500, 512, 1000, 1024)
    for i, n1 in enumerate(lens):
        for j, n2 in enumerate(lens):
            n0 = lens[(3 * i + 5 * j) % len(lens)]
            for kind in (0, 1):
                if kind and n2 % 2:
                    continue
                for prec in (0, 1):
                    _lists((n0, n1, n2), kind, prec)


def test_switches_keep_the_one_axis_passes(monkeypatch):
    for env in ("MIFFT_CHUNK_MIB", "MIFFT_BLOCKED", "MIFFT_PLANES"):
        monkeypatch.setenv(env, "0")
        lists, _ = _lists((64, 64, 64), 1, 0)
        assert not [k for k in lists if k.startswith("plane_")]
        monkeypatch.delenv(env)
    lists, _ = _lists((64, 64, 64), 1, 0)
    assert [p["kind"] for p in lists["plane_forward"]] == ["plane_r2c", "strided"]
    assert [p["kind"] for p in lists["plane_poisson"]] == ["plane_r2c", "poisson_x", "plane_c2r"]


@pytest.mark.parametrize("split,shape", [("2,8", (6, 8, 60)), ("3,16", (5, 12, 64)), ("4,8", (4, 256, 128)),
                                         ("5,8", (3, 20, 40)), ("8,8", (5, 32, 36))])
def test_split_spectral_maps(monkeypatch, split, shape):
    """plane pass, columns there and back with a multiplier per (k0, k1, k2),
    plane pass: the multiplier sees the frequencies it should."""
    monkeypatch.setenv("MIFFT_SPLIT", split)
    n0, n1, n2 = shape
    lists, _ = _lists(shape, 1, 1)
    po = lists["plane_poisson"]
    assert [p["kind"] for p in po] == ["plane_r2c", "cols_mid", "plane_c2r"]
    a, c, b = po
    rng = np.random.default_rng(5)
    x = rng.standard_normal(shape)
    m = rng.standard_normal((n0, n1, n2 // 2 + 1))
    m[..., 0] = m[..., -1] = 0.5  # (real data: keep the ends Hermitian)
    flat = x.reshape(-1, 2) @ [1, 1j]
    D = np.zeros(c["groups"] * c["gs"][0], complex)
    _plane(a, flat, D, n1)
    L, B, A = c["rows"], c["nb"], c["groups"]
    for g in range(A):
        idx = np.array([[g * c["gs"][0] + i * c["es"][0] + y * c["ys"][0] for y in range(B)] for i in range(L)])
        idx = idx[:, :, None] + np.arange(c["cols"])
        v = _dft(_dft(D[idx], 1, 1), 1, 0) * m[:, g + A * np.arange(B), :]
        v = _dft(_dft(v, -1, 1), -1, 0) * np.exp(2j * np.pi * np.arange(B) * g / n1)[None, :, None]
        D[idx] = v
    out = np.zeros(x.size // 2, complex)
    _plane(b, D, out, n1)
    full = np.fft.irfftn(np.fft.rfftn(x) * m, s=shape, axes=(0, 1, 2)) * x.size
    want = full.reshape(-1, 2) @ [1, 1j]
    assert np.linalg.norm(out - want) <= 1e-12 * np.linalg.norm(want)


def test_tile_order_is_the_plans():
    """Which tiles an XCD takes is fixed when the plan is made (the environment
    is not read at launch): consecutive ones where their number divides by 8."""
    seen = set()
    for shape, kind, prec in (((256, 256, 256), 1, 0), ((256, 256, 256), 1, 1), ((100, 120, 144), 0, 0), ((200, 200, 200), 0, 0)):
        lists, _ = _lists(shape, kind, prec)
        for name, passes in lists.items():
            for p in passes:
                if p["kind"] in ("cols", "cols_mid"):
                    assert p["xcd"] == (p["tiles"] % 8 == 0), (shape, name)
                    seen.add(p["xcd"])
                else:
                    assert p["xcd"] == 0
    assert seen == {0, 1}


@pytest.mark.parametrize("shape,kind", [((200, 20, 900), 1), ((300, 9, 480), 0), ((200, 20, 972), 1), ((300, 9, 450), 0),
                                        ((375, 30, 750), 1), ((120, 135, 486), 1), ((64, 10, 810), 1), ((200, 16, 500), 0)])
def test_long_fp64_lines_keep_the_one_axis_passes(shape, kind):
    """Lines whose plane kernels would not fit the registers, or take five
    stages: the one-axis passes are faster."""
    lists, _ = _lists(shape, kind, 1)
    assert not [k for k in lists if k.startswith("plane_")]
    lists, _ = _lists((200, 20, 720 if kind else 360), kind, 1)
    assert lists["plane_forward"] and lists["plane_inverse"]


@pytest.mark.parametrize("shape,kind,prec", [((24, 60, 300), 1, 0), ((10, 45, 300), 1, 0), ((12, 20, 750), 1, 0), ((8, 108, 60), 0, 0),
                                             ((2, 243, 180), 0, 0), ((3, 243, 162), 1, 1), ((8, 256, 256), 0, 1),
                                             ((8, 81, 864), 1, 0), ((4, 600, 240), 0, 0), ((40, 12, 750), 1, 0)])
def test_few_large_planes_keep_the_one_axis_passes(monkeypatch, shape, kind, prec):
    """A plane is one workgroup's work: few and large ones are slower than the
    separate passes.  Small ones, and many, keep the two-axis passes, and
    MIFFT_PLANES=1 takes them wherever they fit."""
    lists, _ = _lists(shape, kind, prec)
    assert not [k for k in lists if k.startswith("plane_")]
    monkeypatch.setenv("MIFFT_PLANES", "1")
    lists, _ = _lists(shape, kind, prec)
    assert lists["plane_forward"] and lists["plane_inverse"]
    monkeypatch.delenv("MIFFT_PLANES")
    for s, k, pr in (((2, 64, 64), 0, 0), ((64, 64, 64), 0, 1), ((32, 32, 32), 0, 1), ((200, 128, 128), 0, 0),
                     ((1024, 60, 300), 1, 0)):
        assert _lists(s, k, pr)[0]["plane_forward"]


def test_plane_rows_do_not_share_banks():
    """The rows of a wavefront's lines are no multiple of 16 elements apart in
    LDS (tile, two twiddle tables, digit reversal, split factors make its size)."""
    for n2 in (15, 30, 48, 60, 90, 96, 120, 128, 150, 240, 256):
        for prec in (0, 1):
            p = _lists((1024, 20, n2), 0, prec)[0]["plane_forward"][0]
            assert p["kind"] == "plane" and p["nb"] == 1
            A, L, esz = p["rows"], p["L"], 16 if prec else 8
            pitch, rest = divmod(p["lds"] // esz - L - 2 * A - (A + 3) // 4, A)
            assert rest == 0 and pitch > L and pitch % 16 != 0, (n2, prec, pitch)


@pytest.mark.parametrize("shape,kind", [((72, 160, 288), 0), ((72, 216, 180), 0), ((100, 150, 576), 1), ((96, 120, 864), 1)])
def test_wide_columns_tiles_count_as_alone(shape, kind):
    """More than 512 threads take a CU's registers: with more tiles than CUs,
    such a tile is weighed as one that is alone there, and narrower ones or the
    one-axis passes run."""
    lists, _ = _lists(shape, kind, 0)
    for name in ("plane_forward", "plane_inverse"):
        for p in lists.get(name, []):
            assert p["kind"] != "cols" or p["block"] <= 512
