"""Plane passes (z- and y-axis of a plane in LDS, one pass): against the oracle
at the sizes where they can go wrong -- the shortest and longest lines and
columns, lines that leave lanes of a wavefront idle, rows that do not fill a
wavefront, one to four column stages, planes near the LDS limit and more
planes than the device holds at once -- and in place, grouped and inside the
spectral operators."""
import numpy as np
import pytest

import oracle
from paper_1506_07933_amd import synth
from conftest import TOL, rel_l2

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

C2C = [(3, 2, 2), (1, 3, 4), (5, 125, 100), (2, 250, 10), (1, 8, 15), (3, 8, 512), (2, 18, 486), (200, 128, 128),
       (2, 81, 48), (10, 1000, 16, 8), (2, 3, 5, 6, 36), (300, 4, 9, 30), (6, 96, 90), (2, 600, 5)]


def _plane_lines(p, which):
    return [line for line in p.describe().splitlines() if line.startswith("plane_" + which)]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", C2C)
def test_c2c_planes(shape, prec):
    from paper_1506_07933_amd import Plan
    cd = np.complex64 if prec == "fp32" else np.complex128
    x = synth.uniform_complex(shape, cd, seed=sum(shape))
    p = Plan(shape, "c2c", prec)
    print("  ", shape, prec, [line.split()[1:4] for line in _plane_lines(p, "forward")], flush=True)
    xd = torch.from_numpy(x).cuda()
    X = p.forward(xd)
    ref = oracle.fftnd_c2c(x.astype(np.complex128), -1)
    assert rel_l2(X.cpu().numpy(), ref) <= TOL[prec]
    y = p.inverse(X)
    assert rel_l2(y.cpu().numpy(), np.prod(shape) * x.astype(np.complex128)) <= TOL[prec]
    z = xd.clone()
    p.forward(z, out=z)
    assert torch.equal(z, X)
    p.inverse(z, out=z)
    assert torch.equal(z, y)
    p.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [(3, 2, 4), (4, 9, 30), (2, 128, 90), (2, 16, 1024), (200, 100, 192), (1, 64, 64),
                                   (9, 1000, 15, 18), (3, 4, 10, 50)])
def test_real_planes(shape, prec):
    """Forward, and C2R of a spectrum that is not Hermitian (the imaginary
    parts of its ends do not count); inputs are kept."""
    from paper_1506_07933_amd import Plan
    rd = np.float32 if prec == "fp32" else np.float64
    x = synth.normal_real(shape, rd, seed=sum(shape))
    p = Plan(shape, "r2c", prec)
    print("  ", shape, prec, [line.split()[1:4] for line in _plane_lines(p, "forward")], flush=True)
    xd = torch.from_numpy(x).cuda()
    Y = p.forward(xd)
    assert rel_l2(Y.cpu().numpy(), oracle.fftnd_r2c(x.astype(np.float64))) <= TOL[prec]
    half = shape[:-1] + (shape[-1] // 2 + 1,)
    h = synth.uniform_complex(half, np.complex64 if prec == "fp32" else np.complex128, seed=7)
    hd = torch.from_numpy(h).cuda()
    u = p.inverse(hd)
    assert rel_l2(u.cpu().numpy(), oracle.fftnd_c2r(h.astype(np.complex128), shape[-1])) <= TOL[prec]
    np.testing.assert_array_equal(hd.cpu().numpy(), h)
    np.testing.assert_array_equal(xd.cpu().numpy(), x)
    p.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [(8, 6, 4), (40, 48, 100), (1, 16, 36)])
def test_spectral_operators_on_planes(shape, prec):
    from paper_1506_07933_amd import Plan
    rd = np.float32 if prec == "fp32" else np.float64
    f = synth.normal_real(shape, rd, seed=5)
    f = (f - f.mean(dtype=np.float64)).astype(rd)
    p = Plan(shape, "r2c", prec)
    assert len(_plane_lines(p, "poisson")) == 3
    fd = torch.from_numpy(f).cuda()
    assert rel_l2(p.poisson(fd).cpu().numpy(), oracle.poisson_solve(f.astype(np.float64))) <= TOL[prec]
    g = p.gradient(fd)
    ref = oracle.gradient(f.astype(np.float64))
    for j in range(3):
        if np.linalg.norm(ref[j]) > 0:
            assert rel_l2(g[j].cpu().numpy(), ref[j]) <= TOL[prec]
        assert torch.equal(g[j], p.spectral(oracle.OP_DX + j, fd))
    p.close()


def test_grouped_planes_equal_single_ones():
    """20 members of one shape (two launches of a pass), planes of each."""
    from paper_1506_07933_amd import BatchPlan, Plan
    shapes = [(12, 20, 36)] * 20 + [(30, 64, 64)] * 3
    data = [synth.uniform_complex(s, np.complex64, seed=i) for i, s in enumerate(shapes)]
    xs = [torch.from_numpy(d).cuda() for d in data]
    outs = [torch.empty_like(x) for x in xs]
    b = BatchPlan(shapes, "fp32", mode="grouped")
    b.forward(xs, outs)
    for s, x, o in zip(shapes, xs, outs):
        p = Plan(s, "c2c", "fp32")
        assert torch.equal(p.forward(x), o)
        p.close()
    b.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("split,shape", [("2,16", (6, 8, 12)), ("3,16", (5, 12, 18)), ("4,8", (40, 8, 20)), ("5,8", (3, 100, 10)),
                                         ("6,16", (9, 24, 8)), ("8,8", (125, 32, 6)), ("4,8", (30, 256, 128)),
                                         ("8,4", (2, 512, 64)), ("2,32", (2, 4, 2))])
def test_split_planes(monkeypatch, split, shape, prec):
    """Every B of a split y-axis, through the workspace and through the output,
    ragged column tiles: C2C in both directions (in place: the one-axis passes
    or the same bits), R2C, and C2R of a spectrum that is not Hermitian."""
    from paper_1506_07933_amd import Plan
    monkeypatch.setenv("MIFFT_SPLIT", split)
    cd, rd = (np.complex64, np.float32) if prec == "fp32" else (np.complex128, np.float64)
    x = synth.uniform_complex(shape, cd, seed=sum(shape))
    p = Plan(shape, "c2c", prec)
    print("  ", shape, prec, [line.split()[1:4] for line in _plane_lines(p, "forward")], flush=True)
    assert any("kind=cols" in line for line in _plane_lines(p, "forward"))
    xd = torch.from_numpy(x).cuda()
    X = p.forward(xd)
    ref = oracle.fftnd_c2c(x.astype(np.complex128), -1)
    assert rel_l2(X.cpu().numpy(), ref) <= TOL[prec]
    np.testing.assert_array_equal(xd.cpu().numpy(), x)
    n = float(np.prod(shape))
    assert rel_l2(p.inverse(X).cpu().numpy(), n * x.astype(np.complex128)) <= TOL[prec]
    z = xd.clone()
    p.forward(z, out=z)
    assert rel_l2(z.cpu().numpy(), ref) <= TOL[prec]
    p.inverse(z, out=z)
    assert rel_l2(z.cpu().numpy(), n * x.astype(np.complex128)) <= TOL[prec]
    p.close()
    if shape[2] < 4:
        return
    p = Plan(shape, "r2c", prec)
    r = synth.normal_real(shape, rd, seed=3)
    Y = p.forward(torch.from_numpy(r).cuda())
    assert rel_l2(Y.cpu().numpy(), oracle.fftnd_r2c(r.astype(np.float64))) <= TOL[prec]
    h = synth.uniform_complex(shape[:-1] + (shape[-1] // 2 + 1,), cd, seed=7)
    hd = torch.from_numpy(h).cuda()
    assert rel_l2(p.inverse(hd).cpu().numpy(), oracle.fftnd_c2r(h.astype(np.complex128), shape[-1])) <= TOL[prec]
    np.testing.assert_array_equal(hd.cpu().numpy(), h)
    p.close()


def test_grouped_split_planes(monkeypatch):
    """Grouped launches of both passes, with some transforms in place (those
    run the one-axis passes)."""
    from paper_1506_07933_amd import BatchPlan
    monkeypatch.setenv("MIFFT_SPLIT", "4,8")
    shapes = [(12, 20, 36)] * 19
    data = [synth.uniform_complex(s, np.complex64, seed=i) for i, s in enumerate(shapes)]
    xs = [torch.from_numpy(d).cuda() for d in data]
    outs = [x if i % 4 == 1 else torch.empty_like(x) for i, x in enumerate(xs)]
    b = BatchPlan(shapes, "fp32", mode="grouped")
    b.forward(xs, outs)
    for d, o in zip(data, outs):
        assert rel_l2(o.cpu().numpy(), oracle.fft3d_c2c(d.astype(np.complex128), -1)) <= TOL["fp32"]
    b.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("split,shape", [("2,8", (6, 8, 60)), ("3,16", (125, 12, 30)), ("4,8", (16, 256, 128)),
                                         ("5,8", (2, 20, 64)), ("6,8", (81, 24, 60)), ("8,4", (10, 32, 50))])
def test_split_spectral_operators(monkeypatch, split, shape, prec):
    """Every operator, gradient and divergence on a split y-axis, one to four
    stages along x; with a caller workspace too; inputs are kept."""
    from paper_1506_07933_amd import Plan
    monkeypatch.setenv("MIFFT_SPLIT", split)
    rd = np.float32 if prec == "fp32" else np.float64
    f = synth.normal_real(shape, rd, seed=5)
    f = (f - f.mean(dtype=np.float64)).astype(rd)
    f64 = f.astype(np.float64)
    p = Plan(shape, "r2c", prec)
    assert [line.split()[1] for line in _plane_lines(p, "poisson")] == ["kind=plane_r2c", "kind=cols_mid", "kind=plane_c2r"]
    fd = torch.from_numpy(f).cuda()
    for op in range(6):
        ref = oracle.spectral_apply(f64, op, 1.5)
        assert rel_l2(p.spectral(op, fd, alpha=1.5).cpu().numpy(), ref) <= TOL[prec], op
    g = p.gradient(fd)
    for j, r in enumerate(oracle.gradient(f64)):
        assert rel_l2(g[j].cpu().numpy(), r) <= TOL[prec]
        assert torch.equal(g[j], p.spectral(oracle.OP_DX + j, fd))
    v = [synth.normal_real(shape, rd, seed=20 + j) for j in range(3)]
    d = p.divergence([torch.from_numpy(u).cuda() for u in v])
    assert rel_l2(d.cpu().numpy(), oracle.divergence(*[u.astype(np.float64) for u in v])) <= TOL[prec]
    np.testing.assert_array_equal(fd.cpu().numpy(), f)
    p.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_persistent_plane_items(prec):
    """Plane items of the one-launch batch beside z- and y-items: the smallest
    planes, lines that leave lanes idle, one plane per item and several, planes
    too large for LDS; in place gives the same bits."""
    from paper_1506_07933_amd import BatchPlan
    shapes = [(3, 2, 2), (1, 128, 64), (40, 4, 3), (2, 125, 100), (9, 16, 256), (5, 250, 8), (2, 256, 256), (32, 45, 27)]
    cd = np.complex64 if prec == "fp32" else np.complex128
    data = [synth.uniform_complex(s, cd, seed=i) for i, s in enumerate(shapes)]
    xs = [torch.from_numpy(d).cuda() for d in data]
    outs = [torch.empty_like(x) for x in xs]
    b = BatchPlan(shapes, prec)
    print(b.describe().splitlines()[0], flush=True)
    b.forward(xs, outs)
    torch.cuda.synchronize()
    assert not b.aborted()
    for s, d, o in zip(shapes, data, outs):
        assert rel_l2(o.cpu().numpy(), oracle.fft3d_c2c(d.astype(np.complex128), -1)) <= TOL[prec], s
    b.forward(xs, xs)
    torch.cuda.synchronize()
    assert not b.aborted()
    for x, o in zip(xs, outs):
        assert torch.equal(x, o)
    b.close()


@pytest.mark.parametrize("mode,shape,together", [("kernels", (64, 128, 128), 1), ("grouped", (64, 128, 128), 4),
                                                 ("grouped", (4, 256, 128), 1), ("kernels", (4, 256, 128), 1),
                                                 ("grouped", (48, 64, 96), 4), ("grouped", (20, 96, 90), 4)])
def test_batches_of_plans_run_the_schedule_of_single_transforms(mode, shape, together):
    """How many transforms run together (one by one in a batch of per-pass
    kernels, and where they need a workspace) shapes the launches, not the
    passes: every mode gives the bits of single transforms."""
    from paper_1506_07933_amd import BatchPlan, Plan
    xs = [torch.from_numpy(synth.uniform_complex(shape, np.complex64, seed=i)).cuda() for i in range(4)]
    b = BatchPlan([shape] * 4, "fp32", mode=mode)
    assert "shape=%dx%dx%d launched_together=%d " % (*shape, together) in b.describe()
    outs = b.forward(xs)
    p = Plan(shape, "c2c", "fp32")
    for x, o in zip(xs, outs):
        assert torch.equal(o, p.forward(x))
    p.close()
    b.close()


def test_batch_report_tells_plane_items_from_lines():
    """A plane pass and a z-pass of one length: both are listed, as what they are."""
    from paper_1506_07933_amd import BatchPlan
    shapes = [(40, 4, 100), (2, 125, 100), (6, 240, 100), (3, 256, 250)]
    b = BatchPlan(shapes, "fp64")
    lines = [dict(kv.split("=") for kv in line.split() if "=" in kv) for line in b.describe().splitlines()
             if line.startswith("stage=")]
    assert len([1 for d in lines if d["stage"] == "zy"]) == 1
    assert [(d["L"], d["rows"]) for d in lines if d["stage"] == "zy"] == [("100", "4")]
    assert sorted(int(d["L"]) for d in lines if d["stage"] == "z") == [100, 250]
    assert sorted(int(d["L"]) for d in lines if d["stage"] == "y") == [125, 240, 256]
    assert sorted(int(d["L"]) for d in lines if d["stage"] == "x") == [2, 3, 6, 40]
    assert all(d["policy"] in ("0", "2") and d["emul"] in ("1", "2") for d in lines if d["stage"] != "zy")
    b.close()


@pytest.mark.parametrize("split,shape,prec", [(None, (40, 48, 100), "fp32"), (None, (8, 6, 4), "fp64"), ("2,8", (6, 8, 60), "fp32"),
                                              ("4,8", (16, 256, 128), "fp64"), ("6,8", (81, 24, 60), "fp32")])
def test_spectral_operators_in_a_callers_workspace(monkeypatch, split, shape, prec):
    """Workspaces of exactly the reported sizes: the bits of the plan's own, and
    nothing written past their ends."""
    from paper_1506_07933_amd import Plan
    if split:
        monkeypatch.setenv("MIFFT_SPLIT", split)
    rd = np.float32 if prec == "fp32" else np.float64
    f = torch.from_numpy(synth.normal_real(shape, rd, seed=5)).cuda()
    v = [torch.from_numpy(synth.normal_real(shape, rd, seed=20 + j)).cuda() for j in range(3)]
    p = Plan(shape, "r2c", prec)
    assert _plane_lines(p, "poisson")

    def guarded(nbytes):
        t = torch.full((nbytes + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        return t, t[:nbytes]

    full, ws = guarded(p.poisson_ws_bytes)
    for op in range(6):
        assert torch.equal(p.spectral(op, f, alpha=1.5, ws=ws), p.spectral(op, f, alpha=1.5))
    assert bool((full[p.poisson_ws_bytes:] == 0x5A).all())
    full, ws = guarded(p.spectral_ws_bytes)
    for a, b in zip(p.gradient(f, ws=ws), p.gradient(f)):
        assert torch.equal(a, b)
    assert torch.equal(p.divergence(v, ws=ws), p.divergence(v))
    assert bool((full[p.spectral_ws_bytes:] == 0x5A).all())
    p.close()


def _no_element_finite(t):
    r = torch.view_as_real(t) if t.is_complex() else t.unsqueeze(-1)
    return not bool(torch.isfinite(r).all(-1).any())


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("split,shape", [(None, (20, 36, 100)), (None, (3, 16, 30)), ("2,16", (6, 8, 12)), ("4,8", (40, 8, 20)),
                                         ("4,8", (30, 256, 128)), ("5,8", (9, 100, 10))])
def test_nan_and_infinity_reach_every_output(monkeypatch, split, shape, prec):
    """Every output depends on every input: one NaN or infinity leaves no
    element finite (no padding, idle lane or masked column takes its place)."""
    from paper_1506_07933_amd import Plan
    if split:
        monkeypatch.setenv("MIFFT_SPLIT", split)
    cd, rd = (np.complex64, np.float32) if prec == "fp32" else (np.complex128, np.float64)
    at = tuple(n - 1 for n in shape)
    for bad in (float("nan"), float("inf"), float("-inf")):
        p = Plan(shape, "c2c", prec)
        x = torch.from_numpy(synth.uniform_complex(shape, cd, seed=1)).cuda()
        x[at] = complex(bad, 0.25)
        assert _no_element_finite(p.forward(x)) and _no_element_finite(p.inverse(x))
        z = x.clone()
        assert _no_element_finite(p.forward(z, out=z))
        p.close()
        p = Plan(shape, "r2c", prec)
        r = torch.from_numpy(synth.normal_real(shape, rd, seed=1)).cuda()
        r[at] = bad
        assert _no_element_finite(p.forward(r))
        if bad != bad:
            assert _no_element_finite(p.poisson(r))
            assert all(_no_element_finite(g) for g in p.gradient(r))
            h = p.forward(torch.from_numpy(synth.normal_real(shape, rd, seed=2)).cuda())
            h[0, 0, 1] = complex(bad, bad)
            assert _no_element_finite(p.inverse(h))
        p.close()


@pytest.mark.parametrize("mode", ["grouped", "persistent"])
def test_nan_stays_in_its_transform(mode):
    from paper_1506_07933_amd import BatchPlan
    shapes = [(12, 20, 36)] * 5 + [(30, 64, 64)] * 2
    xs = [torch.from_numpy(synth.uniform_complex(s, np.complex64, seed=i)).cuda() for i, s in enumerate(shapes)]
    b = BatchPlan(shapes, "fp32", mode=mode)
    want = b.forward(xs)
    bad = [x.clone() for x in xs]
    for k in (1, 6):
        bad[k][3, 4, 5] = complex(float("nan"), 0.0)
    got = b.forward(bad)
    torch.cuda.synchronize()
    assert mode == "grouped" or not b.aborted()
    for k, (g, w) in enumerate(zip(got, want)):
        assert _no_element_finite(g) if k in (1, 6) else torch.equal(g, w)
    b.close()


def test_first_call_of_a_plan_under_capture():
    """A large-LDS kernel whose first launch is a capture: replays give the
    eager result, with eager work between them."""
    from paper_1506_07933_amd import Plan
    p = Plan((300, 96, 90), "c2c", "fp64")
    assert _plane_lines(p, "forward")
    x = torch.from_numpy(synth.uniform_complex((300, 96, 90), np.complex128, seed=2)).cuda()
    y = torch.zeros_like(x)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        p.forward(x, out=y)
    for seed in (2, 3, 4):
        x.copy_(torch.from_numpy(synth.uniform_complex((300, 96, 90), np.complex128, seed=seed)))
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, p.forward(x))
    p.close()


@pytest.mark.parametrize("split,shape,prec", [(None, (100, 120, 144), "fp32"), (None, (100, 100, 100), "fp64"),
                                              ("3,16", (50, 96, 90), "fp32"), ("8,8", (125, 32, 60), "fp64")])
def test_in_place_split_calls_need_no_memory_and_agree(monkeypatch, split, shape, prec):
    """A plan that reports no workspace has none: creating it takes less memory
    than its array.  In place, the plain call, the one with a workspace, the
    static one and the members of a batch give the same bits, also on two
    streams at once; they run the one-axis passes, so the out-of-place call's
    bits are near, not equal."""
    from paper_1506_07933_amd import BatchPlan, Plan
    from paper_1506_07933_amd._lib import check, lib
    if split:
        monkeypatch.setenv("MIFFT_SPLIT", split)
    cd = np.complex64 if prec == "fp32" else np.complex128
    x = torch.from_numpy(synth.uniform_complex(shape, cd, seed=3)).cuda()
    x2 = torch.from_numpy(synth.uniform_complex(shape, cd, seed=4)).cuda()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    plans = [Plan(shape, "c2c", prec) for _ in range(4)]
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < 4 * max(x.numel() * x.element_size() // 2, 2 << 20)
    p = plans[0]
    assert p.workspace_bytes == 0 and any("kind=cols" in line for line in _plane_lines(p, "forward"))
    X = p.forward(x)
    assert rel_l2(X.cpu().numpy(), oracle.fftnd_c2c(x.cpu().numpy().astype(np.complex128), -1)) <= TOL[prec]
    z, z2 = x.clone(), x2.clone()
    Z, Z2 = p.forward(z, out=z).clone(), p.forward(z2, out=z2).clone()
    assert rel_l2(Z.cpu().numpy(), X.cpu().numpy()) <= TOL[prec]
    Y = p.inverse(z, out=z).clone()
    assert rel_l2(Y.cpu().numpy(), x.numel() * x.cpu().numpy().astype(np.complex128)) <= TOL[prec]
    ws = torch.empty(16, dtype=torch.uint8, device="cuda")
    z = x.clone()
    assert torch.equal(p.forward(z, out=z, ws=ws), Z) and torch.equal(p.inverse(z, out=z, ws=ws), Y)
    z = x.clone()
    s = torch.cuda.current_stream().cuda_stream or None
    check(lib.mifft_execute_forward_static(p.handle, z.data_ptr(), z.data_ptr(), s), "static")
    assert torch.equal(z, Z)
    za, zb = x.clone(), x2.clone()
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(8):
        za.copy_(x)
        zb.copy_(x2)
        torch.cuda.synchronize()
        p.forward(za, out=za, stream=sa)
        p.forward(zb, out=zb, stream=sb)
        torch.cuda.synchronize()
        assert torch.equal(za, Z) and torch.equal(zb, Z2)
    for q in plans:
        q.close()
    for mode in ("grouped", "kernels"):
        b = BatchPlan([shape] * 3, prec, mode=mode)
        xs = [x.clone(), x2.clone(), x.clone()]
        b.forward(xs, [xs[0], torch.empty_like(x2), xs[2]])
        assert torch.equal(xs[0], Z) and torch.equal(xs[2], Z) and torch.equal(xs[1], x2)
        b.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [(5, 125, 100), (2, 250, 10), (3, 8, 512), (2, 18, 360), (3, 128, 128), (2, 81, 48),
                                   (6, 96, 90), (2, 600, 5), (4, 108, 80), (3, 243, 54)])
def test_planes_wherever_they_fit(monkeypatch, shape, prec):
    """The schedules that the planner leaves out for speed (MIFFT_PLANES=1): near
    the LDS limit, few planes, three and four stages."""
    from paper_1506_07933_amd import Plan
    monkeypatch.setenv("MIFFT_PLANES", "1")
    cd, rd = (np.complex64, np.float32) if prec == "fp32" else (np.complex128, np.float64)
    x = synth.uniform_complex(shape, cd, seed=sum(shape))
    p = Plan(shape, "c2c", prec)
    assert _plane_lines(p, "forward") and _plane_lines(p, "inverse")
    X = p.forward(torch.from_numpy(x).cuda())
    assert rel_l2(X.cpu().numpy(), oracle.fftnd_c2c(x.astype(np.complex128), -1)) <= TOL[prec]
    assert rel_l2(p.inverse(X).cpu().numpy(), np.prod(shape) * x.astype(np.complex128)) <= TOL[prec]
    p.close()
    real = shape[:2] + (2 * shape[2],)
    if real[2] > 1024:
        return
    p = Plan(real, "r2c", prec)
    assert _plane_lines(p, "forward") and _plane_lines(p, "inverse")
    r = synth.normal_real(real, rd, seed=3)
    Y = p.forward(torch.from_numpy(r).cuda())
    assert rel_l2(Y.cpu().numpy(), oracle.fftnd_r2c(r.astype(np.float64))) <= TOL[prec]
    assert rel_l2(p.inverse(Y).cpu().numpy(), np.prod(real) * r.astype(np.float64)) <= TOL[prec]
    p.close()
