"""bench.py's host-side contract, without a GPU: more than one GPU is refused
with a message and exit status 2 (the measurement is of one GPU), and the
counter traffic is reported only for the kernel sources it was taken from."""
import json
import os
import subprocess
import sys

from conftest import ROOT


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr or "single MI355X" in r.stderr


def test_traffic_only_for_matching_sources(monkeypatch):
    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    import bench
    t = json.load(open(os.path.join(ROOT, "profiles", "traffic.json")))
    heads = {"z_contig", "y_strided", "x_strided"}   # the headline transform's passes
    assert heads <= set(t["kernels"])
    for name in heads:   # counter bytes near the algorithmic 2 GiB per pass
        assert 0.99 < t["kernels"][name]["hbm_bytes_per_launch"] / 2 ** 31 < 1.05
    for name, k in t["kernels"].items():   # other workloads' kernels: per-dispatch bytes
        if k.get("alg_bytes_per_launch"):
            assert 0.99 < k["hbm_bytes_per_launch"] / k["alg_bytes_per_launch"] < 1.5, name
    monkeypatch.setattr(bench, "csrc_hash", lambda: t["csrc_hash"])
    assert bench.load_traffic("y_strided", 2 ** 31) == t["kernels"]["y_strided"]["hbm_bytes_per_launch"]
    monkeypatch.setattr(bench, "csrc_hash", lambda: "0" * 16)
    assert bench.load_traffic("y_strided", 2 ** 31) is None


def test_rates_count_the_passes_that_run():
    """A schedule with two axes per pass reads and writes the array fewer times
    than it has axes; the rates count what runs."""
    import ctypes
    from paper_1506_07933_amd._lib import MIFFT_PLAN_ONLY, lib
    from paper_1506_07933_amd.fft import plan_describe, plan_destroy
    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    import bench

    def report(dims, kind):
        h = ctypes.c_void_p()
        arr = (ctypes.c_int * len(dims))(*dims)
        assert lib.mifft_plan_create_nd(ctypes.byref(h), len(dims), arr, kind, 0, MIFFT_PLAN_ONLY) == 0
        text = plan_describe(h.value)
        plan_destroy(h.value)
        return text

    for dims, kind, passes in (((512, 256, 128, 64), 0, 3), ((256, 256, 256), 1, 2), ((512, 512, 512), 0, 3),
                               ((100, 120, 144), 0, 2)):
        text = report(dims, kind)
        assert bench.passes_run(text, "forward") == bench.passes_run(text, "inverse") == passes
    shapes = [(8, 64, 64), (8, 256, 256), (1, 64, 64), (4, 1, 16)]
    persistent = "mode=persistent transforms=4 passes=7\nstage=zy L=64 rows=64 tpl=8 sub_per_item=8\n" \
                 "stage=z L=256 variant=0 chosen\n"
    assert bench.batch_bytes(persistent, shapes) == 16 * (2 * 8 * 64 * 64 + 3 * 8 * 256 * 256 + 64 * 64 + 2 * 64)
    grouped = "mode=grouped transforms=4 shapes=4\nshape=8x64x64 launched_together=1 passes=2\n" \
              "shape=8x256x256 launched_together=1 passes=3\nshape=1x64x64 launched_together=1 passes=1\n" \
              "shape=4x1x16 launched_together=1 passes=2\n"
    assert bench.batch_bytes(grouped, shapes) == bench.batch_bytes(persistent, shapes)
