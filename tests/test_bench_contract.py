"""Host-side checks of bench.py's command line (no GPU needed)."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_bench(*args, env=None):
    e = dict(os.environ)
    e.update(env or {})
    return subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), *args], capture_output=True, text=True,
                          env=e, timeout=120)


def test_more_than_one_gpu_is_refused_with_a_message():
    r = run_bench("--gpus", "2")
    assert r.returncode != 0
    assert "one-GPU" in r.stderr + r.stdout and "--gpus 1" in r.stderr + r.stdout
    assert not r.stdout.strip().startswith("{")  # no result line


def test_a_multi_rank_launch_is_refused_too():
    r = run_bench("--gpus", "1", env={"WORLD_SIZE": "2", "RANK": "0"})
    assert r.returncode != 0
    assert "one-GPU" in r.stderr + r.stdout


@pytest.mark.parametrize("cfg", ["dsv3", "qwen", "stress"])
def test_traffic_of_a_label_is_that_of_all_its_launches(cfg):
    """The roofline's time and FLOPs per launch are means over a label's launches, so its bytes have to be; the kernel
    that the label names is the one that layers with shared experts run, or layers without."""
    sys.path.insert(0, ROOT)
    import bench
    import workloads as wl

    path = os.path.join(ROOT, "profiles", f"hbm_traffic_{cfg}.txt")
    rows = [ln.rstrip("\n").split("\t") for ln in open(path) if not ln.startswith("#")]
    of = {r[4]: (int(r[0]), float(r[3])) for r in rows}
    gemms = [n for n in of if "gemm_kernel" in n or "w_light_kernel" in n]
    named = []
    for label in bench.GEMM_LABELS:
        symbol = bench.symbol(label, wl.CONFIGS[cfg].n_shared > 0)
        assert symbol in of, label
        assert bench.measured_traffic(cfg, label)[0] == pytest.approx(of[symbol][1])
        named.append(symbol)
    assert sorted(named) == sorted(gemms)   # every GEMM kernel of the profile belongs to one label
    assert bench.measured_traffic("tiny", bench.GEMM_LABELS[0])[0] is None


@pytest.mark.parametrize("shared", [False, True])
def test_the_kernels_of_the_labels_are_those_of_the_library(shared):
    """The table of kernel names is written by hand: it names kernels that the built library holds."""
    sys.path.insert(0, ROOT)
    import bench

    lib = os.path.join(ROOT, "paper_2502_02581_amd", "libmoe_hip.so")
    if shutil.which("nm") is None or not os.path.exists(lib):
        pytest.skip("needs nm and the built library")
    names = subprocess.run(["nm", "-C", lib], capture_output=True, text=True, check=True, timeout=120).stdout
    held = {ln.split(" ", 2)[2].removeprefix("void ") for ln in names.splitlines() if "moe::" in ln and ln.count(" ") >= 2}
    for label in bench.GEMM_LABELS:
        assert bench.symbol(label, shared) in held, label
