"""The library's host code, linked with its kernel objects, over a HIP runtime
that launches nothing (tests/fake_hip/driver.cpp): launch sizes, announced
LDS, allocations and error paths at any size, without a GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    from paper_2101_08763_amd import build as B
    if not os.path.exists(B.HIPCC):
        pytest.skip("hipcc not available")
    os.makedirs(B.OBJDIR, exist_ok=True)
    objs = []
    for src in B.SOURCES:
        obj = os.path.join(B.OBJDIR, os.path.splitext(src)[0] + ".o")
        if not os.path.exists(obj):
            B._compile(src, False)
        objs.append(obj)
    tmp = tmp_path_factory.mktemp("fake_hip")
    drv, exe = str(tmp / "driver.o"), str(tmp / "driver")
    for cmd in ([B.HIPCC, "-O1", "-std=c++17", f"-I{B.INCLUDE}", "-Wno-unused-value", "-c",
                 os.path.join(ROOT, "tests", "fake_hip", "driver.cpp"), "-o", drv],
                [B.HIPCC, f"--offload-arch={B.ARCH}", drv, *objs, "-o", exe]):
        r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, r.stdout + r.stderr
    return exe


def test_bench_names_the_kernel_that_runs(driver):
    """bench.dominant_kernel (which prices a workload) against the library's
    own choice, on both sides of every rule."""
    import bench
    env = {k: v for k, v in os.environ.items() if not k.startswith("EXEMCL_")}
    r = subprocess.run([driver, "kernels"], capture_output=True, text=True, timeout=300, env=env)
    lines = [ln.split() for ln in r.stdout.splitlines() if "eval_" in ln]
    assert r.returncode == 0 and len(lines) == 3 * 4 * 11, r.stdout + r.stderr
    for prec, n, d, name in lines:
        want = bench.dominant_kernel(["fp32", "fp16", "bf16"][int(prec)], int(n), int(d))
        assert want in name, (prec, n, d, name, want)


@pytest.mark.parametrize("check", ["grids", "devices", "counter", "limits"])
def test_host_runtime(driver, check):
    env = {k: v for k, v in os.environ.items() if not k.startswith("EXEMCL_")}
    r = subprocess.run([driver, check], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0 and "checks passed" in r.stdout, r.stdout + r.stderr
