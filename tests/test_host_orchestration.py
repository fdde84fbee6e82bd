"""The library's host code (graph loads, work lists, workspace, host copies,
batches and their schedules) under AddressSanitizer and
UndefinedBehaviorSanitizer, without a GPU.

``csrc/ef_api.cpp``, ``csrc/batch.cpp`` and ``csrc/csr_check.cpp`` are built
from source on test doubles of the HIP runtime and of the kernel launchers
(``tests/native/host_stub.cpp``): device memory is heap memory of exactly the
size asked for, the preparation of a graph is computed on the CPU, and every
launcher touches the extents its kernels may. The scenarios are in
``tests/native/host_driver.cpp``."""
import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2306_00606_amd", "csrc")
NATIVE = os.path.join(ROOT, "tests", "native")
HIP_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
FLAGS = ["-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
         "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__", "-I", HIP_INCLUDE,
         "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", NATIVE]

pytestmark = pytest.mark.skipif(
    shutil.which("g++") is None or not os.path.isdir(os.path.join(HIP_INCLUDE, "hip")),
    reason="needs g++ and the HIP headers")


def _run(cmd, **kw):
    return subprocess.run(cmd, capture_output=True, text=True, **kw)


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    td = tmp_path_factory.mktemp("host")
    srcs = [os.path.join(CSRC, f) for f in ("ef_api.cpp", "batch.cpp", "csr_check.cpp")]
    srcs += [os.path.join(NATIVE, f) for f in ("host_stub.cpp", "host_driver.cpp")]
    objs = [str(td / (os.path.basename(s) + ".o")) for s in srcs]
    with ThreadPoolExecutor(max_workers=len(srcs)) as ex:
        for r in ex.map(lambda so: _run(["g++", *FLAGS, "-c", so[0], "-o", so[1]]),
                        zip(srcs, objs)):
            assert r.returncode == 0, r.stderr
    exe = str(td / "host_driver")
    r = _run(["g++", "-fsanitize=address,undefined", *objs, "-o", exe])
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("scenario", ["calls", "batches", "first_use", "captured", "streams", "idle",
                                      "batch_room", "limits"])
def test_host_code(driver, scenario):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0",
               UBSAN_OPTIONS="print_stacktrace=1")
    env.pop("EF_MAX_DEVICE_BYTES", None)
    r = _run([driver, scenario], env=env, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.startswith("ok"), r.stdout
