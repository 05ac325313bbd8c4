"""pf_graph_run and stream capture, on the CPU stand-in runtime
(tests/hostcheck): a call inside a caller's capture that is refused leaves the
handle as it was, and a run waits for a capture only where it has to."""
import os
import subprocess

import pytest
from test_host_runtime import CSRC, CXX, HERE, ROOT, launcher_stubs


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    tmp_path = tmp_path_factory.mktemp("capture")
    if not os.path.exists(CXX):
        pytest.skip("ROCm clang++ not found")
    stubs, names = launcher_stubs()
    for name in names:  # every stub also tells the driver its name
        stubs = stubs.replace(f"hipError_t {name}(", f"hipError_t {name} (")
        head, tail = stubs.split(f"hipError_t {name} (", 1)
        stubs = (head + f"hipError_t {name}(" +
                 tail.replace("{ fake_kernel(", f'{{ note_kernel("{name}"); fake_kernel(', 1))
    (tmp_path / "stubs.cpp").write_text('extern "C" void note_kernel(const char* name);\n' + stubs)
    exe = str(tmp_path / "driver")
    cmd = [CXX, "-std=c++17", "-g", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-w", "-fsanitize=address,undefined",
           "-fno-omit-frame-pointer", "-o", exe, os.path.join(CSRC, "pf_api.cpp"),
           os.path.join(HERE, "fake_hip.cpp"), os.path.join(HERE, "driver_capture.cpp"),
           str(tmp_path / "stubs.cpp")]
    r = subprocess.run(cmd, capture_output=True, text=True, cwd=str(tmp_path))
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return exe


def _run(exe, scenario):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1",
               UBSAN_OPTIONS="halt_on_error=1")
    r = subprocess.run([exe, scenario], capture_output=True, text=True, env=env, timeout=120)
    assert r.returncode == 0 and "done" in r.stdout, (r.stdout + r.stderr)[-4000:]


def test_refused_capture_leaves_the_pending_ancestors(driver):
    _run(driver, "refused")


def test_a_later_run_goes_from_the_graphs_there_are(driver):
    _run(driver, "ladder")


def test_first_run_refused_inside_a_capture(driver):
    _run(driver, "first")
