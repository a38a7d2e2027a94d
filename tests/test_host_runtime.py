"""Host code of the library on a host-side stand-in for the HIP runtime
(hip_host.h), where streams run only when waited for and freed memory comes
back at the same address: ordering and memory accounting without a device."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1011_3318_amd", "csrc")


def run_driver(tmp_path, name):
    exe = str(tmp_path / name)
    # what a driver does not call (kernel launches) stays unresolved
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        f"-I{ROOT}/include", f"-I{CSRC}", f"-I{HERE}", "-o", exe, os.path.join(HERE, name + ".cpp"),
                        "-lpthread", "-no-pie", "-Wl,--unresolved-symbols=ignore-all"], capture_output=True, text=True)
    if r.returncode != 0:
        pytest.fail(r.stdout + r.stderr)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    return out.stdout


def test_staged_transfers_are_ordered(tmp_path):
    out = run_driver(tmp_path, "stage_driver")
    for name in ("default-stream", "own-stream", "per-thread-stream"):
        assert f"ok {name}" in out


def test_workspaces(tmp_path):
    out = run_driver(tmp_path, "workspace_driver")
    for name in ("kept-fields-give-way", "rebuilt-after-failed-growth", "small-staging-beside-idle-block", "failed-call-leaves-no-work",
                 "failed-request-releases-source"):
        assert f"ok {name}" in out
