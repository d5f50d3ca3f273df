"""Host-only checks under AddressSanitizer and UBSan: the ratio stop rule (against pow()),
which batches have results that are other matrices' inputs (against every pair of ranges),
the workgroups of teams (whole, consecutive, on one XCD), how many calls go without a team
after a late one, and the XCDs' runs of tiles for grids that 8 does not divide.  Compiled for the host only (hipcc --offload-host-only), so no GPU is needed."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC) and not shutil.which("hipcc"), reason="needs hipcc")
def test_batch_arithmetic_sanitized(tmp_path):
    exe = tmp_path / "batch_check"
    cmd = [HIPCC, "--offload-host-only", "-x", "hip", "-std=c++17", "-O1", "-g",
           "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
           "-Xarch_host", "-fno-sanitize-recover=all",
           "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2404_19163_amd", "csrc"),
           os.path.join(ROOT, "tests", "host", "batch_check.hip"), "-o", str(exe)]
    cc = subprocess.run(cmd, capture_output=True, text=True)
    assert cc.returncode == 0, cc.stderr[-4000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1",
               UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300, env=env)
    assert run.returncode == 0, (run.stdout[-2000:], run.stderr[-4000:])
    assert run.stdout.startswith("ok "), run.stdout
