"""Bookkeeping of steps that are queued without their routing, without a GPU: the library's source built for the host alone into
tests/sanitize/queued_steps_harness.cpp, whose launches count and fail where a check wants them to."""
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bookkeeping_of_queued_steps():
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        exe = os.path.join(tmp, "queued_steps_harness")
        subprocess.run([hipcc, "--offload-host-only", "-fuse-cuid=none", "-O1", "-std=c++17", "-pthread", "-o", exe, "-x", "hip",
                        os.path.join(ROOT, "tests", "sanitize", "queued_steps_harness.cpp")], check=True, cwd=tmp,
                       stdout=subprocess.PIPE, stderr=subprocess.PIPE)
        run = subprocess.run([exe], cwd=tmp, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout == "ok\n", run.stdout + run.stderr
