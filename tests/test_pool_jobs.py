"""Jobs of the host thread pool, as it is and under the compiler's sanitizers (CPU only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("sanitize", ["", "thread", "address,undefined"])
def test_every_task_runs_once(tmp_path, sanitize):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path / "pool_jobs")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wextra", "-pthread", *(["-fsanitize=" + sanitize] if sanitize else []),
                        "-I", os.path.join(ROOT, "paper_2104_07857_amd", "csrc"), os.path.join(ROOT, "tests", "c", "pool_jobs.cpp"),
                        "-o", exe], capture_output=True, text=True)
    if r.returncode != 0 and "cannot find -l" in r.stderr:
        pytest.skip("sanitizer runtime not installed: " + r.stderr.strip().splitlines()[-1])
    assert r.returncode == 0, r.stderr
    env = dict(os.environ, ASAN_OPTIONS="verify_asan_link_order=0", TSAN_OPTIONS="halt_on_error=1")
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env)
    assert run.returncode == 0 and "pool jobs ok" in run.stdout, run.stdout + run.stderr[-3000:]
