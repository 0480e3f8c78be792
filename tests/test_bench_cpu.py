"""bench.py's command-line contract, checked without a GPU: it measures one
MI355X only, so a request for more GPUs ends with status 2 and a message,
before any device work; the options the driver passes are accepted."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(*args):
    return subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), *args],
                          capture_output=True, text=True, timeout=120, cwd=ROOT)


def test_more_than_one_gpu_is_refused():
    r = _run("--gpus", "2", "--steps", "3", "--warmup", "1")
    assert r.returncode == 2
    assert "one GPU" in (r.stdout + r.stderr)


def test_help_lists_the_driver_options():
    r = _run("--help")
    assert r.returncode == 0
    for opt in ("--gpus", "--steps", "--warmup", "--only", "--no-cpu-baseline"):
        assert opt in r.stdout


def test_gemm_traffic_is_reported():
    """The traffic constants belong to the kernel source that is built: a change
    of that file needs them measured again."""
    sys.path.insert(0, ROOT)
    import bench
    assert bench.gemm_traffic_bytes() is not None
