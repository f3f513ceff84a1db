"""The library's host code from several threads under ThreadSanitizer, over the HIP
runtime of host_stubs.cpp (CPU)."""
import subprocess

from test_host_stubs_cpu import _build


def test_first_calls_of_two_threads(tmp_path):
    """Two threads that size a 3-D launch for the first time: no data race."""
    exe = _build(str(tmp_path / "stubs_tsan"), ["-fsanitize=thread"])
    syms = subprocess.run(["nm", exe], capture_output=True, text=True, check=True).stdout
    assert "__tsan_read" in syms   # instrumented
    for _ in range(3):
        p = subprocess.run([exe, "threads"], capture_output=True, text=True, timeout=60)
        assert "data race" not in p.stderr, p.stderr[:2000]
        assert p.returncode == 0 and p.stdout == "done\n", p.stderr[:2000]
