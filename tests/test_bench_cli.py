"""bench.py's command line on the CPU: more than one GPU is refused with a
message (the multi-GPU split is a design note, not a path of this library)."""
import os
import re
import shutil
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bench_refuses_more_than_one_gpu():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120, cwd=ROOT)
    assert r.returncode == 2
    assert "one GPU" in (r.stdout + r.stderr)


def test_counters_are_of_the_built_kernel(tmp_path, monkeypatch):
    """The committed counters are reported only for the kernel source that they
    were taken on: a change of the kernel or of a header it includes drops them."""
    sys.path.insert(0, ROOT)
    import bench
    text = open(bench.KERNEL_SOURCES[0]).read()
    csrc = os.path.dirname(bench.KERNEL_SOURCES[0])
    names = [os.path.basename(f) for f in bench.KERNEL_SOURCES]
    included = [n for n in re.findall(r'#include "(\w+\.h)"', text) if os.path.exists(os.path.join(csrc, n))]
    assert names[0] == "attn_fwd.hip" and sorted(names[1:]) == sorted(included)
    copies = [str(tmp_path / n) for n in names]
    for src, dst in zip(bench.KERNEL_SOURCES, copies):
        shutil.copy(src, dst)
    monkeypatch.setattr(bench, "KERNEL_SOURCES", copies)
    taken = tmp_path / "counters.txt"
    taken.write_text(f"kernel_source_sha256_16: {bench.source_hash()}\nhbm_bytes_per_launch: 5\n"
                     "mfma_busy_fraction: 0.5\n")
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(taken))
    assert bench.measured_counters("ref5") == (5.0, 0.5)
    for f in copies:
        before = open(f).read()
        open(f, "a").write("// changed\n")
        assert bench.measured_counters("ref5") == (None, None), f
        open(f, "w").write(before)
    assert bench.measured_counters("ref5") == (5.0, 0.5)
