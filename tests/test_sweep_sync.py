"""The flags by which the extrapolation's blocks step through the sweeps, with
host threads for blocks: a flag that arrives with the last poll counts, a wait
for a missing block ends, and blocks that come late take part from the next
sweep, or end when the sweeps are over."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_flags_between_host_threads(tmp_path):
    exe = str(tmp_path / "sweep_sync_host")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-pthread", "-I",
                           os.path.join(ROOT, "paper_2604_14938_amd", "csrc"), "-o", exe,
                           os.path.join(ROOT, "tests", "sweep_sync_host.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
