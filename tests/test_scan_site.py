"""Forward progress and bookkeeping of the look-back scans' block shares (C++
model check, CPU)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_scan_site(tmp_path):
    exe = str(tmp_path / "scan_site_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", "-o", exe,
                           os.path.join(HERE, "scan_site_check.cpp")])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr
    assert "scan ok" in out.stdout
