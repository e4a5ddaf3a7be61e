"""Arena blocks taken before their size is known (C++ model check, CPU)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_arena_front(tmp_path):
    exe = str(tmp_path / "arena_front_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-o", exe,
                           os.path.join(HERE, "arena_front_check.cpp")])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr
    assert "front ok" in out.stdout
