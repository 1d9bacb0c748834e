"""The library's host-side rules on the CPU: tests/host_rules/host_rules.hip,
compiled for the host only (it calls no HIP function) with undefined behaviour
trapped, against the library's internal header."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_host_rules(tmp_path):
    import sys
    sys.path.insert(0, ROOT)
    from paper_2505_08098_amd import build as lib_build
    exe = tmp_path / "host_rules"
    subprocess.run([lib_build.hipcc(), "-O1", "-std=c++17", "-Wall", "--offload-host-only",
                    "-Xarch_host", "-fsanitize=undefined",
                    "-Xarch_host", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2505_08098_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host_rules", "host_rules.hip"),
                    "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
    assert res.stdout.split("\n")[-2] == "ok"
