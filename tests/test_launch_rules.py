"""The launch rules that are plain arithmetic (csrc/launch_rules.h), compiled by themselves under AddressSanitizer and
UndefinedBehaviorSanitizer and checked by tests/launch_rules_main.cpp against what they promise (no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launch_rules(tmp_path):
    exe = str(tmp_path / "launch_rules")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Werror", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "paper_2601_02360_amd", "csrc"),
                    os.path.join(ROOT, "tests", "launch_rules_main.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120,
                         env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout + out.stderr
