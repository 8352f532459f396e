"""How the subspace calls' expand kernel shares its tiles (csrc/launch_rules.h), compiled by itself (no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_expand_rules(tmp_path):
    exe = str(tmp_path / "expand_rules")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Werror", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "paper_2601_02360_amd", "csrc"),
                    os.path.join(ROOT, "tests", "expand_rules_main.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120,
                         env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout + out.stderr
