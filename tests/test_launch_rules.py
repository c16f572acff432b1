"""The rules that choose a launch shape from sizes (csrc/launch_rules.h), compiled by themselves on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(not shutil.which("g++"), reason="no g++")


def evaluate(tmp_path, expressions):
    """Values of C++ expressions over the header, as integers."""
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    lines = "\n".join(f'    std::printf("%lld\\n", (long long)({e}));' for e in expressions)
    src.write_text('#include <cstdio>\n#include "launch_rules.h"\nusing namespace cams;\nint main()\n{\n' + lines + "\n}\n")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2111_00705_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], check=True, stdout=subprocess.PIPE, text=True).stdout
    return [int(x) for x in out.split()]


def test_quarter_tile_update_only_where_the_lists_are_short(tmp_path):
    cases = {(1, 320): 1, (1, 321): 0, (16, 320): 1, (17, 320): 0, (20, 256): 1, (32, 160): 1, (32, 161): 0, (32, 288): 0,
             (64, 80): 1, (64, 128): 0, (65535, 1): 0, (65535, 524288): 0}
    got = evaluate(tmp_path, [f"short_final({n}, {tiles})" for n, tiles in cases])
    assert got == list(cases.values())
