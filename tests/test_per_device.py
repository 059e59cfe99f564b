"""per_device.h: what is asked of the runtime is asked once on every device, and again after a refusal (host code, no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cassert>
#include "per_device.h"
int main()
{
    static cr::PerDevice p;
    int asked = 0;
    auto grant = [&] { ++asked; return true; };
    auto refuse = [&] { ++asked; return false; };
    assert(p.once(0, grant) && asked == 1);
    assert(p.once(0, refuse) && asked == 1);          // granted before
    assert(!p.once(1, refuse) && asked == 2);         // another device asks for itself, and a refusal is not kept
    assert(p.once(1, grant) && asked == 3 && p.once(1, refuse) && asked == 3);
    assert(p.once(63, grant) && p.once(63, grant) && asked == 4);
    assert(p.once(64, grant) && p.once(64, grant) && asked == 6 && !p.once(-1, refuse) && asked == 7);
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_once_on_every_device(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    build = subprocess.run(["g++", "-std=c++17", "-Wall", "-UNDEBUG", "-I", os.path.join(ROOT, "paper_2504_18082_amd", "csrc"), str(src), "-o", str(exe)],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    assert subprocess.run([str(exe)]).returncode == 0
