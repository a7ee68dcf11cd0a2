"""The host code that asks for large dynamic LDS, compiled alone: each device is asked, and a refusal is not remembered."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))

MAIN = r"""
#include "lds_grant.h"
#include <stdio.h>
int main()
{
    hb::LdsGrant g;
    int asked = 0;
    auto yes = [&]() { ++asked; return 0; };
    auto no = [&]() { ++asked; return 7; };
    auto step = [&](int rc) { printf("%d:%d ", rc, asked); asked = 0; };
    step(g.ensure(0, 70000, yes));
    step(g.ensure(0, 70000, yes));
    step(g.ensure(1, 70000, yes));   // another device
    step(g.ensure(1, 100000, no));
    step(g.ensure(1, 100000, yes));  // refused before
    step(g.ensure(0, 100000, yes));
    step(g.ensure(1, 90000, yes));
    step(g.ensure(64, 5, yes));      // beyond the table
    step(g.ensure(64, 5, yes));
    return 0;
}
"""


def test_each_device_is_asked_for_its_lds(tmp_path):
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(MAIN)
    inc = os.path.join(HERE, "..", "paper_2004_08771_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-I", inc, str(src), "-o", str(exe), "-pthread"])
    assert subprocess.check_output([str(exe)], text=True).split() == [
        "0:1", "0:0", "0:1", "7:1", "0:1", "0:1", "0:0", "0:1", "0:1"]
