"""What is set up once per device (csrc/per_device.h): the attention kernels'
LDS attribute, which belongs to the device that is current when it is set
(CPU only: the header is compiled alone)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_15650_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include <initializer_list>
#include "per_device.h"
int main() {
  ditango::OncePerDevice once;
  int calls[70] = {}, fail = 0;
  auto on = [&](int dev) { return once.run(dev, [&] { ++calls[dev]; return fail; }); };
  for (int i = 0; i < 3; ++i) for (int dev : {0, 1, 7, 63}) if (on(dev) != 0) return 1;
  for (int dev : {0, 1, 7, 63}) if (calls[dev] != 1) return 2;
  fail = 9;                                   // an error is returned and tried again
  if (on(2) != 9 || on(2) != 9 || calls[2] != 2 || on(0) != 0) return 3;
  fail = 0;
  if (on(2) != 0 || on(2) != 0 || calls[2] != 3) return 4;
  if (on(64) != 0 || on(64) != 0 || calls[64] != 2) return 5;   // not remembered: every time
  puts("ok");
}
"""


def test_once_per_device(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src = tmp_path / "t.cpp"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(tmp_path / "t")], check=True)
    assert subprocess.run([str(tmp_path / "t")], capture_output=True, text=True).stdout == "ok\n"


def test_kernel_attributes_are_set_per_device():
    """No attribute of a kernel is set by a static initialiser, which runs on
    whatever device comes first."""
    n = 0
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".hip", ".cpp", ".h")):
            text = open(os.path.join(CSRC, name)).read()
            for m in re.finditer(r"hipFuncSetAttribute", text):
                n += 1
                assert ".run(" in text[max(0, m.start() - 200):m.start()], name
    assert n == 2
