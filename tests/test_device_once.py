"""What the launchers do once per device (leave for a kernel's dynamic LDS): a second device of the
process has it done too, a failure is tried again, and no launcher keeps a once-per-process flag."""
import glob
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_23317_amd", "csrc")

DRIVER = """
#include "device_once.h"
#include <cstdio>
#include <initializer_list>
int main() {
  static cfdetr::DeviceOnce once, other;
  int calls = 0, answer = 0;
  auto f = [&] { ++calls; return answer; };
  auto tell = [&](cfdetr::DeviceOnce& which, int device) {
    const int got = which.run(device, f);
    std::printf("%d:%d ", got, calls);
  };
  for (int device : {0, 0, 3, 0, 3, 63, 63}) tell(once, device);
  answer = 7;
  for (int i = 0; i < 2; ++i) tell(once, 5);
  answer = 0;
  for (int i = 0; i < 2; ++i) tell(once, 5);
  for (int i = 0; i < 2; ++i) tell(once, 64);
  tell(other, 0);
}
"""


def test_every_device_of_the_process(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    (tmp_path / "driver.cc").write_text(DRIVER)
    exe = str(tmp_path / "driver")
    subprocess.run([gxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(tmp_path / "driver.cc"), "-o", exe], check=True)
    got = subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split()
    assert got == ["0:1", "0:1", "0:2", "0:2", "0:2", "0:3", "0:3", "7:4", "7:5", "0:6", "0:6", "0:7", "0:8", "0:9"]


def test_no_launcher_goes_by_a_flag_of_the_process():
    for path in glob.glob(os.path.join(CSRC, "*.hip")):
        with open(path) as f:
            assert not re.search(r"\bstatic bool\s+\w+\s*=", f.read()), path


NUMBERS = """
#include "device_once.h"
#include <cstdio>
#include <initializer_list>
int main() {
  static cfdetr::DeviceNumber number;
  int calls = 0;
  auto tell = [&](int device, int answer) {
    const int got = number.get(device, [&] { ++calls; return answer; });
    std::printf("%d:%d ", got, calls);
  };
  for (int device : {0, 0, 3, 0, 3, 63, 63}) tell(device, 100 + device);
  for (int answer : {0, -1, 5, 6}) tell(7, answer);
  for (int device : {64, 64, -1}) tell(device, 9);
}
"""


def test_a_number_of_every_device(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    (tmp_path / "driver.cc").write_text(NUMBERS)
    exe = str(tmp_path / "driver")
    subprocess.run([gxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(tmp_path / "driver.cc"), "-o", exe], check=True)
    got = subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split()
    assert got == ["100:1", "100:1", "103:2", "100:2", "103:2", "163:3", "163:3", "0:4", "-1:5", "5:6", "5:6", "9:7", "9:8", "9:9"]


def test_no_launcher_goes_by_a_number_of_the_process():
    for path in glob.glob(os.path.join(CSRC, "*.hip")):
        with open(path) as f:
            assert not re.search(r"^\s+static (int|long|unsigned)\s+\w+\s*=", f.read(), re.M), path
