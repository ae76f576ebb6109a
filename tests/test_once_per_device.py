"""Work that is due once per GPU (csrc/once_per_device.h), run on the host: every device has its turn, a failure is
reported and tried again, and ordinals without a place are refused."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "once_per_device.h"
int main() {
  mdi::OncePerDevice once;
  int calls = 0;
  auto works = [&]() { ++calls; return true; };
  auto fails = [&]() { ++calls; return false; };
  const int order[] = {0, 0, 1, 0, 63, 1, 63};
  for (int device : order) std::printf("%d ", once.run(device, works));
  std::printf("%d ", calls);
  std::printf("%d ", once.run(5, fails));
  std::printf("%d ", once.run(5, works));
  std::printf("%d ", once.run(5, fails));
  std::printf("%d ", calls);
  std::printf("%d ", once.run(-1, works));
  std::printf("%d ", once.run(64, works));
  std::printf("%d\n", calls);
}
"""


def test_every_device_has_its_turn(tmp_path):
    src = tmp_path / "once.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "once")
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2505_18164_amd", "csrc"), str(src), "-o", exe], check=True)
    got = [int(v) for v in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()]
    assert got == [1] * 7 + [3] + [0, 1, 1] + [5] + [0, 0, 5]


def test_nothing_is_prepared_for_the_first_device_only():
    """Kernel attributes are set by functions that mdi_partition_create calls per device: no static or call_once around them."""
    csrc = os.path.join(ROOT, "paper_2505_18164_amd", "csrc")
    for name in sorted(os.listdir(csrc)):
        text = open(os.path.join(csrc, name)).read()
        assert "call_once" not in text, name
        assert not any("static" in line and "hip" in line and "=" in line for line in text.splitlines() if "hipFuncSetAttribute" in line or "hipGetDevice" in line), name
