"""The rule by which the waits of a persistent kernel end (csrc/bounded_wait.h), run on the host: a wait that never sees
its word expires once, and the waits of the same workgroup that come after it end at their next look at the failure."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "bounded_wait.h"
int main() {
  const int limit = 1 << 21;
  bool failed = false;
  int expired = 0;
  auto wait = [&](int arrives) {                    // polls until the word is there or the wait ends
    int polls = 0;
    while (polls < arrives && mdi::may_poll_again(polls, limit, [&]() { return failed; }, [&]() { failed = true; ++expired; })) {}
    return polls;
  };
  std::printf("%d", wait(40));                      // an ordinary wait
  std::printf(" %d", wait(limit));                  // the longest that is allowed
  std::printf(" %d", expired);
  std::printf(" %d", wait(1 << 30));                // one that never sees its word
  for (int i = 0; i < 8; ++i) std::printf(" %d", wait(1 << 30));
  std::printf(" %d\n", expired);
}
"""


def test_waits_after_an_expired_one_end_at_once(tmp_path):
    src = tmp_path / "wait.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "wait")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2505_18164_amd", "csrc"), str(src), "-o", exe], check=True)
    got = [int(v) for v in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()]
    assert got[:4] == [40, 1 << 21, 0, (1 << 21) + 1]
    assert all(n <= 64 for n in got[4:12])
    assert got[12] == 1
