"""The ring of pinned staging slots (host code, no GPU): no slot is handed out while work that reads it may be running,
also after calls that ended in an error between taking a slot and giving it back, or whose event could not be recorded."""
from __future__ import annotations

import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_11517_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include <random>
#include "staging_ring.hpp"
// a stream that never gets on by itself: work enqueued runs only when somebody waits for it
int main(int argc, char** argv) {
  std::mt19937 rng((unsigned)atoi(argv[1]));
  pasta::StagingRing<8> ring;
  long clock = 0, done = 0, event[2] = {0, 0}, reader[8] = {};  // time of the last reader enqueued per slot
  int waits = 0, drains = 0;
  for (int call = 0; call < 4000; ++call) {
    int s = -1;
    const bool fail_wait = rng() % 50 == 0;
    if (!ring.take(&s, [&](int half) { if (fail_wait) return false; ++waits; if (event[half] > done) done = event[half]; return true; },
                   [&] { if (fail_wait) return false; ++drains; done = clock; return true; })) continue;
    if (reader[s] > done) { std::printf("call %d: slot %d is still being read\n", call, s); return 1; }
    const int how = (int)(rng() % 10);
    if (how == 0) continue;           // an error before anything was enqueued
    reader[s] = ++clock;
    if (how == 1) continue;           // ... and after it was
    ring.give([&](int half) { if (how == 2) return false; event[half] = ++clock; return true; });
  }
  std::printf("%d waits %d drains\n", waits, drains);
  return waits > 400 && drains > 400 ? 0 : 2;
}
"""


@pytest.mark.parametrize("seed", range(3))
def test_slots_are_not_reused_under_their_readers(tmp_path, seed):
    src, exe = tmp_path / "ring.cpp", tmp_path / "ring"
    src.write_text(PROGRAM.replace("#include <cstdio>", "#include <cstdio>\n#include <cstdlib>"))
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe), str(seed)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
