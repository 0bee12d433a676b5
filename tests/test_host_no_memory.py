"""An allocation that fails inside append_kv comes back as E_NOMEM with the handle unchanged, wherever it is: the library's
operator new is replaced by one that refuses a given size (CPU; a process of its own)."""
from __future__ import annotations

import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NEW = r"""
#include <cstdlib>
#include <new>
static size_t refused = 0;
extern "C" void refuse(size_t n) { refused = n; }
void* operator new(size_t n) { if (refused && n == refused) throw std::bad_alloc(); if (void* p = std::malloc(n ? n : 1)) return p; throw std::bad_alloc(); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
"""
PROGRAM = r"""
import ctypes, sys
new = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
new.refuse.argtypes = [ctypes.c_size_t]
import numpy as np
from paper_2502_11517_amd import binding as B
FAKE = 0x7000_0000_0000
cfg = B.make_config("bf16", 4, 1, 128, 1.0, max_requests=2, pool_tokens=4096, max_ranges=8192)
h = B.PastaAttn(cfg, FAKE, FAKE, FAKE, B.query_workspace_bytes(cfg))
n = 1001  # alternating requests: a run per row, so that the rows' list is made
rid, sid = np.arange(n, dtype=np.int32) % 2, np.zeros(n, np.int32)
new.refuse(4 * n)
try:
    h.append_kv(0, rid, sid, FAKE, FAKE)
    print("no error")
except B.PastaError as e:
    print("code", e.code)
new.refuse(0)
print(h.append_kv(0, rid[:2], sid[:2], None, None, want_slots=True, flags=B.APPEND_RESERVE_ONLY).tolist())
"""


def test_the_list_of_destination_rows(tmp_path):
    lib = tmp_path / "refuse.so"
    (tmp_path / "refuse.cpp").write_text(NEW)
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", str(tmp_path / "refuse.cpp"), "-o", str(lib)], check=True)
    r = subprocess.run([sys.executable, "-c", PROGRAM, str(lib)], capture_output=True, text=True, cwd=ROOT, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split("\n")[:2] == ["code -3", "[0, 0]"], r.stdout
