"""The helper behind the complex64 workspace: a set of buffers is had whole or not at all, also
when an earlier attempt failed half way (host code, compiled here with a counting allocator)."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1102_2143_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "alloc_all.h"

int main() {
  for (int fail = -1; fail < 4; ++fail) {
    int calls = 0, live = 0;
    void *p[4] = {nullptr, nullptr, nullptr, nullptr};
    auto get = [&](void** q, size_t b) {
      if (calls++ == fail) {
        *q = reinterpret_cast<void*>(8);  // what a failed call leaves is not looked at
        return 2;
      }
      *q = std::malloc(b);
      ++live;
      return 0;
    };
    auto put = [&](void* q) {
      std::free(q);
      --live;
    };
    for (int attempt = 0; attempt < 2; ++attempt) {  // the second one: a retry that succeeds
      const int e = msc::alloc_all({{&p[0], 16}, {&p[1], 1}, {&p[2], 8}, {&p[3], 64}}, get, put);
      const bool whole = p[0] && p[1] && p[2] && p[3];
      const bool none = !p[0] && !p[1] && !p[2] && !p[3];
      const bool failed = attempt == 0 && fail >= 0;
      if (e != (failed ? 2 : 0) || !(failed ? none : whole) || live != (failed ? 0 : 4)) {
        std::printf("fail=%d attempt=%d e=%d live=%d\n", fail, attempt, e, live);
        return 1;
      }
      if (!failed) break;
    }
  }
  return 0;
}
"""


def test_whole_or_none(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run([gxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


def test_complex64_workspace_goes_through_it():
    text = open(os.path.join(CSRC, "capi.cpp")).read()
    for name in ("ring32", "u32", "s32", "pk32"):
        assert not re.search(r"hipMalloc\(&w\.%s\b" % name, text), name
        assert re.search(r"\{&w\.%s," % name, text), name
