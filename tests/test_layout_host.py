"""The index arithmetic of csrc/layout.hpp that kernels and launchers share, compiled for
the host under the undefined-behaviour sanitizer and run at the ends of its range."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_07508_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no C++ compiler")


def run(tmp_path, body):
    src = tmp_path / "layout.cpp"
    src.write_text('#include <cstdio>\n#include "layout.hpp"\nusing namespace sao;\nint main() {\n' + body + "\n}\n")
    exe = tmp_path / "layout"
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
           "-I", CSRC, str(src), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_step_chunks_cover_every_step_once(tmp_path):
    """Up to 2^30 steps (2^31 tokens, every other one in the loss mask) and 1024 threads."""
    run(tmp_path, """
  const int ns[] = {0, 1, 2, 255, 256, 257, 1000, 65536, (1 << 29) - 1, 1 << 29, 537000001, (1 << 30) - 512, 1 << 30};
  for (int n : ns) {
    if (step_chunk_begin(n, 0) != 0 || step_chunk_begin(n, kStepChunks) != n) return 1;
    for (int i = 0; i < 1024; ++i) {
      const int p = step_chunk_begin(n, i), q = step_chunk_begin(n, i + 1);
      if (p < 0 || q < p || q > n || q - p > step_chunk_len(n)) return 2;
      if (i >= kStepChunks && p != n) return 3;
      const int64_t chunks = step_chunk_len(n) > 0 ? (int64_t{n} + step_chunk_len(n) - 1) / step_chunk_len(n) : 0;
      if ((p < q) != (i < chunks)) return 4;
    }
  }
  return 0;""")
