"""The words that the surrogate's kernel reads ahead of its weights lie inside them, wherever
they start and end (CPU: host code, compiled from the header that the kernel includes)."""
import os
import subprocess

import pytest

from paper_2503_12749_amd import build

PROGRAM = r"""
#include "common.h"
#include <cstdio>
int main() {
  // a buffer on any byte, in the middle of memory that is not read: addresses only
  for (int shift = 0; shift < 256; ++shift)
    for (int64_t bytes = 0; bytes < 700; ++bytes) {
      const char *p = (const char*)(uintptr_t)(4096 + shift), *q;
      int64_t i = 0, after = (int64_t)(uintptr_t)p;  // first byte whose line is not touched yet
      for (; (q = mp::touch_word(p, bytes, i)) != nullptr; ++i) {
        if ((uintptr_t)q % 4 != 0 || q < p || q + 4 > p + bytes) {
          std::printf("word at %td of %lld bytes on %d\n", q - p, (long long)bytes, shift);
          return 1;
        }
        if ((int64_t)((uintptr_t)q / 128) > (after + 3) / 128) return 2;  // a line left out
        after = ((int64_t)(uintptr_t)q / 128 + 1) * 128;
      }
      if (bytes >= 7 && i == 0) return 3;
    }
  return 0;
}
"""


def test_touched_words_lie_in_the_buffer(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    src = tmp_path / "touch.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "touch"
    subprocess.run([build.HIPCC, "-O1", "-std=c++17", f"--offload-arch={build.ARCH}", "-I", build.CSRC,
                    str(src), "-o", str(exe)], check=True, stderr=subprocess.DEVNULL)
    run = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert run.returncode == 0, run.stdout
