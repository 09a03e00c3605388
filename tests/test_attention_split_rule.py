"""The rule that gives the fused attention's waves their tokens, on the host: few tokens a wave for
small calls, but no more splits per head than the combine walks in the time they save."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <initializer_list>
#include <stdio.h>
#include "hq_internal.h"
int main() {
  for (long spr : {1, 2, 4, 8, 16})
    for (long batch : {1, 2, 3, 16, 64, 512})
      for (int b = 0; b < 21; ++b)
        for (long t : {(1L << b) - 1, 1L << b, (1L << b) + 1, 3L << b})
          if (t > 0) printf("%ld %ld %ld %ld\n", spr, batch, t, (long)hq_attn_chunk(spr, batch, t));
}
"""


def test_splits_per_head(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2606_23406_amd", "csrc"),
                    "-o", str(exe), str(src)], check=True, timeout=120)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.split("\n")
    rows = [tuple(int(v) for v in line.split()) for line in lines if line]
    assert len(rows) > 2000
    for spr, batch, tokens, chunk in rows:
        even = -(-batch * spr * tokens // 16384)
        assert 4 <= chunk <= 1024 and (chunk <= max(16, even))
        assert chunk >= min(1024, even)  # no more waves than the call wants
        splits = -(-tokens // (4 * chunk))
        assert splits <= max(512, -(-tokens // 64)), (spr, batch, tokens, chunk)
        if tokens <= 8192 and even <= 4:
            assert chunk == 4
