"""The rule that gives a block-scaled product its workgroup tile, on the host: the least rounds weighted
by a round's time, the 256 x 128 tile among the choices where one round of it replaces two of 128 x 128."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <initializer_list>
#include <stdio.h>
#include "hq_internal.h"
int main() {
  for (int mode : {0, 1, 2})
    for (int lng : {0, 1})
      for (long M : {1, 64, 129, 384, 500, 768, 1000, 1024, 1100, 1500, 2000, 2049, 4096, 8192, 100000})
        for (long N : {1, 130, 500, 1024, 2050, 4096, 6144, 8192, 11008, 14336, 128256})
          printf("%d %d %ld %ld %d\n", mode, lng, M, N, (int)hq_gemm_tile_of(mode, lng && mode != 2, M, N));
}
"""


def test_tile_is_the_cheapest(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2606_23406_amd", "csrc"),
                    "-o", str(exe), str(src)], check=True, timeout=120)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    rows = [tuple(int(v) for v in line.split()) for line in out.split("\n") if line]
    sizes = [(64, 64), (128, 128), (256, 128), (256, 256)]
    seen = set()
    for mode, lng, M, N, t in rows:
        tiles = [-(-M // a) * -(-N // b) for a, b in sizes]
        seen.add((mode, lng and mode != 2, t))
        if tiles[0] <= 512:
            assert t == 0
            continue
        weights = [99, 8, 13 if mode == 2 else 12, 19 if mode == 2 or not lng else 99]
        cost = [w * -(-n // 256) for w, n in zip(weights, tiles)]
        assert t > 0 and cost[t] == min(cost[1:])
        assert all(cost[u] > cost[t] for u in range(t + 1, 4))
    assert len(seen) == 4 * 3 + 3 * 2
    chosen = {r[:4]: r[4] for r in rows}
    for mode in (0, 1, 2):  # one round instead of two
        for M, N in ((500, 14336), (768, 6144), (768, 8192), (1000, 6144), (384, 11008)):
            assert chosen[mode, 0, M, N] == 2
