"""Which tile a workgroup of a product works on (tile_index)."""
import subprocess

from launches import program

SOURCE = r"""
#include <cstdio>
#include "common.h"
int main() {
  for (int total = 1; total <= 1300; total += total < 520 ? 1 : 37) {
    printf("%d", total);
    for (int vb = 0; vb < (total + 255) / 256 * 256; ++vb) printf(" %d", fc::tile_index(vb, total));
    printf("\n");
  }
}
"""


def test_every_tile_once_and_how_a_last_round_is_dealt_out(tmp_path):
    for line in subprocess.run([program(tmp_path, SOURCE)], check=True, capture_output=True, text=True).stdout.splitlines():
        total, *tiles = map(int, line.split())
        assert sorted(t for t in tiles if t < total) == list(range(total))
        for first in range(0, len(tiles), 256):
            shares = [[t for t in tiles[first + xcd:first + 256:8] if t < total] for xcd in range(8)]
            assert all(s == list(range(s[0], s[0] + len(s))) for s in shares if s)          # consecutive tiles in an XCD
            left = min(total - first, 256)
            assert max(map(len, shares)) == -(-left // 8)                                   # an eighth of the round each
