"""The walk over the key tiles of a chunked prefix (KvWalk), compiled for the host, against 64-bit positions worked out afresh
for every tile: ordinary chunk lists, and chunks of more rows than 31 bits count."""
import subprocess

from paper_2504_14519_amd.build import CSRC, HIPCC

PROGRAM = r"""
#include <stdio.h>
#include "tile_common.hpp"
using namespace slimpipe;

// every tile of keys [key0, key_end): address and rows of the walk against the definition; -> tiles that differ
static long long walk(int64_t len, int n, int tile, int64_t key0, int64_t key_end, int64_t stride, int64_t head_off) {
  static const bf16_t* table[kMaxChunks];
  KvChunks kv = {};
  kv.len = len;
  kv.n = n;
  for (int i = 0; i < n; ++i) table[i] = reinterpret_cast<const bf16_t*>((uintptr_t)1 << 56) + (int64_t)i * ((int64_t)1 << 48);   // never dereferenced
  KvWalk w;
  w.seek(table, kv, n > 1 ? (int)(key0 / len) : 0, key0, head_off, stride);
  long long bad = 0;
  for (int64_t t = 0, key = key0; key < key_end; ++t, key += tile) {
    const int c = n > 1 ? (int)(key / len) : 0;
    const int64_t row = key - c * len, left = len - row;
    bad += w.ptr != table[c] + head_off + row * stride;
    bad += w.chunk != c;
    bad += w.rows(tile) != (left < tile ? (int)left : tile);
    if (key + tile < key_end) w.step(table, kv, tile, tile * stride, head_off, stride, [&] { return key + tile; });
  }
  return bad;
}

int main() {
  const int64_t big = (int64_t)1 << 31;
  long long bad = 0;
  for (int tile : {64, 128}) {
    for (int64_t len : {1, 63, 64, 127, 128, 129, 777, 4096, 33777})
      for (int64_t key0 : {(int64_t)0, len / 2, len - 1}) bad += walk(len, 1, tile, key0, len, 128, 640);
    for (int64_t len : {256, 512, 4096})
      for (int n : {2, 3, 64})
        for (int64_t key0 : {(int64_t)0, len - tile, len, 2 * len - tile}) bad += walk(len, n, tile, key0, n * len - 5, 1024, 64);
  }
  printf("ordinary chunks: %lld\n", bad);
  bad = 0;
  for (int64_t len : {big - 129, big - 1, big, big + 1, 2 * big + 777, 5 * big + 130})           // one chunk, around every 2^31 rows
    for (int64_t key0 = 0; key0 < len; key0 += big)
      for (int64_t back : {0, 1, 1000}) {
        const int64_t a = key0 < back ? 0 : key0 - back;
        bad += walk(len, 1, 128, a, a + 3000 < len ? a + 3000 : len, 64, 64);
        const int64_t z = len - 3000 - back;
        bad += walk(len, 1, 128, z, len, 64, 64);
      }
  bad += walk(2 * big + 130, 1, 128, 77, 2 * big + 130, 64, 0);                                  // all of it, from the start
  bad += walk(big + 256, 2, 128, 128, 2 * big + 500, 64, 0);                                     // two chunks
  printf("chunks past 31 bits: %lld\n", bad);
  return 0;
}
"""


def test_walk_over_key_tiles(tmp_path):
    src, exe = str(tmp_path / "walk.hip"), str(tmp_path / "walk")
    with open(src, "w") as f:
        f.write(PROGRAM)
    r = subprocess.run([HIPCC, "--offload-host-only", "-O2", "-std=c++17", "-w", "-I", CSRC, src, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0
    assert r.stdout == "ordinary chunks: 0\nchunks past 31 bits: 0\n"
