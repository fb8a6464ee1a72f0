"""Whether two strided tensors can share memory (Span in kernels.hpp, compiled for the host): never "no" where an element of one overlaps
an element of the other, and "no" for tensors one behind the other, down to the last byte."""
import subprocess

from paper_2504_14519_amd.build import CSRC, HIPCC

PROGRAM = r"""
#include <stdio.h>
#include <set>
#include "kernels.hpp"
using namespace slimpipe;

struct Tensor { int64_t first, bytes, b, s, h, d, sb, ss, sh; };
static Span span(const Tensor& t) { return span_of(reinterpret_cast<const void*>((uintptr_t)(1 << 20) + t.first), t.bytes, t.b, t.s, t.h, t.d, t.sb, t.ss, t.sh); }
static std::set<int64_t> memory(const Tensor& t) {
  std::set<int64_t> m;
  for (int64_t b = 0; b < t.b; ++b) for (int64_t s = 0; s < t.s; ++s) for (int64_t h = 0; h < t.h; ++h) for (int64_t d = 0; d < t.d; ++d)
    for (int64_t i = 0; i < t.bytes; ++i) m.insert(t.first + (b * t.sb + s * t.ss + h * t.sh + d) * t.bytes + i);
  return m;
}

int main() {
  int missed = 0, ends = 0, behind = 0;
  for (int64_t elem : {2, 4})
    for (int64_t b : {1, 2})
      for (int64_t s : {1, 3})
        for (int64_t h : {1, 2})
          for (int64_t pad : {0, 8})
            for (int64_t batch_gap : {0, 40}) {
              Tensor t{4096, elem, b, s, h, 16, s * (h * 16 + pad) + batch_gap, h * 16 + pad, 16};
              const std::set<int64_t> m = memory(t);
              const int64_t base = 1 << 20, lo = *m.begin(), hi = *m.rbegin() + 1;
              ends += span(t).begin != (uintptr_t)(base + lo) || span(t).end != (uintptr_t)(base + hi);
              for (int64_t elem2 : {2, 4})
                for (int64_t at = lo - 300; at <= hi + 16; at += 16) {
                  Tensor u{at, elem2, 1, 2, 1, 16, 64, 24, 16};
                  bool shared = false;
                  for (int64_t x : memory(u)) shared |= m.count(x) != 0;
                  missed += shared && (!share_memory(span(t), span(u)) || !share_memory(span(u), span(t)));
                }
              Tensor next{hi, 4, 1, 1, 1, 8, 8, 8, 8}, none{lo, 4, 1, 0, 1, 8, 8, 8, 8};
              behind += share_memory(span(t), span(next)) || share_memory(span(next), span(t)) || share_memory(span(t), span(none));
            }
  printf("missed %d ends %d behind %d\n", missed, ends, behind);
  return 0;
}
"""


def test_spans_that_share_memory(tmp_path):
    src, exe = str(tmp_path / "spans.hip"), str(tmp_path / "spans")
    with open(src, "w") as f:
        f.write(PROGRAM)
    r = subprocess.run([HIPCC, "--offload-host-only", "-O2", "-std=c++17", "-w", "-I", CSRC, src, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0
    assert r.stdout == "missed 0 ends 0 behind 0\n"
