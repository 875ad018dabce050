"""The rule that lets a kernel address a population plane with 32-bit byte
offsets (offsets_fit), against the offsets themselves: a host program built
from the kernels' own header, no kernel is launched."""
import os
import subprocess

from paper_1110_0270_amd import build

SRC = r"""
#include <cstdint>
#include <cstdio>
#include "lbm_site.h"
using namespace lbm;
// the last element's byte offset survives 32 bits
template <class T> bool reaches(long long elems) {
  const uint32_t off = (uint32_t)(elems - 1) * (uint32_t)sizeof(T);
  return (unsigned long long)off == (unsigned long long)(elems - 1) * sizeof(T);
}
template <class T> int check(long long elems) {
  if (offsets_fit<T>(elems) == reaches<T>(elems)) return 0;
  std::printf("%lld elements of %d bytes: %d\n", elems, (int)sizeof(T), (int)offsets_fit<T>(elems));
  return 1;
}
int main() {
  int bad = 0;
  const long long around[] = {1ll << 20, 1ll << 29, 1ll << 30, 32832ll * 32768, 1ll << 31};
  for (long long e : around)
    for (long long d = -64; d <= 64; d += 1) bad += check<float>(e + d) + check<double>(e + d);
  return bad != 0;
}
"""


def test_offsets_fit_is_where_32_bits_reach(tmp_path):
    src, exe = tmp_path / "t.hip", tmp_path / "t"
    src.write_text(SRC)
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
