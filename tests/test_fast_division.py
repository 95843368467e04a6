"""Division of node numbers by a row length through a multiplication, as the
step kernels do it: every divisor up to 4096 and others up to the largest, at
the multiples of the divisor and next to them, against integer division."""
import re
import subprocess
from pathlib import Path

SRC = Path(__file__).resolve().parent.parent / "paper_1206_0389_amd" / "csrc" / "kernels.h"

MAIN = r"""
#include <cstdint>
#include <cstdio>
#define __device__
#define __forceinline__ inline
static uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
%s
int main() {
  const uint64_t top = 0x7fffffffull;
  long long bad = 0;
  auto check = [&](uint32_t d) {
    FastDiv f;
    f.set(d);
    auto at = [&](uint64_t n) {
      if (n <= top && f((uint32_t)n) != (uint32_t)(n / d)) ++bad;
    };
    const uint64_t stride = top / d / 61 + 1;
    for (uint64_t k = 0; k * d <= top; k += stride) { at(k * d); at(k * d + 1); at(k * d + d - 1); }
    const uint64_t last = top / d * d;
    at(last); at(last - 1); at(top); at(top - 1);
    for (uint64_t n = 0; n < 300; ++n) at(n);
  };
  for (uint32_t d = 1; d <= 4096; ++d) check(d);
  for (uint64_t d = 4097; d <= top; d = d * 9 / 8 + 3) check((uint32_t)d);
  for (int b = 1; b < 31; ++b) { check(1u << b); check((1u << b) + 1); check((1u << b) - 1 ? (1u << b) - 1 : 1); }
  check((uint32_t)top);
  printf("%%lld\n", bad);
}
"""


def test_division_by_multiplication(tmp_path):
    struct = re.search(r"struct FastDiv \{.*?\n\};", SRC.read_text(), re.S).group(0)
    src = tmp_path / "d.cpp"
    src.write_text(MAIN % struct)
    subprocess.run(["g++", "-O2", "-std=c++17", "-o", str(tmp_path / "d"), str(src)], check=True)
    out = subprocess.run([str(tmp_path / "d")], check=True, capture_output=True, text=True).stdout
    assert out.strip() == "0"
