"""The pass plans of the FP64 tube transforms, from the library's host code."""
import functools
import shutil
import subprocess

from paper_2005_09838_amd import _build

PROGRAM = r'''
#include <cstdio>
#include "fft64_plan.h"
int main() {
  for (int n = 1; n <= 8192; ++n) {
    const tctf::Fft64Plan p = tctf::fft64_plan(n);
    printf("%d", p.n);
    for (int k = 0; k < p.passes; ++k) printf(" %d", p.radix[k]);
    printf("\n");
  }
}
'''


@functools.lru_cache(None)
def _best(n, cap=12):
    """(passes, largest radix) of the best plan of a product of 2, 3, 5 and 7."""
    if n == 1:
        return (0, 0)
    found = [(1 + _best(n // r, r)[0], r) for r in (12, 10, 9, 8, 7, 6, 5, 4, 3, 2)
             if r <= cap and n % r == 0 and _best(n // r, r)]
    return min(found) if found else None


def test_fewest_passes_then_the_smallest_largest_radix(tmp_path):
    cc = shutil.which("g++") or _build.hipcc()
    (tmp_path / "plans.cpp").write_text(PROGRAM)
    exe = tmp_path / "plans"
    subprocess.run([cc, "-O1", "-std=c++17", "-I", _build.CSRC, str(tmp_path / "plans.cpp"), "-o", str(exe)], check=True)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()
    assert len(lines) == 8192
    for n, line in enumerate(lines, 1):
        got, *radices = map(int, line.split())
        product = 1
        for r in radices:
            product *= r
        assert got == n and product == n, (n, radices)
        primes = [r for r in radices if r > 7 and all(r % d for d in (2, 3, 5, 7))]
        small = [r for r in radices if r not in primes]
        assert all(p % d for p in primes for d in range(2, int(p**0.5) + 1)), (n, radices)
        assert set(small) <= {2, 3, 4, 5, 6, 7, 8, 9, 10, 12}, (n, radices)
        m = n
        for p in primes:
            m //= p
        assert (len(small), max(small, default=0)) == _best(m), (n, radices)
