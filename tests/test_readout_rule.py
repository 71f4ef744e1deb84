"""Which device destinations a read-out writes with one kernel: aligned
outputs, each whole inside one allocation of the context's device, none
overlapping another.  The rule is compiled for the host and asked about
outputs of every other kind, which take the copies (no GPU needed)."""
import itertools
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_16623_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "wake_rows.h"
// per line: device n rows, then per row: pointer base size device
int main() {
  long long dev, n, rows;
  while (std::scanf("%lld %lld %lld", &dev, &n, &rows) == 3) {
    double* outs[6];
    OutMem mem[6];
    for (long long q = 0; q < rows; ++q) {
      unsigned long long p, b, z;
      long long d;
      if (std::scanf("%llu %llu %llu %lld", &p, &b, &z, &d) != 4) return 1;
      outs[q] = reinterpret_cast<double*>((uintptr_t)p);
      mem[q] = {(uintptr_t)b, (size_t)z, (int)d};
    }
    std::printf("%d\n", rows_by_kernel(outs, mem, (int)rows, (size_t)n, (int)dev) ? 1 : 0);
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "rows")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "main.cpp"), "-o", exe], check=True)

    def run(dev, n, rows):
        """rows: (pointer, allocation, its size, its device) each"""
        text = f"{dev} {n} {len(rows)}\n" + "".join(" ".join(str(x) for x in r) + "\n" for r in rows)
        return subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.strip() == "1"
    return run


A, SIZE = 1 << 40, 1 << 20       # an allocation


def test_apart_rows_of_one_device_take_the_kernel(ask):
    n = 1000
    rows = [(A + 8 * n * q, A, SIZE, 0) for q in range(6)]
    assert ask(0, n, rows)
    assert ask(0, n, [(A + SIZE - 8 * n, A, SIZE, 0)])          # up to the allocation's last byte
    for skip in itertools.product((0, 1), repeat=6):            # any of them left out
        assert ask(0, n, [r if k else (0, 0, 0, -1) for r, k in zip(rows, skip)])
    assert ask(3, n, [(A, A, SIZE, 3), (2 * A, 2 * A, SIZE, 3)])


@pytest.mark.parametrize("row", [
    (A, A, SIZE, 1),                          # another GPU's memory
    (A, 0, 0, -1),                            # host memory, or unknown
    (A + 4, A, SIZE, 0),                      # not aligned
    (A + SIZE - 8 * 1000 + 8, A, SIZE, 0),    # past the allocation's end
    (A - 8, A, SIZE, 0),                      # before it
    (A, A, 8 * 1000 - 8, 0),                  # an allocation too short
    (A + 2 * SIZE, A, SIZE, 0),               # outside it
])
def test_other_memory_takes_the_copies(ask, row):
    good = (4 * A, 4 * A, SIZE, 0)
    for rows in ([row], [good, row], [row, good], [(0, 0, 0, -1), row]):
        assert not ask(0, 1000, rows)


@pytest.mark.parametrize("shift", [0, 8, -8, 8 * 999, -8 * 999])
def test_overlapping_outputs_take_the_copies(ask, shift):
    p = A + SIZE // 2
    for rows in ([p, p + shift], [p + shift, p], [p, p + 8 * 4000, p + shift]):
        assert not ask(0, 1000, [(x, A, SIZE, 0) for x in rows])
    assert ask(0, 1000, [(p, A, SIZE, 0), (p + 8 * 1000, A, SIZE, 0)])
