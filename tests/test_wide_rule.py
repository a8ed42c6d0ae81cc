"""The rule that chooses the kernel of the wide network's 16-bit step, against
what both kernels were measured to take on 256 compute units (CPU: the rule is
plain host code)."""
import os
import shutil
import subprocess

import pytest

from paper_2403_18466_amd import build

# batch, nx, ny, nz, us per step by row items, by blocks (bf16, unforced)
MEASURED = [
    (1, 16, 16, 16, 28.8, 8.8), (1, 28, 28, 28, 55.0, 12.0), (1, 32, 32, 32, 29.4, 12.5),
    (1, 40, 40, 40, 30.7, 21.9), (1, 44, 44, 44, 60.2, 31.0), (1, 48, 48, 48, 62.7, 35.0),
    (1, 52, 52, 52, 64.3, 44.4), (1, 56, 56, 56, 64.2, 53.8), (1, 60, 60, 60, 62.7, 68.3),
    (1, 64, 64, 64, 64.7, 79.1), (1, 96, 64, 64, 128.7, 119.8), (2, 62, 62, 62, 123.7, 143.7),
    (1, 72, 72, 72, 188.2, 112.2), (1, 80, 80, 80, 214.7, 155.2), (1, 128, 128, 128, 490.5, 632.8),
    (1, 117, 150, 131, 623.6, 687.3), (1, 148, 148, 148, 1016.2, 971.9),
    (1, 152, 152, 152, 1040.6, 1053.7),
    (1, 256, 256, 1, 27.7, 20.9), (2, 256, 256, 1, 30.4, 38.1), (4, 200, 300, 1, 83.2, 67.2),
    (1, 333, 333, 1, 55.6, 32.4), (1, 400, 400, 1, 57.0, 46.7), (1, 500, 500, 1, 57.6, 71.9),
    (1, 4000, 31, 1, 55.6, 38.1), (64, 64, 33, 1, 57.0, 40.4), (1, 1024, 1024, 1, 224.9, 281.7),
    (1, 1111, 777, 1, 200.5, 234.7),
]


def test_the_faster_kernel_is_chosen(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    calls = "".join(f"  std::printf(\"%d\\n\", (int)lbm::wide_by_blocks({b}, {nx}, {ny}, {nz}, 256));\n"
                    for b, nx, ny, nz, _, _ in MEASURED)
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text('#include <cstdio>\n#include "wide_rule.hpp"\nint main() {\n' + calls + "}\n")
    subprocess.run([cxx, "-std=c++17", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    chosen = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    slower = [c for c, blocks in zip(MEASURED, chosen) if (blocks == "1") != (c[5] < c[4])]
    assert not slower, slower


def test_gradient_ranges(tmp_path):
    """The 16-bit adjoint's node ranges, from one workgroup of nodes to beyond
    any grid: they cover every step, their number is a multiple of eight where it
    exceeds eight, no float32 sum runs over more nodes than 5,120 or, on the
    largest grids, than a 128th of all (the lengths of the chain of products
    that the kernel replaced), and the workspace is the records and the slabs."""
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    sizes = sorted({max(64, int(64 * 1.13 ** k) // 64 * 64) for k in range(120)} |
                   {32768, 73344, 73408, 327680, 327744, 373248, 655360})
    src, exe = tmp_path / "ranges.cpp", tmp_path / "ranges"
    src.write_text("""#include <cstdio>
#include <initializer_list>
#include "wide_rule.hpp"
int main() {
  for (long long Np : {%s}) {
    const lbm::WideAdjRanges r = lbm::wide_adj_ranges(Np);
    std::printf("%%lld %%d %%d %%lld\\n", Np, r.per, r.nsplit, lbm::wide_adj_workspace_bytes(Np));
  }
}
""" % ", ".join(f"{n}LL" for n in sizes))
    subprocess.run([cxx, "-std=c++17", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    assert len(out.splitlines()) == len(sizes)
    for line in out.splitlines():
        Np, per, nsplit, nbytes = map(int, line.split())
        assert per >= 1 and per * nsplit >= Np // 32, line
        assert 1 <= nsplit <= 128 and (nsplit <= 8 or nsplit % 8 == 0), line
        assert 32 * per <= max(5120, (Np // 32 + 127) // 128 * 32), line
        assert nbytes == 3200 * Np + 546 * 1024 * nsplit, line
