"""Launch sizes and small work items of the learned step (CPU: the rules are
plain host code)."""
import shutil
import subprocess

import pytest

from paper_2403_18466_amd import build

# Q, H, fp32, forced, 16-node items per wavefront, us per step with 16-node items,
# with 64-node items (256 compute units)
MEASURED = [
    (9, 32, 1, 0, 2.0, 11.3, 10.5), (9, 32, 1, 1, 2.0, 12.0, 10.5), (9, 32, 0, 0, 2.0, 10.8, 9.6),
    (9, 32, 0, 1, 2.0, 9.4, 9.7), (9, 64, 1, 0, 2.0, 13.0, 15.4), (9, 64, 0, 0, 2.0, 12.3, 13.6),
    (9, 64, 0, 1, 2.0, 9.1, 13.9), (19, 32, 1, 0, 2.0, 10.9, 10.5), (19, 32, 1, 1, 2.0, 11.5, 10.8),
    (19, 32, 1, 0, 1.5, 9.6, 10.4), (19, 32, 0, 0, 2.0, 9.2, 11.2), (19, 32, 0, 1, 2.0, 9.9, 8.2),
    (19, 64, 0, 0, 2.0, 11.3, 15.9), (19, 64, 0, 1, 2.0, 11.8, 10.2), (19, 64, 1, 0, 1.5, 14.8, 17.7),
]


def run(tmp_path, body):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text('#include <cstdio>\n#include "step_rule.hpp"\nint main() {\n' + body + "}\n")
    subprocess.run([cxx, "-std=c++17", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    return [list(map(int, line.split())) for line in out.splitlines()]


def test_no_second_round_while_places_are_empty(tmp_path):
    """Workgroups of 4 to 16 wavefronts, one to three per compute unit: as many
    items per wavefront as the chip's places ask for, no more; a multiple of the
    eight XCDs beyond eight workgroups; never more than fit."""
    out = run(tmp_path, """
  for (int wb : {4, 8, 12, 16})
    for (int occ : {1, 2, 3})
      for (long long n = 1; n < 60000; n += 1 + n / 61)
        std::printf("%d %d %lld %u\\n", wb, occ, n, lbm::persistent_grid(256, occ, wb, n));
""".replace("{4, 8, 12, 16}", "(int[]){4, 8, 12, 16}").replace("{1, 2, 3}", "(int[]){1, 2, 3}"))
    assert len(out) > 1000
    for wb, occ, n, nb in out:
        places = 256 * occ * wb
        assert 1 <= nb <= 256 * occ and (nb <= 8 or nb % 8 == 0)
        assert -(-n // (nb * wb)) == -(-n // places), (wb, occ, n, nb)


def test_the_faster_items_are_taken(tmp_path):
    body = "".join(f'  std::printf("%d\\n", lbm::step_item_halves({q}, {h}, {s}, {f}));\n'
                   for q, h, s, f, *_ in MEASURED)
    for (q, h, s, f, items, t16, t64), (halves,) in zip(MEASURED, run(tmp_path, body)):
        assert (2 * items <= halves) == (t16 < t64), (q, h, s, f, items)
