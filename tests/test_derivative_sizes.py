"""Sizes of the thickness-derivative buffers over a plan's geometries (host
arithmetic of csrc/derivative_sizes.hpp, compiled here without HIP)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_1910_07054_amd", "csrc")


def _run(tmp_path, body: str) -> list[int]:
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src = tmp_path / "t.cpp"
    src.write_text('#include <cstdio>\n#include "derivative_sizes.hpp"\nusing namespace hfd;\n'
                   "int main() {\n" + body + "\nreturn 0; }\n")
    exe = tmp_path / "t"
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return [int(x) for x in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()]


# (tables, most offsets of a table) of successive geometries.  The first row: 16
# stacks of 256 x 256 x 10 that differ in the last layer, then 16 unrelated ones,
# whose offsets fill more tables of the same length.
RESETS = [
    [(2, 166), (6, 166)],
    [(1, 41), (3, 41), (1, 41)],
    [(3, 41), (2, 50), (4, 30), (12, 11)],
    [(1, 5), (1, 5), (1, 4)],
]


@pytest.mark.parametrize("resets", RESETS, ids=str)
def test_offset_tables_fit_after_every_reset(tmp_path, resets):
    """Every geometry's tables, at the stride of the spectra, lie inside what is
    allocated, and neither size shrinks."""
    body = "DerivativeSizes s;\n" + "".join(
        f's = derivative_sizes(s, {t}, {n}); printf("%d %lld\\n", s.slots, s.offsets);\n' for t, n in resets)
    out = _run(tmp_path, body)
    slots = offsets = 0
    for k, (t, n) in enumerate(resets):
        assert out[2 * k] >= max(n, slots)
        assert out[2 * k + 1] >= max(t * out[2 * k], offsets)
        slots, offsets = out[2 * k], out[2 * k + 1]


# (slots, Ly / 2 + 1, bytes per value): whether one row and whether two rows lie
# within 2 GiB; 21835 slots of 2049 FP32 values pass 1 GiB, 43670 pass 2 GiB
ROWS = [(21834, 2049, 4, 1, 1), (21835, 2049, 4, 1, 0), (43669, 2049, 4, 1, 0), (43670, 2049, 4, 0, 0),
        (10917, 2049, 8, 1, 1), (10918, 2049, 8, 1, 0), (10, 5, 4, 1, 1), (1 << 30, 2049, 8, 0, 0)]


def test_rows_of_the_spectra_within_a_descriptor(tmp_path):
    body = "".join(f'printf("%d %d\\n", (int)derivative_rows_fit(1, {s}, {q}, {b}), '
                   f'(int)derivative_rows_fit(2, {s}, {q}, {b}));\n' for s, q, b, _, _ in ROWS)
    out = _run(tmp_path, body)
    assert out == [v for r in ROWS for v in r[3:]]
    for s, q, b, one, two in ROWS:
        assert (6 * s * q * b < 2**31, 12 * s * q * b < 2**31) == (bool(one), bool(two))
