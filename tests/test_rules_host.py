"""Rules of the kernels' launches that are plain functions, compiled for the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2202_13538_amd", "csrc")


def evaluate(tmp_path, includes, expressions):
    """The values of C++ expressions (integers), with the given headers of csrc/ included."""
    if shutil.which("g++") is None:
        pytest.skip("no host compiler here")
    source = "".join(f'#include "{name}"\n' for name in includes)
    source += "#include <cstdio>\nusing namespace surel;\nint main() {\n"
    source += "".join(f'printf("%lld\\n", (long long)({e}));\n' for e in expressions) + "}\n"
    (tmp_path / "main.cpp").write_text(source)
    subprocess.run(["g++", "-O0", "-std=c++17", "-I" + CSRC, "-o", str(tmp_path / "main"),
                    str(tmp_path / "main.cpp")], check=True)
    out = subprocess.run([str(tmp_path / "main")], capture_output=True, text=True, check=True).stdout
    return [int(x) for x in out.split()]


def test_rounds_of_the_join_lie_in_the_lines_of_outputs_that_start_anywhere(tmp_path):
    # ids and vectors that start the same number of rows behind a line both lie in lines; vectors that
    # start elsewhere lie in lines if any place of a round does that
    line, rows = 128, 32
    cases = []
    for row_bytes in sorted({2 * k * L for k in (2, 3) for L in range(2, 17)} | {12}):
        for skip in range(rows + 1):
            cases.append((4 * skip, row_bytes * skip, row_bytes))
        cases += [(0, 3 * row_bytes, row_bytes), (5 * 4, 0, row_bytes), (4, 2, row_bytes), (8, 4, row_bytes)]
    base = 1 << 40
    places = evaluate(tmp_path, ["lines.h"], [
        f"join_first_place((const void*){base + ids}ull, (const void*){base + cnt}ull, {b})"
        for ids, cnt, b in cases])
    for (ids, cnt, b), place in zip(cases, places, strict=True):
        assert 0 <= place < rows
        fits = [p for p in range(rows) if (cnt - p * b) % line == 0]
        if ids // 4 * b == cnt or not fits:
            assert place == ids // 4 % rows
        else:
            assert place in fits


def test_codes_that_the_memory_side_cache_holds_stay_in_the_caches(tmp_path):
    # pruning reads them back; half of the 256 MB are theirs
    half = (128 << 20) // 4
    rows = [0, 1, 8_400_000, half, half + 1, 146_000_000, 1 << 31]
    past = evaluate(tmp_path, ["lines.h"], [f"codes_go_past({n}ll)" for n in rows])
    assert past == [0, 0, 0, 0, 1, 1, 1]
