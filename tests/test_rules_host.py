"""Rules of the kernels' launches that are plain functions, compiled for the host."""
import math
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


def evaluate_list(tmp_path, includes, expression, values):
    """The values of one C++ expression for every tuple x of `values`."""
    rows = ", ".join("{" + ", ".join(map(str, v)) + "}" for v in values)
    source = "".join(f'#include "{name}"\n' for name in includes)
    source += f"#include <cstdio>\nusing namespace surel;\nstatic const int all[][{len(values[0])}] = {{{rows}}};\n"
    source += f'int main() {{ for (auto& x : all) printf("%lld\\n", (long long)({expression})); }}\n'
    (tmp_path / "list.cpp").write_text(source)
    subprocess.run(["g++", "-O0", "-std=c++17", "-I" + CSRC, "-o", str(tmp_path / "list"),
                    str(tmp_path / "list.cpp")], check=True)
    out = subprocess.run([str(tmp_path / "list")], capture_output=True, text=True, check=True).stdout
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


def test_every_slot_of_a_set_is_reached_from_every_other(tmp_path):
    # ids that meet go on in steps that no number of slots may have a factor in common with; the set holds all
    # nodes of a seed's walks, and a workgroup's four fit a compute unit's LDS
    sizes = [(M, m) for m in range(1, 16) for M in range(1, 2048 // (m + 1) + 1)]
    steps = evaluate(tmp_path, ["walk_table.h"], [f"kDistinctSteps >> {8 * i} & 0xFF" for i in range(4)])
    slots = evaluate_list(tmp_path, ["walk_table.h"], "walk_table(x[0], x[1]).slots", sizes)
    for (M, m), s in zip(sizes, slots, strict=True):
        assert s % 64 == 0 and 1 + M * m < s and max(steps) < s
        assert s <= 64 * 64, (M, m)
        assert all(math.gcd(s, step) == 1 for step in steps)
        assert 4 * (2 * 64 * (m + 1) + s) * 4 <= 160 * 1024
