"""Which of two kernels a call takes (csrc/routes.h), compiled for the CPU: the calls whose two sides were measured, on a chip of 256 compute units.  No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    """Evaluates C++ expressions over csrc/routes.h: a list of them to the list of their values."""
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no host compiler")

    def values(expressions):
        d = tmp_path_factory.mktemp("routes")
        src, exe = d / "routes.cpp", d / "routes"
        src.write_text('#include "routes.h"\n#include <cstdio>\nusing namespace slim;\nint main() {\n'
                       + "".join(f'    printf("%d\\n", (int)({e}));\n' for e in expressions) + "}\n")
        subprocess.run([gxx, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2508_06447_amd", "csrc"), str(src), "-o", str(exe)], check=True)
        return [int(v) for v in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()]
    return values


def check(routes, cases):
    got = routes([e for e, _ in cases])
    assert [(e, v) for (e, _), v in zip(cases, got)] == [(e, int(w)) for e, w in cases]


def test_row_strides_that_only_the_few_row_tiles_take(routes):
    """The two-size launch refuses output rows of 2^23 elements and more: such a call stays where it is served."""
    check(routes, [(f"in_few_row_tiles({m}, {n}, 4096, {ldo}, {res}, true, 256)", ldo >= 1 << 23)
                   for m, n in ((64, 54016), (2048, 4096)) for res in ("false", "true") for ldo in (54016, (1 << 23) - 8, 1 << 23, 1 << 24)])


def test_residuals_that_the_two_size_launch_would_add_in_its_eight_wave_tile(routes):
    """Widths that are no multiple of 256 and residuals that are not aligned: only short rows leave the few-row tiles, with the four-wave tile long ones too."""
    shapes = ((1600, 4104), (1900, 3904), (2048, 4000), (3300, 2056), (1400, 5000), (640, 12104))
    check(routes, [(f"in_few_row_tiles({m}, {n}, {k}, {n}, true, {four}, 256)", four == "false" and k > 640)
                   for m, n in shapes for k in (256, 640, 1024, 4096, 14336) for four in ("false", "true")])


def test_residuals_of_short_rows(routes):
    """Fewer than 448 features: in the few-row tiles where these divide evenly over the XCDs in less than 15/16 of a round; fewer than 256: everywhere."""
    even, other = ((1665, 4096), (1792, 4096), (896, 8192), (768, 9216), (2300, 2880)), ((2048, 4096), (1408, 5120), (1920, 3840), (1500, 5120), (1400, 5000))
    check(routes, [(f"in_few_row_tiles({m}, {n}, {k}, {n}, true, {'true' if n % 256 == 0 else 'false'}, 256)",
                    k < 256 or ((m, n) in even and (k < 448 or n % 256 != 0)))
                   for m, n in even + other for k in (64, 192, 256, 384, 448, 512)])
    check(routes, [(f"in_few_row_tiles({m}, {n}, {k}, {n}, false, false, 256)", False) for m, n in even + other for k in (64, 256, 4096)])


def test_attention_that_would_begin_a_second_round_for_few_keys(routes):
    """(rows, query heads, kv heads): calls on both sides of the line, as measured, and what the few-row kernel does not cover."""
    few = ((512, 64, 8), (2048, 32, 8), (2048, 28, 4), (1024, 64, 16), (1024, 48, 16), (8192, 8, 1), (16384, 4, 1), (256, 128, 8), (256, 112, 16), (512, 96, 24), (504, 96, 8),
           (672, 96, 8), (280, 192, 16), (320, 192, 16), (160, 96 * 4, 96), (288, 56 * 4, 56), (320, 112, 28), (288, 90, 30))
    other = ((384, 112, 16), (320, 112, 16), (512, 112, 16), (384, 96, 32), (512, 128, 32), (384, 128, 8), (160, 256, 8), (192, 192, 16), (240, 192, 16), (640, 96, 24),
             (800, 80, 20), (352, 112, 28), (288, 128, 32), (2049, 32, 8), (2049, 28, 4))
    check(routes, [(f"few_row_attention({n}, {hq}, {hkv}, 0.1f, 256)", True) for n, hq, hkv in few]
          + [(f"few_row_attention({n}, {hq}, {hkv}, 0.1f, 256)", False) for n, hq, hkv in other]
          + [(f"few_row_attention(64, {hq}, 2, {scale}, 256)", False) for hq, scale in ((2, "0.1f"), (4, "0.1f"), (10, "0.1f"), (12, "0.f"), (8, "-0.1f"), (8, "__builtin_nanf(\"\")"))])


def test_compactions_that_select_their_blocks(routes):
    """(workgroups per block, kept, blocks): the small float32 layer's 6 (3 with blocks of 8 rows), and a bf16 layer of 4096 with folded gains and 64-row blocks, 161."""
    check(routes, [(f"compact_selects({chunks}, {keep}, {nb})", want) for chunks, keep, nb, want in (
        (6, 1, 2, True), (6, 16, 32, True), (6, 32, 64, True), (3, 63, 64, True), (6, 63, 64, False), (3, 1, 65, False), (161, 4, 16, True), (161, 8, 16, False),
        (161, 24, 47, False))])


def test_splits_of_the_output_projection(routes):
    check_values = ((1, 4096, 4), (64, 3584, 4), (65, 4096, 2), (128, 8192, 2), (129, 4096, 1), (256, 4096, 1), (257, 4096, 2), (512, 8192, 2), (513, 8192, 1), (1024, 4096, 2),
                    (1025, 4096, 1), (1024, 2048, 2), (1025, 2048, 1), (819, 5120, 2), (820, 5120, 1), (64, 1024, 1), (64, 16384, 1))
    assert routes([f"out_splits({m}, {n}, 4096)" for m, n, _ in check_values]) == [s for _, _, s in check_values]
