"""The limits of the launches (csrc/launch_rules.hpp, plain host arithmetic),
compiled with the host compiler and compared with what the kernels' 32-bit
numbers and a launch's thread count allow, at the edges of their ranges."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_22099_amd", "csrc")


def run(tmp_path, body):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text('#include "launch_rules.hpp"\n#include <cstdio>\n#include <initializer_list>\nusing namespace bandlu;\n'
                   "typedef long long ll;\nint main() {\n" + body + "\n}\n")
    subprocess.run(["g++", "-std=c++20", "-Wall", "-Werror", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    return [[int(v) for v in line.split()] for line in out.splitlines()]


def test_threads_of_a_launch(tmp_path):
    rows = run(tmp_path, 'for (int t : {64, 128, 256, 320, 512, 1024}) printf("%d %lld\\n", t, (ll)max_groups(t));')
    for threads, groups in rows:
        assert groups * threads < 2 ** 32 <= (groups + 1) * threads


def test_tiled_cholesky_row_numbers(tmp_path):
    """Rows and columns that the tiled kernel numbers: up to the tile row that
    enters two panels past the last one (13 tiles beyond n with the widest
    window), all in 32 bits wherever it is taken."""
    ns = [1, 2, 15, 16, 17, 32768] + [2 ** 31 - 1 - d for d in range(0, 420)]
    kds = [0, 1, 16, 143, 144, 145, 200]
    body = "".join(f'printf("{n} {kd} %d\\n", (int)chol_tile_fits({n}LL, {kd}));\n' for n in ns for kd in kds)
    taken = 0
    for n, kd, fits in run(tmp_path, body):
        panels, T = (n + 15) // 16, max(2, (kd + 15) // 16 + 1)
        last = 16 * (panels + 1 + T) + 15  # row of the entry fetched for panel `panels`
        assert not fits or (last < 2 ** 31 and kd <= 144)
        assert fits or kd > 144 or n > 2 ** 31 - 1 - 224
        taken += fits
    assert taken > 0


def test_small_cholesky_fits_lds(tmp_path):
    """The column kernel's window (kd+2 columns of kd+1 entries, kd < n) stays
    within the 64 KiB that need no attribute; beyond n = 8, few systems and
    long ones keep the tiles."""
    rows = run(tmp_path, """for (ll batch : {1LL, 512LL, 513LL, 1023LL, 1024LL, 2048LL, 4096LL, 16384LL, 1LL << 31})
        for (ll n = 1; n <= 300; ++n)
            for (ll kd = 0; kd < n && kd < 80; ++kd)
                printf("%lld %lld %lld %d\\n", batch, n, kd, (int)chol_columns(n, kd, batch));""")
    for batch, n, kd, col in rows:
        assert not col or (kd + 2) * (kd + 1) * 8 <= 64 * 1024
        if n <= 8:
            assert col
        elif batch <= 512 or n > 192:
            assert not col
    assert any(col and n > 8 for _, n, _, col in rows)


def test_halves_of_the_lt_pass(tmp_path):
    """Every row of every accepted n (up to 2^31 - 1) is staged, in 32 bits."""
    ns = list(range(2, 140)) + [2 ** 31 - 1 - d for d in range(70)]
    body = "".join(f'printf("{n} {b} %d\\n", lt_halves({n}, {b}));\n' for n in ns for b in range(7))
    for n, nbs, halves in run(tmp_path, body):
        assert halves == -(-(n - 1) // 2 ** nbs)
