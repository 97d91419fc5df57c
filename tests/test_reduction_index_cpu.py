"""Index arithmetic of the global reductions (csrc/lbm_reduce.hpp) at the
largest lattices that lbm_create takes, compiled with the host compiler:
evaluated in constant expressions, where an overflow is a compile error, and
against 128-bit arithmetic."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1107_4543_amd", "csrc")
# the largest width (pitch a multiple of 64, pitch * ny < 2^31)
WIDEST = 2 ** 31 - 64


def check(tmp_path, body, asserts=()):
    src = os.path.join(str(tmp_path), "t.cpp")
    with open(src, "w") as fh:
        fh.write('#include <cstdio>\n#include <initializer_list>\n#include "lbm_reduce.hpp"\nusing namespace lbm;\ntypedef __int128 wide;\n')
        for a in asserts:
            fh.write(f'static_assert({a}, "");\n')
        fh.write("int main()\n{\n" + body + "\n    return 0;\n}\n")
    exe = src[:-4]
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-ftrapv", "-Wall", "-I", CSRC, src, "-o", exe], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout[-2000:])


def test_modes_of_very_wide_lattices(tmp_path):
    check(tmp_path, """
    const int ks[] = {0, 1, -1, 12345, -70001, 1500000000, -1500000000, 2147483647, -2147483647 - 1};
    const int ns[] = {1, 2, 3, 64, 65535, 1 << 30, (1 << 30) + 1, 1600000000, %d};
    for (int n : ns)
        for (int k : ks) {
            wide want = (wide)k %% n;
            if (want < 0) want += n;
            if (wrap_mode(k, n) != want) { printf("%%d mod %%d: %%d", k, n, wrap_mode(k, n)); return 1; }
        }""" % WIDEST, ["wrap_mode(1500000000, 1600000000) == 1500000000", f"wrap_mode(-1, {WIDEST}) == {WIDEST - 1}"])


def test_blocks_share_out_every_column_and_band_once(tmp_path):
    # widths around a block's threads and up to the widest lattice; bands are
    # counted for the tallest lattice of the width, and for few rows
    check(tmp_path, """
    const int ns[] = {1, 2, 3, 255, 256, 257, 1023, 1025, 40000, 524287, 524289, (1 << 30) + 1, 1600000000, 2143400000, %d};
    for (int threads : {256, 1024})
        for (int nx : ns)
            for (int rows = 0; rows < 4; ++rows) {
                const wide pitch = ((wide)nx + 63) / 64 * 64;
                const int tallest = (int)((((wide)1 << 31) - 1) / pitch);
                const int ny = rows == 3 ? tallest : rows + 1 < tallest ? rows + 1 : tallest;
                const RedShape g = red_shape(nx, ny, threads, 512);
                const int w = 1 << g.shift, h = threads >> g.shift;
                printf("%%d x %%d, %%d threads: bx %%d by %%d cols %%d shift %%d\\n", nx, ny, threads, g.bx, g.by, g.cols, g.shift);
                if (g.bx < 1 || g.by < 1 || g.blocks() > 512 || g.cols < 1 || g.cols %% w || w * h != threads) return 1;
                wide at = 0;
                for (int b = 0; b < g.bx; ++b) {
                    const RedCols c = red_cols(g, b, nx);
                    if (c.from != at || c.to <= c.from || c.to > (uint32_t)nx) return 2;
                    // the last column of the last thread, and the one after it that ends its loop
                    if ((uint32_t)(c.to - 1 + w) < c.to) return 3;
                    at = c.to;
                }
                if (at != nx) return 4;
            }""" % WIDEST, [f"red_shape({WIDEST}, 1, 1024, 512).bx == 512", "red_shape(2143400000, 1, 1024, 512).bx > 0"])


def test_phase_products_up_to_the_edges_of_the_32_bit_path(tmp_path):
    check(tmp_path, """
    const int ns[] = {1, 2, 46341, 46342, 60000, 65535, 65536, 65537, 1 << 20, 1600000000, %d};
    for (int n : ns)
        for (int m : {0, 1, n / 2, n - 2, n - 1})
            for (int v : {-1, 0, 1, n / 2, n - 2, n - 1}) {
                if (m < 0 || m >= n || v >= n) continue;
                wide want = (wide)m * v %% n;
                if (want < 0) want += n;
                if (phase_index(m, v, n) != want) { printf("%%d * %%d mod %%d: %%u", m, v, n, phase_index(m, v, n)); return 1; }
            }""" % WIDEST, ["phase_index(65534, 65534, 65535) == 1", "phase_index(46341, 46341, 46342) == 1",
                            "phase_index(65534, -1, 65535) == 1"])
