"""Arithmetic of the kernels' lattice indices on the host: the same device
header, its host side compiled by hipcc (no GPU code, no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1903_03356_amd", "csrc")

DRIVER = r"""
#include "lbib_device.h"
#include <limits.h>
#include <stdio.h>

int main()
{
    const int sizes[] = {8, 9, 64, 65, 1000, 4095, 1 << 20};
    int bad = 0;
    for (int n : sizes) {
        const int bases[] = {0, 1, n / 2, n - 1};
        const long long near[] = {0, n, -n, 2LL * n, -2LL * n, 12345LL * n, INT_MAX, INT_MIN};
        for (int base : bases)
            for (long long c : near)
                for (long long d = -300; d <= 300; d++) {
                    const long long off = c + d;
                    if (off < INT_MIN || off > INT_MAX) continue;
                    const int sum = (int)((unsigned)base + (unsigned)off);  // wraps at 2^31
                    const long long want = ((long long)sum % n + n) % n;
                    if (lbib::wrap_add(base, (int)off, n) != want && bad++ < 5)
                        printf("wrap_add(%d, %lld, %d), want %lld\n", base, off, n, want);
                }
    }
    return bad != 0;
}
"""


def compiled(tmp_path, source):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(source)
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I",
                    os.path.join(ROOT, "include"), "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    return exe


def test_wrap_of_any_offset(tmp_path):
    """Offsets from -2^31 to 2^31 - 1 (a diverged capsule's): the remainder, in a
    bounded number of operations.  100,000 of them in well under a second; a loop
    over the period takes a minute for n = 8 alone."""
    exe = compiled(tmp_path, DRIVER)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=20)
    assert r.returncode == 0, r.stdout


RECTS = r"""
#include "lbib_device.h"
#include <limits.h>
#include <stdio.h>
#include <vector>
using namespace lbib;

static int bad = 0;

static void check(const NearRect& r, const GridArgs& g, bool sane)
{
    const NearCells c = near_cells(r, g, 3);
    const RectUnits u = rect_units(r, g);
    bool ok = c.w >= 0 && c.w <= g.nx && c.rows >= 0 && c.rows <= g.ny && c.x0 >= 0 && c.x0 < g.nx;
    ok = ok && (c.rows == 0 || (c.y0 >= 0 && c.y0 < g.ny && (g.periodic_y || c.y0 + c.rows <= g.ny)));
    ok = ok && u.nrows >= 0 && u.nrows <= g.ny && u.nsegs >= 0 && u.nsegs <= g.nseg + 1;
    ok = ok && u.nA <= u.nsegs && (u.nsegs == 0 || (u.sa >= 0 && u.sa + u.nA <= g.nseg));
    ok = ok && (u.nrows == 0 || (u.ry0 >= 0 && u.ry0 < g.ny && (g.periodic_y || u.ry0 + u.nrows <= g.ny)));
    if (ok && sane) {  // exactly the cells of the grown box, and the segments of the box
        std::vector<int> want(g.nx * g.ny), got(g.nx * g.ny), seg(g.nseg * g.ny), has(g.nseg * g.ny);
        auto mark = [&](std::vector<int>& cells, std::vector<int>* segs, int more) {
            for (int y = r.y0 - more; y <= r.y1 + more; y++) {
                const int yy = g.periodic_y ? ((y % g.ny) + g.ny) % g.ny : y;
                if (yy < 0 || yy >= g.ny) continue;
                for (int x = r.x0 - more; x <= r.x1 + more; x++) {
                    const int xx = ((x % g.nx) + g.nx) % g.nx;
                    cells[yy * g.nx + xx] = 1;
                    if (segs) (*segs)[yy * g.nseg + xx / kSegW] = 1;
                }
            }
        };
        mark(want, nullptr, 3);
        std::vector<int> box(g.nx * g.ny);
        mark(box, &seg, 0);
        for (int i = 0; i < c.rows; i++)
            for (int j = 0; j < c.w; j++)
                got[((c.y0 + i) % g.ny) * g.nx + (c.x0 + j) % g.nx] = 1;
        for (int i = 0; i < u.nrows; i++)
            for (int j = 0; j < u.nsegs; j++)
                has[((u.ry0 + i) % g.ny) * g.nseg + (j < u.nA ? u.sa + j : j - u.nA)] = 1;
        ok = want == got;
        for (size_t i = 0; i < seg.size(); i++) ok = ok && has[i] >= seg[i];
    }
    if (!ok && bad++ < 5)
        printf("rect %d %d %d %d on %d x %d, periodic_y %d\n", r.x0, r.y0, r.x1, r.y1, g.nx, g.ny,
               g.periodic_y);
}

int main()
{
    const int v[] = {INT_MIN, INT_MIN + 2, -2000000000, -1500000000, -70000, 0, 40, 70000, 1500000000,
                     2000000000, INT_MAX - 2, INT_MAX};
    unsigned long long s = 1;
    auto rnd = [&](int n) { s = s * 6364136223846793005ull + 1442695040888963407ull; return (int)((s >> 33) % n); };
    for (int nx : {8, 100, 192})
        for (int py : {0, 1}) {
            GridArgs g = {};
            g.nx = nx;
            g.ny = 45;
            g.nseg = (nx + 63) / 64;
            g.periodic_y = py;
            g.periodic_x = 1;
            for (int a : v) for (int b : v) for (int c : v) for (int d : v) check({a, b, c, d}, g, false);
            for (int k = 0; k < 400; k++) {
                const int x0 = rnd(3000) - 1500, y0 = py ? rnd(3000) - 1500 : rnd(80) - 20;
                check({x0, y0, x0 + rnd(60), y0 + rnd(40)}, g, true);
            }
        }
    return bad != 0;
}
"""


def test_near_regions_of_any_box(tmp_path):
    """The near region of a capsule: exactly its cells for the boxes of a running
    simulation, and inside the lattice for any box (a diverged capsule's
    coordinates convert to arbitrary ints)."""
    exe = compiled(tmp_path, RECTS)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


OTHERS = r"""
#include "lbib_device.h"
#include <stdio.h>
#include <vector>
using namespace lbib;

int main()
{
    int bad = 0;
    for (int nx : {8, 11, 30})
        for (int ny : {9, 25})
            for (int px = 0; px < 2; px++)
                for (int py = 0; py < 2; py++)
                    for (int w = 3; w <= 12; w += 3)
                        for (int h = 3; h <= 12; h += 2)
                            for (int x0 = px ? -1 : -w - 2; x0 <= nx + 2; x0++)
                                for (int y0 = py ? -1 : -h - 2; y0 <= ny + 2; y0++) {
                                    GridArgs g = {};
                                    g.nx = nx;
                                    g.ny = ny;
                                    g.periodic_x = px;
                                    g.periodic_y = py;
                                    const OtherCells o(g, false, x0, y0, w, h);
                                    std::vector<int> got(w * h);
                                    bool ok = true;
                                    for (int j = 0; j < o.n; j++) {
                                        int lx, ly;
                                        o.cell(j, lx, ly);
                                        ok = ok && lx >= 0 && lx < w && ly >= 0 && ly < h;
                                        if (ok) got[ly * w + lx] = 1;
                                    }
                                    const bool all = (px && w > nx) || (py && h > ny);
                                    for (int ly = 0; ly < h; ly++)
                                        for (int lx = 0; lx < w; lx++) {
                                            const int x = px ? ((x0 + lx) % nx + nx) % nx : x0 + lx;
                                            const int y = py ? ((y0 + ly) % ny + ny) % ny : y0 + ly;
                                            const int want = all || !plain_cell(g, x, y);
                                            ok = ok && got[ly * w + lx] == want;
                                        }
                                    if (!ok && bad++ < 5)
                                        printf("box %d x %d at (%d, %d) on %d x %d, periodic %d %d\n", w,
                                               h, x0, y0, nx, ny, px, py);
                                }
    return bad != 0;
}
"""


def test_cells_of_a_patch_at_the_ends(tmp_path):
    """The cells of a patch that do not take the nine plain loads: exactly those on the
    lattice's end rows and columns and off it, for every place of a box on walls, open
    ends and wraps; all cells of a box that wraps onto itself."""
    exe = compiled(tmp_path, OTHERS)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
