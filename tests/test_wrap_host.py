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
