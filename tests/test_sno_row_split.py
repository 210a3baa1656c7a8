"""The split of the surrogate's rows over workgroups (sno_rows.h), on the host:
while a workgroup holds several rows, the launch has at least one workgroup
for each of the 256 CUs, a row's tiles keep the waves they can use, and the
LDS of a workgroup stays within 160 KiB (a CU's)."""
import os
import subprocess

import pytest

from paper_1406_7635_amd import build

PROGRAM = r"""
#include "sno_rows.h"
#include <cstdio>
int main() {
    using namespace mm;
    int bad = 0;
    for (int nx = 32; nx <= 512; ++nx)
        for (long long rows = 16; rows <= 256LL * 512; rows = rows < 4200 ? rows + 1 : rows * 2 + 1) {
            const int s = row_wave_shift(nx, rows), per = ROW_WAVES >> s, tiles = (nx + 31) / 32;
            const long long groups = (rows + per - 1) / per;
            const bool ok = s >= 0 && s <= 3 && (per == 1 || groups >= 256) && ((1 << s) >= tiles || s == 3) &&
                            row_lds(nx, s) <= 160 * 1024 && (long long)row_blocks(rows, s) <= groups &&
                            row_blocks(rows, s) >= 1;
            if (!ok && bad++ < 5) printf("nx %d rows %lld: shift %d groups %lld\n", nx, rows, s, groups);
        }
    printf(bad ? "BAD\n" : "ALL OK\n");
    return bad != 0;
}
"""


def test_row_split(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    src, exe = str(tmp_path / "split.hip"), str(tmp_path / "split")
    with open(src, "w") as f:
        f.write(PROGRAM)
    r = subprocess.run([build.HIPCC] + build.FLAGS + ["-x", "hip", src, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "ALL OK" in r.stdout, r.stdout
