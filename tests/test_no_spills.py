"""Register use of the convolution passes, from the built library's own kernel
descriptions.  The x passes and the staged z convolution keep everything in
registers (no scratch) up to 2048 points; at 4096, where a thread carries 16,
they may not.  And the x passes stay within the registers of the waves per SIMD
that their launches give a CU: 512 / 6 = 80 (in steps of 8), 96 for five waves,
128 for four."""
import os
import re
import struct
import subprocess

import pytest

from paper_1406_7635_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled kernel name: (bytes of scratch per lane, vector registers)}"""
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        lib = f.read()
    path = str(tmp_path_factory.mktemp("code") / "k.co")
    out = {}
    at = lib.find(MAGIC)
    while at >= 0:
        p = at + len(MAGIC)
        (count,) = struct.unpack_from("<Q", lib, p)
        p += 8
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", lib, p)
            name = lib[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" not in name or size == 0:
                continue
            with open(path, "wb") as f:
                f.write(lib[at + off:at + off + size])
            text = subprocess.run([READELF, "--notes", path], capture_output=True, text=True, check=True).stdout
            for k in re.split(r"\n\s+- \.a", text):  # a kernel's entry begins with .agpr_count
                m = re.search(r"\.name:\s+(\w+)", k[k.find(".kernarg_segment_align"):])
                s = re.search(r"\.private_segment_fixed_size:\s+(\d+)", k)
                v = re.search(r"\.vgpr_count:\s+(\d+)", k)
                if m and s and v:
                    out[m[1]] = int(s[1]), int(v[1])
        at = lib.find(MAGIC, at + 1)
    names = subprocess.run(["c++filt"], input="\n".join(out), capture_output=True, text=True).stdout.split("\n")
    return dict(zip(names, out.values()))


def up_to_2048(kernels, kernel):
    """{template arguments: (scratch, registers)} of a kernel's forms up to 2048 points"""
    out = {}
    for name, v in kernels.items():
        m = re.search(r"\b%s<([^>]*)>" % kernel, name)
        if m and int(m[1].split(",")[0]) <= 2048:
            out[tuple(m[1].replace(" ", "").split(","))] = v
    return out


@pytest.mark.parametrize("kernel,forms", [("k_xfwd", 80), ("k_xinv", 120), ("k_xrow", 108), ("k_zconv", 10)])
def test_no_scratch(kernels, kernel, forms):
    got = up_to_2048(kernels, kernel)
    print(kernel, len(got))
    assert len(got) >= forms
    assert {a: s for a, (s, _) in got.items() if s} == {}


def test_registers_of_the_x_passes(kernels):
    over = {}
    for a, (_, v) in up_to_2048(kernels, "k_xfwd").items():  # P, FULL, W, Q4
        if v > (128 if a[1] == "true" else 96):
            over[("k_xfwd",) + a] = v
    for a, (_, v) in up_to_2048(kernels, "k_xrow").items():  # P, DMI, FULL, W, Q4
        if v > (128 if a[2] == "true" else 80):
            over[("k_xrow",) + a] = v
    for a, (_, v) in up_to_2048(kernels, "k_xinv").items():
        five = a[1] == "true" and a[4] == "true" and int(a[0]) < 1024  # x_one
        if v > (96 if five else 80):
            over[("k_xinv",) + a] = v
    assert over == {}
