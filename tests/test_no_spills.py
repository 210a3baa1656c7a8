"""The convolution passes keep everything in registers: the built library's own
kernel descriptions must show no scratch for the x passes and the staged z
convolution up to 2048 points.  (4096 points, where a thread carries 16, are
left out.)"""
import os
import re
import struct
import subprocess

import pytest

from paper_1406_7635_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """{demangled kernel name: bytes of scratch per lane}"""
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
                if m and s:
                    out[m[1]] = int(s[1])
        at = lib.find(MAGIC, at + 1)
    names = subprocess.run(["c++filt"], input="\n".join(out), capture_output=True, text=True).stdout.split("\n")
    return dict(zip(names, out.values()))


@pytest.mark.parametrize("kernel,forms", [("k_xfwd", 80), ("k_xinv", 120), ("k_xrow", 108), ("k_zconv", 10)])
def test_no_scratch(scratch, kernel, forms):
    got = {}
    for name, size in scratch.items():
        m = re.search(r"\b%s<(\d+)" % kernel, name)
        if m and int(m[1]) <= 2048:
            got[name.split("(")[0]] = size
    print(kernel, len(got))
    assert len(got) >= forms
    assert {n: s for n, s in got.items() if s} == {}
