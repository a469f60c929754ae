"""What the compiler gave the library's gfx950 kernels, from the metadata of the code objects built here."""
import os
import re
import struct
import subprocess

import pytest

from paper_1310_0901_amd import xfercheck as X

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The device code objects in a library's offload bundles."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + idlen].decode()
            pos += 24 + idlen
            if "gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def kernels(path, tmp):
    """{demangled kernel name: bytes of scratch per lane}"""
    found = {}
    for k, obj in enumerate(code_objects(path)):
        f = tmp / f"{k}.co"
        f.write_bytes(obj)
        text = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for one in re.split(r"(?m)^ +- \.", text)[1:]:
            name = re.search(r"(?m)^ +\.name: +(\S+)", one)
            size = re.search(r"(?m)^ +\.private_segment_fixed_size: +(\d+)", one)
            if name and size:
                found[name.group(1)] = int(size.group(1))
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True).stdout.split("\n")
    return dict(zip(names, found.values()))


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_no_kernel_uses_scratch(tmp_path):
    """No kernel, and so no launch shape that cg_set_tuning takes, spills to memory."""
    ks = kernels(X.LIB_PATH, tmp_path)
    assert any("k_batched_2d" in k for k in ks) and any("k_race_sweep_apply" in k for k in ks)
    assert {k: n for k, n in ks.items() if n} == {}
