"""What the compiler's metadata in the built library says of the MTTKRP
kernels: none keeps registers in scratch memory (a spill in the inner loop is
memory traffic per gathered entry)."""
import os
import re
import struct
import subprocess

import pytest

from paper_1406_4519_amd import build_ext, dfacto

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _device_objects(lib):
    """The gfx950 code objects in a library's offload bundles."""
    data = open(lib, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if build_ext.ARCH.encode() in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def _kernels(lib, tmp_path):
    readelf = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
    if not os.path.exists(readelf):
        pytest.skip("no llvm-readelf")
    out = {}
    for q, obj in enumerate(_device_objects(lib)):
        f = tmp_path / f"{q}.o"
        f.write_bytes(obj)
        notes = subprocess.run([readelf, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        # one block per kernel; .name precedes its other scalar fields alphabetically
        for block in re.split(r"\n  - \.a", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)\n\s+\.private_segment_fixed_size:\s+(\d+)", block)
            if name:
                out[name.group(1)] = int(name.group(2))
    return out


def test_mttkrp_kernels_use_no_scratch(tmp_path):
    dfacto.load()  # builds it if nothing is there
    k = _kernels(build_ext.LIB, tmp_path)
    mttkrp = {n: s for n, s in k.items() if re.search(r"\d+k_mttkrp(_group|_block)?I", n)}
    kinds = {re.search(r"k_mttkrp[a-z_]*", n).group(0) for n in mttkrp}
    assert kinds == {"k_mttkrp", "k_mttkrp_group", "k_mttkrp_block"}
    assert {n: s for n, s in mttkrp.items() if s} == {}
