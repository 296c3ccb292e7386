"""The search and sweep kernels read their dynamic LDS as 16-byte words.  It
starts where the kernel's static LDS ends, so that size, taken from the
metadata of the built code objects, has to be a multiple of 16 for every
form of the two kernels."""
import os
import re
import struct
import subprocess

import pytest

from paper_1909_07717_amd import build as Bd

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """GPU code objects of a library's offload bundles."""
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, name_len = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + name_len]
            pos += 24 + name_len
            if b"gfx" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


@pytest.mark.skipif(not os.path.exists(READELF), reason="needs llvm-readelf")
def test_dynamic_lds_starts_on_16_bytes(tmp_path):
    with open(Bd.LIB, "rb") as fh:
        blob = fh.read()
    sizes = {}
    for i, obj in enumerate(_code_objects(blob)):
        f = tmp_path / f"{i}.o"
        f.write_bytes(obj)
        notes = subprocess.check_output([READELF, "--notes", str(f)], text=True)
        for rec in re.split(r"\n\s*- \.agpr_count", notes)[1:]:
            name = re.search(r"\.symbol:\s+(\S+)", rec).group(1)
            if "search_kernel" in name or "ray_kernel" in name:
                sizes[name] = int(re.search(r"\.group_segment_fixed_size:\s+(\d+)", rec).group(1))
    assert len(sizes) >= 4 * 3 + 4  # K = 64 .. 256: maps, power, best only; the sweep
    assert {n: s for n, s in sizes.items() if s % 16} == {}
