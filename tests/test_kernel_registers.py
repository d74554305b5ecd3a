"""Vector registers of the wave-pool kernels in the built library: the
instantiations that a set launches alone, without trace, keep their state in
registers (a few spilled ones at most: the streaming kernels' window).  Spills in
the step loop cost the full general level up to twice its time."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2512_02175_amd", "libmetricgraph.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def code_objects(blob):
    """The gfx950 images of the library's offload bundles."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        n, o = struct.unpack_from("<Q", blob, at + 24)[0], at + 32
        for _ in range(n if n < 16 else 0):
            off, size, name = struct.unpack_from("<QQQ", blob, o)
            if size and b"gfx950" in blob[o + 24:o + 24 + name]:
                yield blob[at + off:at + off + size]
            o += 24 + name
        at += len(magic)


@pytest.mark.skipif(not (os.path.exists(LIB) and shutil.which(READELF)),
                    reason="needs the built library and llvm-readelf")
def test_pool_kernels_spill_little(tmp_path):
    spills = {}
    for i, image in enumerate(code_objects(open(LIB, "rb").read())):
        f = tmp_path / f"{i}.o"
        f.write_bytes(image)
        notes = subprocess.run([READELF, "--notes", str(f)], check=True, capture_output=True,
                               text=True).stdout
        for name, n in re.findall(r"\.name:\s+(\S+).*?\.vgpr_spill_count:\s+(\d+)", notes, re.S):
            # <trace, exits in LDS, tables in LDS, streaming, ...>
            m = re.search(r"k_pool(?:32|64)I(Lb0E\S*?)EEv", name)
            if m:
                spills[m[0]] = int(n)
    assert len(spills) >= 40
    assert max(spills.values()) <= 8, {k: v for k, v in spills.items() if v > 8}
