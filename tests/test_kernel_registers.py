"""The register records of the built kernels.  A kernel that runs out of vector
registers still gives the right values, through scratch memory and at a
fraction of its speed, so no other test sees it."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2003_04296_amd as q

READELF = shutil.which("llvm-readelf", path="/opt/rocm/llvm/bin:" + os.environ.get("PATH", ""))


def _code_objects(path):
    """The gfx950 code objects of a library: ELF files inside its offload bundles
    (magic, count, then offset, size and target of each entry)."""
    data = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        (count,), p = struct.unpack_from("<Q", data, at + len(magic)), at + len(magic) + 8
        for _ in range(count):
            off, size, tlen = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + tlen].decode()
            p += 24 + tlen
            if "gfx950" in target and size:
                yield data[at + off:at + off + size]
        at = data.find(magic, p)


def _spills(tmp_path):
    """{kernel: spilled vector registers} of libqconv.so."""
    out = {}
    for i, obj in enumerate(_code_objects(q.LIB_PATH)):
        f = tmp_path / f"{i}.co"
        f.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(f)], check=True, capture_output=True, text=True).stdout
        for rec in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", rec).group(1)
            out[name] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", rec).group(1))
    return out


@pytest.mark.skipif(READELF is None, reason="llvm-readelf reads the kernels' records")
def test_vector_registers_suffice(tmp_path):
    spills = _spills(tmp_path)
    assert sum("conv_mfma_kernel" in k for k in spills) >= 60, len(spills)
    # The store-overlapped kernel has 128 registers a lane (16 waves in one block);
    # its 128-channel shapes spill up to 24, and its speed is measured with them.
    allowed = {k: 32 if "conv_mfma_pp_kernel" in k else 0 for k in spills}
    over = {k: v for k, v in spills.items() if v > allowed[k]}
    assert not over, over
