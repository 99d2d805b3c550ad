"""Registers of the built attention kernels, from the code object's own notes
(no GPU): the kernels of the default launch mode keep everything in registers."""
import os
import re
import struct
import subprocess

import pytest

from paper_2609_34388_amd import binding

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"

pytestmark = pytest.mark.skipif(not (os.path.exists(binding.LIB_PATH) and os.path.exists(READELF)),
                                reason="library not built, or no llvm-readelf")


def _code_objects():
    """The gfx950 code objects bundled in the library, one per source file."""
    blob = open(binding.LIB_PATH, "rb").read()
    for at in (m.start() for m in re.finditer(MAGIC, blob)):
        count, pos = struct.unpack_from("<Q", blob, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, idlen = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + idlen].decode()
            pos += 24 + idlen
            if "gfx950" in name and size:
                yield blob[at + offset:at + offset + size]


def _kernels(tmp_path):
    """{kernel name: {note key: value}}"""
    out = {}
    for i, obj in enumerate(_code_objects()):
        path = tmp_path / f"{i}.co"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for block in notes.split("  - .agpr_count:")[1:]:
            got = dict(re.findall(r"^    \.(\w+): +(\S+)$", block, re.M))
            out[got["name"]] = got
    return out


def test_default_attention_kernels_do_not_spill(tmp_path):
    kernels = {k: v for k, v in _kernels(tmp_path).items() if "attn_fwd_kernel" in k or "attn_combine_kernel" in k}
    # head size x work group x plan form, and the merges of the two forms that split
    assert sum("attn_fwd_kernel" in k for k in kernels) == 2 * 2 * 3
    assert sum("attn_combine_kernel" in k for k in kernels) == 2 * 2 * 2
    for name, k in kernels.items():
        assert int(k["vgpr_spill_count"]) == 0 and int(k["private_segment_fixed_size"]) == 0, name
        assert int(k["vgpr_count"]) <= 168, name  # three waves per SIMD
