"""The decode kernels keep their working set in registers: the built library's
own kernel metadata (written by the compiler) shows no register spilled to
scratch memory.  A spill inside the streaming loop costs up to half of a call's
speed and no result shows it.  Runs without a GPU."""
import re
import shutil
import struct
import subprocess

import pytest

from paper_2405_19888_amd import binding as B

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    """gfx950 ELF images inside the library's offload bundles (one per source)."""
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + tlen]
            p += 24 + tlen
            if triple.endswith(b"gfx950") and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, p)


def test_decode_kernels_do_not_spill(parrot_lib, tmp_path):
    readelf = shutil.which("llvm-readelf", path="/opt/rocm/llvm/bin") or shutil.which("llvm-readelf")
    if readelf is None:
        pytest.skip("llvm-readelf is not installed")
    found, spilled = set(), []
    for i, image in enumerate(code_objects(open(B.LIB_PATH, "rb").read())):
        f = tmp_path / f"{i}.elf"
        f.write_bytes(image)
        notes = subprocess.run([readelf, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n\s+- \.a", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)", kernel)
            spill = re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel)
            if name and spill and re.search(r"k_partials|k_direct|k_merge", name.group(1)):
                found.add(re.search(r"k_[a-z]+", name.group(1)).group(0))
                if int(spill.group(1)):
                    spilled.append((name.group(1), int(spill.group(1))))
    assert found == {"k_partials", "k_direct", "k_merge"}
    assert not spilled, spilled
