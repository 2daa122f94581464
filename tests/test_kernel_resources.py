"""What the compiler gave the conversion kernels of the small ring, read from the notes of the built library's code objects: the
instantiations for up to four sources spill nothing, those for five to eight keep what they were timed with."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _spills(tmp_path):
    data = open(os.path.join(ROOT, "paper_2602_11470_amd", "libcachemir.so"), "rb").read()
    spills, magic = {}, b"__CLANG_OFFLOAD_BUNDLE__"
    for i, m in enumerate(re.finditer(magic, data)):
        at = m.start() + len(magic)
        (count,) = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + idlen]
            at += 24 + idlen
            if b"gfx950" not in target or not size:
                continue
            path = tmp_path / f"{i}.elf"
            path.write_bytes(data[m.start() + off:m.start() + off + size])
            notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            for k in re.split(r"\n  - \.", notes):
                name, n = re.search(r"\.name: +(\S+)", k), re.search(r"\.vgpr_spill_count: (\d+)", k)
                if name and n:
                    spills[name.group(1)] = int(n.group(1))
    return spills


@pytest.mark.skipif(not os.path.exists(READELF), reason="needs the compiler's llvm-readelf")
def test_conversions_of_the_small_ring_spill_no_more_than_they_did(tmp_path):
    spills = {k: v for k, v in _spills(tmp_path).items() if "conv_full_fwd" in k}
    assert len(spills) >= 20
    for name, n in spills.items():
        sources, tail, fold = re.search(r"conv_full_fwdILi(\d)ELb(\d)ELb(\d)", name).groups()
        assert n <= (0 if sources != "8" else 60 if fold == "1" else 32), name
