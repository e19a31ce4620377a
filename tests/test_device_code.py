"""What the compiler made of the row kernels: the Gibbs instances with an explicit right-hand side
at seven and eight tiles run at two waves per SIMD because their registers are full, so a spill
there is a scratch round trip inside the factorisation's dependent chain."""
import os
import re
import struct
import subprocess

import pytest

import paper_1108_2580_amd as pkg

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def device_objects():
    """The gfx950 code objects inside the library's offload bundles."""
    data = open(pkg.LIB_PATH, "rb").read()
    for m in re.finditer(MAGIC, data):
        (n,) = struct.unpack_from("<Q", data, m.start() + len(MAGIC))
        at = m.start() + len(MAGIC) + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in triple and size:
                yield data[m.start() + off:m.start() + off + size]


def row_kernels(tmp_path):
    """(DP, AUG, BAYES, spilled registers, scratch bytes) of every instance of k_rows."""
    out = []
    for i, obj in enumerate(device_objects()):
        path = tmp_path / f"{i}.co"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True,
                               check=True).stdout
        for entry in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", entry).group(1)
            m = re.match(r"_ZN3als6k_rowsILi(\d+)ELb([01])ELb[01]ELb([01])E", name)
            if m:
                field = lambda k: int(re.search(rf"\.{k}:\s+(\d+)", entry).group(1))
                out.append((int(m[1]), m[2] == "1", m[3] == "1", field("vgpr_spill_count"),
                            field("private_segment_fixed_size")))
    return out


@pytest.mark.skipif(not os.path.exists(READELF), reason="needs the ROCm toolchain")
def test_wide_gibbs_rows_without_augmented_column_do_not_spill(tmp_path):
    kernels = row_kernels(tmp_path)
    wide = [k for k in kernels if k[0] >= 112 and not k[1] and k[2]]
    assert len(kernels) > 80 and len(wide) == 4  # 112 and 128, with one fixed table and two
    assert all(spills == 0 and scratch == 0 for *_, spills, scratch in wide), wide
