"""What the compiler gave the kernels of the built library, from the metadata of its gfx950 code objects."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2407_09453_amd as bsp

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 code objects of a library: entries of (offset, size, triple) behind each bundle's magic and count."""
    at = blob.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", blob, at + len(MAGIC))[0]):
            off, size, n = struct.unpack_from("<QQQ", blob, pos)
            if b"gfx950" in blob[pos + 24:pos + 24 + n]:
                yield blob[at + off:at + off + size]
            pos += 24 + n
        at = blob.find(MAGIC, pos)


def _kernels(tmp_path):
    out = {}
    for n, co in enumerate(_code_objects(open(bsp.binding.lib_path(), "rb").read())):
        f = tmp_path / ("%d.co" % n)
        f.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n\s*- \.(?=agpr_count|args)", notes)[1:]:
            name = re.search(r"\.symbol:\s+(\S+?)\.kd", part)
            if name:
                out[name.group(1)] = {k: int(v) for k, v in re.findall(r"\.(private_segment_fixed_size|sgpr_spill_count|vgpr_spill_count|vgpr_count):\s+(\d+)", part)}
    return out


@pytest.mark.skipif(not os.path.exists(READELF) or not shutil.which("hipcc"), reason="no ROCm toolchain")
def test_any_shape_kernel_keeps_its_registers(tmp_path):
    """No scratch and no spilled vector register in any instance, one lane tile in the registers of five waves a SIMD
    (512 / 5 in eights); eight scalars at most wait in lanes of a vector register until the results need them."""
    found = {k: v for k, v in _kernels(tmp_path).items() if "conv_anyILi" in k}
    assert len(found) == 18, sorted(found)  # bf16: three lane tiles, aligned pixels or not, two ways out; int8: one way out
    for name, r in found.items():
        assert r["private_segment_fixed_size"] == 0 and r["vgpr_spill_count"] == 0, (name, r)
        assert r["sgpr_spill_count"] <= 8, (name, r)
        assert r["vgpr_count"] <= (96 if "ELi1ELb" in name else 128), (name, r)
