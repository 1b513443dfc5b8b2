"""Registers of the compiled kernels, read from the library built here (CPU
only): the composition is bound by memory, and what hides its latency is the
number of waves a SIMD holds (512 / registers, at most 8)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
READELF = shutil.which("llvm-readelf", path="/opt/rocm/llvm/bin") or shutil.which("llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def vgprs(tmp_path_factory):
    """Kernel name (mangled) -> vector registers."""
    if READELF is None:
        pytest.skip("no llvm-readelf")
    from paper_2607_15650_amd import _lib
    _lib.lib()                                            # raises if it is not built
    data = open(os.path.join(ROOT, "paper_2607_15650_amd", "libditango.so"), "rb").read()
    out, at, d = {}, data.find(MAGIC), tmp_path_factory.mktemp("co")
    while at >= 0:
        n, pos = struct.unpack_from("<Q", data, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + ln].decode()
            pos += 24 + ln
            if "gfx950" in triple and size:
                f = d / f"{at}.elf"
                f.write_bytes(data[at + off:at + off + size])
                text = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
                for name, count in re.findall(r"\.name:\s+(\S+).*?\.vgpr_count:\s+(\d+)", text, re.S):
                    out[name] = int(count)
        at = data.find(MAGIC, at + 1)
    if not out:
        pytest.skip("the library's code objects are not in a plain bundle")
    return out


# (slots of the instance, waves per SIMD of a composition of bf16 states
# without weights); 64 slots hold their weights in registers
@pytest.mark.parametrize("slots,waves", [(4, 8), (8, 8), (16, 7), (64, 3)])
@pytest.mark.parametrize("D", [64, 128])
def test_composition_without_weights_keeps_its_waves(vgprs, D, slots, waves):
    names = [n for n in vgprs if re.search(rf"merge_kernelIDF16b(DF16b|f)Li{D}ELi{slots}ELb1E(Lb0E)?E", n)]
    assert len(names) == 2, sorted(n for n in vgprs if "merge_kernel" in n)[:8]
    for n in names:
        regs = -(-vgprs[n] // 8) * 8
        assert min(8, 512 // regs) >= waves, (n, vgprs[n])
