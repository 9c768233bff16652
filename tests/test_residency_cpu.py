"""Registers that the built gfx950 kernels are allocated, read from their kernel
descriptors in lib/libonebit.so, where a kernel's residency is meant to be held
by them."""
import os
import struct

import pytest

from paper_2102_02888_amd.build import LIB

VGPRS_PER_SIMD = 512  # per lane, architectural and accumulation registers together
EM_AMDGPU = 224


def _kernel_vgprs(blob):
    """{kernel symbol: allocated VGPRs} of every AMDGPU ELF inside the library."""
    out = {}
    at = blob.find(b"\x7fELF", 1)
    while at >= 0:
        elf = blob[at:]
        if len(elf) > 64 and struct.unpack_from("<H", elf, 18)[0] == EM_AMDGPU:
            shoff, = struct.unpack_from("<Q", elf, 40)
            size, count = struct.unpack_from("<HH", elf, 58)
            secs = [struct.unpack_from("<IIQQQQIIQQ", elf, shoff + i * size) for i in range(count)]
            for sec in secs:
                if sec[1] != 2:  # SHT_SYMTAB
                    continue
                names = secs[sec[6]][4]
                for k in range(sec[5] // 24):
                    name, _, _, shndx, value, _ = struct.unpack_from("<IBBHQQ", elf, sec[4] + 24 * k)
                    text = elf[names + name:elf.index(b"\0", names + name)].decode()
                    if text.endswith(".kd"):
                        home = secs[shndx]
                        rsrc1, = struct.unpack_from("<I", elf, home[4] + value - home[3] + 48)
                        out[text[:-3]] = ((rsrc1 & 63) + 1) * 8
        at = blob.find(b"\x7fELF", at + 4)
    return out


@pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")
def test_row_walk_runs_one_workgroup_per_cu():
    """The fp32-momentum row walk has 16 waves per workgroup, four on each SIMD,
    and is meant to run alone on its CU: a second workgroup's registers must not
    fit, however few the code itself needs."""
    with open(LIB, "rb") as f:
        vgprs = _kernel_vgprs(f.read())
    walks = {k: v for k, v in vgprs.items() if "k_worker_rows" in k}
    assert len(walks) == 3, sorted(vgprs)  # fp32, bf16 and fp16 gradients
    for name, v in walks.items():
        assert VGPRS_PER_SIMD // v == 4, (name, v)
