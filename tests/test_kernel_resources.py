"""Registers of the built kernels, from the metadata of the code objects in libqift.so (no GPU needed).

A spill in a loop that counts its outstanding loads costs more than the access: the reload's wait also waits for
the loads sent ahead.  So these kernels hold everything in registers, in every instance.
"""
import struct

import msgpack
import pytest

from paper_2606_02823_amd import qift

EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def kernels(path):
    """name -> metadata of every kernel of the code objects embedded in a shared library."""
    with open(path, "rb") as f:
        d = f.read()
    out, p = {}, d.find(b"\x7fELF\x02\x01\x01")
    while p >= 0:
        if struct.unpack_from("<H", d, p + 18)[0] == EM_AMDGPU:
            (shoff,), (size, n) = struct.unpack_from("<Q", d, p + 40), struct.unpack_from("<HH", d, p + 58)
            for i in range(n):
                sec = p + shoff + i * size
                if struct.unpack_from("<I", d, sec + 4)[0] != SHT_NOTE:
                    continue
                off, length = struct.unpack_from("<QQ", d, sec + 24)
                q, end = p + off, p + off + length
                while q < end:
                    nname, ndesc, kind = struct.unpack_from("<III", d, q)
                    q += 12 + (nname + 3) // 4 * 4
                    if kind == NT_AMDGPU_METADATA:
                        for k in msgpack.unpackb(d[q:q + ndesc])["amdhsa.kernels"]:
                            out[k[".name"]] = k
                    q += (ndesc + 3) // 4 * 4
        p = d.find(b"\x7fELF\x02\x01\x01", p + 4)
    return out


@pytest.mark.parametrize("name", ["k_gemm32", "k_gemm_split", "k_batch", "k_skinny", "k_decode_chain"])
def test_no_spills(name):
    ks = {k: v for k, v in kernels(qift.LIB_PATH).items() if f"{len(name)}{name}" in k}
    assert ks, name
    spilled = {k: v[".vgpr_spill_count"] for k, v in ks.items()
               if v[".vgpr_spill_count"] or v[".private_segment_fixed_size"]}
    assert not spilled


def test_scale_search_leaves_four_workgroups_a_cu():
    # PoT (1) and the mirror sets (3) of one- and two-tile rows: a quarter of the 160 KB, a quarter of the registers
    ks = {k: v for k, v in kernels(qift.LIB_PATH).items() if "15k_quant_weights" in k}
    search = {k: v for k, v in ks.items() if any(f"ILi{f}ELi{t}E" in k for f in (1, 3) for t in (1, 2))}
    assert len(search) == 20
    for k, v in search.items():
        assert v[".group_segment_fixed_size"] <= 40960 and v[".vgpr_count"] <= 128, k
