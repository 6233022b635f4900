"""Registers that the compiler spilled, from the metadata of the built kernels.
A spill in the fused decoder is paid every step of every lane."""
import os
import struct

import msgpack
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_11337_amd", "libboa.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libboa.so not built")


def _kernels():
    """{mangled name: metadata} of every gfx950 code object in libboa.so."""
    blob = open(LIB, "rb").read()
    out = {}
    at = blob.find(b"\x7fELF", 1)
    while at >= 0:
        if blob[at + 18:at + 20] == struct.pack("<H", 224):            # EM_AMDGPU
            phoff, = struct.unpack_from("<Q", blob, at + 32)
            phsize, phnum = struct.unpack_from("<HH", blob, at + 54)
            for i in range(phnum):
                kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", blob, at + phoff + i * phsize)
                p, end = at + off, at + off + size
                while kind == 4 and p + 12 <= end:                     # PT_NOTE
                    nlen, dlen, ntype = struct.unpack_from("<III", blob, p)
                    d = p + 12 + (nlen + 3) // 4 * 4
                    if ntype == 32 and blob[p + 12:p + 18] == b"AMDGPU":
                        for k in msgpack.unpackb(blob[d:d + dlen])["amdhsa.kernels"]:
                            out[k[".name"]] = k
                    p = d + (dlen + 3) // 4 * 4
        at = blob.find(b"\x7fELF", at + 1)
    return out


def test_fused_decoder_keeps_its_registers():
    ks = {n: k for n, k in _kernels().items() if "k_dec_fused" in n}
    assert len(ks) == 69                       # 3 dtypes x (d_model 64, 128, 256: 6 forms; 512: 5)
    bad = {n: k[".vgpr_spill_count"] for n, k in ks.items() if k[".vgpr_spill_count"] > 16}
    assert not bad
