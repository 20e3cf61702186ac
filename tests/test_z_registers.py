"""Registers of the z solve kernels in the built library (its code objects' own
metadata): the near-singular lines and the zero mode, compiled into the same
kernels, leave the tile code the waves per SIMD that it reaches by itself.  A
workgroup of 1024 threads needs 4 or 8 waves on each SIMD, of 512 two more each."""
import os
import re
import struct

import pytest

from paper_2103_15187_amd import fsei

msgpack = pytest.importorskip("msgpack")

pytestmark = pytest.mark.skipif(not os.path.exists(fsei.LIB_PATH), reason="libfsei.so not built")

# waves per SIMD of the tile code by itself: (elem, modes per lane) -> {rows per chunk: waves}
WAVES = {("f", 1): {4: 8, 8: 8, 12: 8, 16: 4, 24: 4, 32: 4}, ("f", 2): {4: 8, 8: 8, 12: 6, 16: 4, 24: 3, 32: 4},
         ("f", 4): {4: 5, 8: 4, 12: 3, 16: 2, 24: 2},
         ("d", 1): {4: 8, 8: 5, 12: 5, 16: 4, 24: 2, 32: 2}, ("d", 2): {4: 6, 8: 4, 12: 3, 16: 2, 24: 2}}


def _kernels():
    """name -> metadata of every kernel of the gfx950 code objects in the library."""
    blob = open(fsei.LIB_PATH, "rb").read()
    out = {}
    for m in re.finditer(b"\x7fELF\x02\x01\x01\x40", blob):     # ELF of the AMDGPU HSA ABI
        o = m.start()
        phoff, = struct.unpack_from("<Q", blob, o + 32)
        size, num = struct.unpack_from("<HH", blob, o + 54)
        for i in range(num):
            kind, _, off, _, _, length = struct.unpack_from("<IIQQQQ", blob, o + phoff + i * size)[:6]
            if kind != 4:                                       # PT_NOTE
                continue
            at, end = o + off, o + off + length
            while at < end:
                nlen, dlen, note = struct.unpack_from("<III", blob, at)
                data = at + 12 + (nlen + 3) // 4 * 4
                if note == 32:                                  # AMDGPU metadata
                    meta = msgpack.unpackb(blob[data:data + dlen], strict_map_key=False)
                    for k in meta.get("amdhsa.kernels", []):
                        out[k[".name"]] = k
                at = data + (dlen + 3) // 4 * 4
    return out


def test_tile_code_keeps_its_waves():
    seen = 0
    for name, k in _kernels().items():
        m = re.match(r"_ZN4fsei3dev8k_zsolveI([fd])[fd]Li\d+ELi(\d+)ELi(\d+)E", name)
        modes, rows = (1, int(m.group(2))) if m else (0, 0)
        if not m:
            m = re.match(r"_ZN4fsei3dev9k_zsolvevI([fd])[fd]Li(\d+)ELi\d+ELi(\d+)ELi(\d+)E", name)
            if not m:
                continue
            modes, rows = int(m.group(2)), int(m.group(3))
        seen += 1
        regs = (k[".vgpr_count"] + 7) // 8 * 8
        assert min(8, 512 // regs) >= WAVES[m.group(1), modes][rows], (name, regs)
    assert seen >= 20
