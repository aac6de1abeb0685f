"""Registers of the compiled prefill kernels: what their main instantiations
spill to scratch memory, read from the metadata of the library built here."""
import re
import struct

import msgpack

from paper_2607_24788_amd import glide


def kernels():
    """name -> metadata of every device kernel in the library (the AMDGPU
    metadata notes, type 32, of its embedded code objects)."""
    blob = open(glide.LIB_PATH, "rb").read()
    out = {}
    for m in re.finditer(re.escape(struct.pack("<I", 32) + b"AMDGPU\0\0"), blob):
        n = struct.unpack_from("<I", blob, m.start() - 4)[0]  # namesz, descsz, type, name, desc
        for k in msgpack.unpackb(blob[m.end():m.end() + n], strict_map_key=False)["amdhsa.kernels"]:
            out[k[".name"]] = k
    return out


def test_prefill_main_spills():
    """fp32 at d = 128 holds S, the band's fragments and the queries in more
    registers than there are, and spills some; the limits are the counts of
    kernels timed without a loss (twice as many cost 3 to 11% per call).
    Everything else fits, up to a few."""
    seen = 0
    for name, k in kernels().items():
        m = re.search(r"prefill_mainI([tf])Li(\d+)ELi(\d+)ELi(\d)ELi(\d)ELb(\d)ELi(\d+)E", name)
        if not m:
            continue
        seen += 1
        t, (d, df, phi, part, gated, rows) = m[1], (int(x) for x in m.groups()[1:])
        limit = 20
        if t == "f" and rows == 256:
            if d == 128 and part == 0:
                limit = 270 if df == 128 else 90
            elif part == 1:
                limit = 60 if (d, df) == (128, 128) else 0
            elif part == 0:
                limit = 45 if df == 128 else 0
            else:
                limit = 30
        elif t == "f" and rows == 128 and (d, df) == (128, 128):
            limit = 60
        elif t == "t" and (d, df) == (128, 64) and not gated:
            limit = 0
        assert k[".vgpr_spill_count"] <= limit, f"{name}: {k['.vgpr_spill_count']} registers spilled, limit {limit}"
    assert seen >= 200
