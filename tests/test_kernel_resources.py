"""Registers of the 2D step kernels in the built library: the waves per SIMD that
the default geometries count on have to fit (512 registers a lane on gfx950, in
steps of 8)."""
import re
import struct

import msgpack
import pytest

from paper_2110_12448_amd import pfiso


def _kernels():
    """Metadata of every device kernel: the code objects' amdhsa notes."""
    pfiso.load()
    blob, out, at = open(pfiso.LIB_PATH, "rb").read(), {}, 0
    while (at := blob.find(b"\x7fELF\x02\x01\x01\x40", at)) >= 0:   # ELF64, AMDGPU HSA
        shoff, = struct.unpack_from("<Q", blob, at + 40)
        shnum, = struct.unpack_from("<H", blob, at + 60)
        for k in range(shnum):
            _, kind, _, _, off, _ = struct.unpack_from("<IIQQQQ", blob, at + shoff + 64 * k)
            if kind == 7:                                           # SHT_NOTE
                name, size, _ = struct.unpack_from("<III", blob, at + off)
                desc = at + off + 12 + (name + 3) // 4 * 4
                for q in msgpack.unpackb(blob[desc:desc + size])["amdhsa.kernels"]:
                    out[q[".name"]] = q
        at += 8
    return out


def _step2d():
    """(precision, frozen, frame, multi, variant) -> (waves per SIMD, scratch bytes)."""
    out = {}
    for name, q in _kernels().items():
        m = re.search(r"step2d_kernelI([fd])Lb(\d)ELb(\d)ELb(\d)ELi(\d)E", name)
        if m:
            regs = -(-q[".vgpr_count"] // 8) * 8    # vector and accumulation registers
            out[(m[1],) + tuple(int(v) for v in m.groups()[1:])] = (
                512 // regs, q[".private_segment_fixed_size"])
    return out


APPROX_SHELLS, FULL_SHELLS, FULL_TWO_POINT, APPROX_TWO_POINT, DIFFUSION = range(5)


@pytest.mark.parametrize("precision,variants,multi,waves", [
    ("f", range(5), (0, 1), 4),
    ("d", (APPROX_SHELLS, APPROX_TWO_POINT, DIFFUSION), (0,), 3),
    ("d", range(5), (0, 1), 2),
])
def test_waves_per_simd(precision, variants, multi, waves):
    ks = _step2d()
    assert len(ks) == 2 * 2 * 2 * 2 * 5
    for k, (fit, scratch) in ks.items():
        if k[0] == precision and k[4] in variants and k[3] in multi:
            assert fit >= waves, k
            if precision == "f":
                assert scratch == 0, k
