"""Registers and scratch memory of the generic step kernels, as the compiler
wrote them into the built library: what decides how many waves fit a SIMD."""
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")


def code_objects(blob):
    """The gfx950 ELF images of every offload bundle in the library."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        p = at + len(magic)
        (n,) = struct.unpack_from("<Q", blob, p)
        p += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if name.endswith(b"gfx950"):
                yield blob[at + off:at + off + size]
        at = blob.find(magic, at + 1)


def kernel_records(elf):
    """amdhsa.kernels of the AMDGPU metadata note (type 32)."""
    (shoff,) = struct.unpack_from("<Q", elf, 40)
    entsize, num = struct.unpack_from("<HH", elf, 58)
    for i in range(num):
        kind, = struct.unpack_from("<I", elf, shoff + i * entsize + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + i * entsize + 24)
        if kind != 7:  # SHT_NOTE
            continue
        namesz, descsz, ntype = struct.unpack_from("<III", elf, off)
        if ntype != 32:
            continue
        desc = off + 12 + (namesz + 3) // 4 * 4
        yield from msgpack.unpackb(elf[desc:desc + descsz], strict_map_key=False)["amdhsa.kernels"]


@pytest.fixture(scope="module")
def kernels(okpz):
    out = {}
    blob = open(okpz.LIB_PATH, "rb").read()
    for elf in code_objects(blob):
        for k in kernel_records(elf):
            out[k[".name"]] = k
    assert out
    return out


def find(kernels, pattern):
    got = [k for name, k in kernels.items() if re.search(pattern, name)]
    assert got, pattern
    return got


# scheme 0 DT, 2 DTr; cells per lane; whether attempts draw for acceptance
@pytest.mark.parametrize("scheme", [0, 2])
@pytest.mark.parametrize("accept,cpt,waves,scratch", [(0, 1, 8, 0), (0, 4, 7, 0), (1, 1, 8, 0), (1, 2, 8, 0),
                                                      (1, 4, 6, 0), (1, 8, 3, 0), (1, 16, 2, 44)])
def test_generic_dt_step_keeps_its_waves(kernels, scheme, accept, cpt, waves, scratch):
    (k,) = find(kernels, r"okpz11step_kernelILi%dELb%dELi%dEE" % (scheme, accept, cpt))
    assert 512 // (-(-k[".vgpr_count"] // 8) * 8) >= waves
    assert k[".private_segment_fixed_size"] <= scratch


@pytest.mark.parametrize("scheme,cpt,scratch", [(0, 4, 52), (2, 4, 52), (0, 16, 276), (2, 16, 268)])
def test_generic_dt_batch_scratch(kernels, scheme, cpt, scratch):
    (k,) = find(kernels, r"batch_kernelILi%dELi%dELb0ELi0ELi0ELi0E" % (scheme, cpt))
    assert k[".private_segment_fixed_size"] <= scratch


# scalar registers spilled by the generic sweeps of the batch: each is a lane move in the loop over the items
@pytest.mark.parametrize("scheme,cpt,spills", [(0, 1, 22), (0, 2, 31), (2, 1, 27), (2, 2, 34), (1, 1, 65), (1, 2, 82)])
def test_generic_batch_scalar_spills(kernels, scheme, cpt, spills):
    for k in find(kernels, r"batch_kernelILi%dELi%dELb0ELi0ELi0ELi0E" % (scheme, cpt)):
        assert k[".sgpr_spill_count"] <= spills
