"""What the built kernels ask of a compute unit, read from the metadata of the code objects in libssd.so.  CPU only."""
import os
import struct

import msgpack
import pytest


def _code_objects(blob):
    """The gfx950 ELF images of the offload bundles in a shared library: header {magic, count, count x (offset, size, length of id, id)}."""
    magic, at, out = b"__CLANG_OFFLOAD_BUNDLE__", 0, []
    while (at := blob.find(magic, at)) >= 0:
        n, p = struct.unpack_from("<Q", blob, at + 24)[0], at + 32
        for _ in range(n if n <= 16 else 0):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if size and b"gfx950" in name:
                out.append(blob[at + off:at + off + size])
        at += 24
    return out


def _kernels(elf):
    """The kernels' entries in the AMDGPU metadata note (type 32, MessagePack) of a 64-bit little-endian ELF."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        _, kind, _, _, off, length = struct.unpack_from("<IIQQQQ", elf, shoff + i * size)
        if kind != 7:                        # SHT_NOTE
            continue
        p = off
        while p < off + length:
            namesz, descsz, note = struct.unpack_from("<III", elf, p)
            desc = p + 12 + (namesz + 3 & ~3)
            if note == 32 and elf[p + 12:p + 18] == b"AMDGPU":
                return msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            p = desc + (descsz + 3 & ~3)
    return []


@pytest.fixture(scope="module")
def kernels():
    import paper_2505_15380_amd as pkg
    if not os.path.exists(pkg.library_path()):
        import __graft_entry__ as g
        g.build()
    blob = open(pkg.library_path(), "rb").read()
    out = {k[".name"]: k for elf in _code_objects(blob) for k in _kernels(elf)}
    assert sum("k_accept" in n for n in out) == 3 and sum("k_forward_dataflow" in n for n in out) == 5, sorted(out)
    return out


def test_no_kernel_spills(kernels):
    """A kernel whose registers do not suffice keeps the rest in scratch memory: the sampler for vocabularies of 8193 to 16384 took
    up to twice its time that way.  The forward with grid barriers, which runs where the barrier-free one does not fit, is known to."""
    spilling = {n: k[".private_segment_fixed_size"] for n, k in kernels.items() if k[".private_segment_fixed_size"]}
    assert not [n for n in spilling if "k_forward_persistent" not in n], spilling
