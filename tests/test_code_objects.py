"""Sizes of the code objects in the built library (no GPU).  The runtime loads a source file's code
object whole with the first kernel of it that a process launches, so files that hold kernels a
process does not run are paid for by its first call: with one object of 2.8 MB and others of 1.1
and 0.8 MB a first gradient took 6.7 ms where it had taken 3.3."""
import struct

from paper_2008_09042_amd import _lib

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects():
    """Bytes of every GPU code object bundled in the library."""
    blob = open(_lib.LIB_PATH, "rb").read()
    sizes, at = [], blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        if n <= 8:  # a bundle's header, not the string in some other section
            for _ in range(n):
                _, size, idlen = struct.unpack_from("<QQQ", blob, p)
                p += 24 + idlen
                if b"gfx950" in blob[p - idlen:p]:
                    sizes.append(size)
        at = blob.find(MAGIC, at + 1)
    return sizes


def test_no_code_object_is_large():
    sizes = code_objects()
    assert len(sizes) > 10
    assert max(sizes) <= 1.75 * 2**20, sorted(sizes)[-4:]
