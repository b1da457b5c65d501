"""The built host extension, as a file."""
import glob
import os
import struct

import paper_2602_03681_amd


def test_it_has_no_thread_local_variables():
    """glibc 2.35 looks every thread-local variable of a process up the slow way once a library with some has been loaded and none
    of its own is touched."""
    (path,) = glob.glob(os.path.join(os.path.dirname(paper_2602_03681_amd.__file__), "_nats_host*.so"))
    with open(path, "rb") as f:
        elf = f.read()
    assert elf[:5] == b"\x7fELF\x02"
    at, (size, n) = struct.unpack_from("<Q", elf, 32)[0], struct.unpack_from("<HH", elf, 54)
    kinds = [struct.unpack_from("<I", elf, at + i * size)[0] for i in range(n)]
    assert 1 in kinds and 7 not in kinds        # PT_LOAD, PT_TLS
