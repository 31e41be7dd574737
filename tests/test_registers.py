"""Register use of the built kernels, from the notes the compiler leaves in the library's code objects."""
import os
import struct

import msgpack
import pytest

from paper_2512_01278_amd import binding as pb

AMDGPU, NOTES = 224, 7                 # ELF machine, section type


def kernels():
    """Name -> metadata of every kernel in the library's gfx950 code objects."""
    if not os.path.exists(pb.LIB_PATH):
        from paper_2512_01278_amd.build import build
        build(verbose=False)
    blob = open(pb.LIB_PATH, "rb").read()
    found, at = {}, blob.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == AMDGPU:
            (table,), (size, count) = struct.unpack_from("<Q", blob, at + 40), struct.unpack_from("<HH", blob, at + 58)
            for i in range(count):
                kind, where, length = struct.unpack_from("<4xI16xQQ", blob, at + table + i * size)
                if kind == NOTES:
                    name_len, desc_len = struct.unpack_from("<II", blob, at + where)
                    start = at + where + 12 + (name_len + 3) // 4 * 4
                    for k in msgpack.unpackb(blob[start:start + desc_len]).get("amdhsa.kernels", []):
                        found[k[".name"]] = k
        at = blob.find(b"\x7fELF", at + 4)
    return found


def test_finish_kernels_spill_no_registers():
    """A workgroup of the finish kernel has 128 registers per lane (two of 512 threads or one of 1024 share a compute unit), in which the
    stash on its way, the partials of a split pair and the keys of up to four chunks have to fit."""
    all_ = kernels()
    finish = {n: k for n, k in all_.items() if "13verify_finishIL" in n}
    if not finish:
        pytest.fail(f"no finish kernel among {len(all_)} kernels")
    bad = {n: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for n, k in finish.items() if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert len(finish) == 28 and not bad, bad
