"""Register use of the built kernels, from the notes the compiler leaves in the library's code objects."""
import os
import re
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


def workgroups(metadata):
    """Workgroups that a compute unit has registers for: 512 per lane and SIMD, given out in eights."""
    return 512 // (-(-metadata[".vgpr_count"] // 8) * 8)


def generic(kernel):
    """Template arguments -> metadata of the generic kernels of that name (256 threads: a wavefront per SIMD)."""
    found = {}
    for name, k in kernels().items():
        m = re.search(rf"\d{kernel}I((?:L[ib]\d+E)+)E", name)
        if m:
            found[tuple(map(int, re.findall(r"L[ib](\d+)E", m.group(1))))] = k
    assert found, f"no {kernel}"
    return found


F32, BF16, FP8 = (pb.DTYPE_CODE[t] for t in ("f32", "bf16", "fp8_e4m3"))


def test_generic_draft_keeps_its_workgroups_per_compute_unit():
    """With a workgroup fewer per compute unit, 600 (request, head) pairs took up to a third longer than before the contractions went to
    the matrix cores."""
    for (_, kv, d), k in generic("decode_generic").items():
        least = (2 if kv == FP8 else 3) if d == 64 else 2 if kv == F32 else 1
        assert workgroups(k) >= least and k[".vgpr_spill_count"] == 0, (kv, d, k[".vgpr_count"], k[".vgpr_spill_count"])


def test_generic_verification_keeps_its_workgroups_per_compute_unit():
    """Chunks of 32 tokens run with up to four workgroups per compute unit.  With head_dim 128 the split kernel holds three, and so does the
    form of the finish kernel that sends for queries and partials early (fp8 two): the host takes that form only for launches that fit so."""
    fine = 32
    for (_, kv, d, chunk), k in generic("verify_split_generic").items():
        assert workgroups(k) >= (2 if chunk != fine else 4 if d == 64 else 3) and k[".vgpr_spill_count"] == 0, (kv, d, chunk, k[".vgpr_count"])
    early_forms = 0
    for (_, kv, d, chunk, merged, early), k in generic("verify_finish_generic").items():
        least = 2 if chunk != fine else 4 if d == 64 or not early else 2 if kv == FP8 else 3
        early_forms += chunk == fine and early
        assert workgroups(k) >= least and k[".vgpr_spill_count"] == 0, (kv, d, chunk, merged, early, k[".vgpr_count"])
    assert early_forms == 24
