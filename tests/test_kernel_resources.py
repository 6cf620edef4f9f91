"""Registers and scratch of the compiled kernels, read from the metadata in the
library (no GPU needed): nothing spills, and the kernels whose launches count on
two workgroups per CU have the registers for it (a SIMD holds 512: 8 wavefronts
at 64, 4 at 128, 3 at 168)."""
import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2005_08028_amd", "libscitv.so")


def _notes(elf):
    shoff, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        if struct.unpack_from("<I", elf, shoff + i * size + 4)[0] != 7:  # SHT_NOTE
            continue
        at, n = struct.unpack_from("<QQ", elf, shoff + i * size + 24)
        end = at + n
        while at < end:
            name, desc, kind = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3) // 4 * 4
            if kind == 32:  # AMDGPU metadata
                yield msgpack.unpackb(elf[at:at + desc])
            at += (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(LIB):
        from paper_2005_08028_amd import build as hipbuild
        hipbuild.build()
    blob = open(LIB, "rb").read()
    magic, out, at = b"__CLANG_OFFLOAD_BUNDLE__", {}, 0
    while (at := blob.find(magic, at)) >= 0:
        entries, = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(entries):
            off, size, n = struct.unpack_from("<QQQ", blob, p)
            target = blob[p + 24:p + 24 + n]
            p += 24 + n
            if b"amdgcn" in target and size:
                for note in _notes(blob[at + off:at + off + size]):
                    out.update({k[".name"]: k for k in note["amdhsa.kernels"]})
        at += len(magic)
    assert len(out) > 1000
    return out


def _templates(kernels, name):
    """{template arguments: registers} of the instantiations of one kernel."""
    out = {}
    for mangled, k in kernels.items():
        m = re.search(r"\d" + name + r"I((?:Li\d+E)+)E", mangled)
        if m:
            out[tuple(int(v) for v in re.findall(r"Li(\d+)E", m.group(1)))] = k[".vgpr_count"]
    assert out
    return out


def test_no_scratch(kernels):
    assert not [n for n, k in kernels.items() if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]]


def test_tall_tile_runs_two_workgroups(kernels):
    # 16 wavefronts of 5 rows a lane: the cost model counts two of them per CU
    tiles = {t: v for t, v in _templates(kernels, "k_fgp_tile").items() if t[3:6] == (5, 16, 1)}
    assert len(tiles) == 20 and max(tiles.values()) <= 64


# (M, frames, mode, Chambolle-2004, dual type, records) beyond the rule below: these
# cross 128 registers in every form ...
OVER = {(2, 4, 0, 1, 0, 0), (4, 2, 2, 0, 0, 0), (4, 2, 2, 0, 0, 1), (4, 2, 2, 0, 1, 0), (4, 2, 2, 0, 1, 2),
        (4, 2, 2, 0, 2, 0), (4, 2, 2, 0, 2, 2), (5, 2, 1, 0, 0, 0), (5, 2, 1, 0, 0, 1), (5, 2, 1, 0, 2, 0),
        (6, 2, 0, 0, 0, 0), (6, 2, 0, 0, 0, 2), (6, 2, 0, 0, 1, 0), (6, 2, 0, 0, 2, 0)}
# ... and these do not
UNDER = {(5, 2, 2, 0, 1, 3), (5, 2, 2, 0, 2, 3)}


def test_vtv_passes_hold_two_workgroups(kernels):
    short = {2: 6, 3: 3, 4: 2}  # largest M + mode at 128 registers, by frames per wavefront
    missed = {t: v for t, v in _templates(kernels, "k_vtv_rows").items()
              if t[1] > 1 and v > 128 and (t[0] + t[2] <= short[t[1]] and t[:6] not in OVER or t[:6] in UNDER)}
    # five slots serve five wavefronts, of which two workgroups fit at 168 too
    assert not {t: v for t, v in missed.items() if t[6] == 8}
    assert all(v <= 168 for v in missed.values())
