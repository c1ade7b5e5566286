"""Register budgets of the built kernels, read from the metadata of the gfx950 code objects in the
library (no GPU needed): values that a kernel holds and that do not fit its registers go to scratch
memory, which costs time and changes no result, so that only a check like this one sees it.
"""
import re
import struct

import pytest

from paper_1406_7416_amd import adg

msgpack = pytest.importorskip("msgpack")


def code_objects(blob):
    """The gfx950 ELF images of the library's offload bundles."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        count, o = struct.unpack_from("<Q", blob, at + 24)[0], at + 32
        for _ in range(count):
            off, size, tlen = struct.unpack_from("<QQQ", blob, o)
            if b"gfx950" in blob[o + 24:o + 24 + tlen]:
                yield blob[at + off:at + off + size]
            o += 24 + tlen
        at += len(magic)


def kernels():
    """{mangled name: metadata} of every kernel (the AMDGPU metadata note of each image)."""
    out = {}
    with open(adg.LIB_PATH, "rb") as f:
        blob = f.read()
    for elf in code_objects(blob):
        phoff, = struct.unpack_from("<Q", elf, 32)
        phsize, phnum = struct.unpack_from("<HH", elf, 54)
        for i in range(phnum):
            kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phsize)
            if kind != 4:   # PT_NOTE
                continue
            end = off + size
            while off + 12 <= end:
                nlen, dlen, ntype = struct.unpack_from("<III", elf, off)
                desc = off + 12 + (nlen + 3) // 4 * 4
                if ntype == 32 and elf[off + 12:off + 18] == b"AMDGPU":
                    for k in msgpack.unpackb(elf[desc:desc + dlen])["amdhsa.kernels"]:
                        out[k[".name"]] = k
                off = desc + (dlen + 3) // 4 * 4
    return out


@pytest.fixture(scope="module")
def built():
    found = kernels()
    assert len(found) > 100
    return found


FORM = {"fp64": "dLb0", "mixed": "fLb0", "dev": "fLb1"}
WIDTH = {"fp64": 8, "mixed": 4, "dev": 4}


def predictor(built, dim, N, form):
    """The metadata of the single problem's predictor of a class."""
    name = [k for k in built if re.match(rf"_ZN3adg11k_predictorILi{dim}ELi{N}ELb1E{FORM[form]}E", k)]
    assert len(name) == 1, name
    return built[name[0]]


@pytest.mark.parametrize("form", ["fp64", "mixed", "dev"])
def test_predictor_3d_degree_9_scratch(built, form):
    """A workgroup of 1024 threads leaves a lane 128 registers, fewer than the pencil and the flux
    sums of a node take in FP64 (2 x 5 x 10 values): scratch has to hold those, and the operands of
    a sum not besides (2196 bytes of them and all when the volume term's sums were sunk into the
    branch that stores them).  Bound: twice the pencil and the flux sums."""
    values = 2 * 5 * 10
    assert predictor(built, 3, 9, form)[".private_segment_fixed_size"] <= 2 * values * WIDTH[form]


@pytest.mark.parametrize("N", range(1, 10))
def test_predictor_2d_fp64_pencils_in_registers(built, N):
    """A lane's 256 registers (168 where three waves share a SIMD) hold the pencil and the flux sums
    of a 2D node, at most 2 x 4 x 10 values.  In chunks of variables whose loop is not unrolled
    they are indexed arrays and live in scratch: less scratch than one pencil shows that they do not."""
    assert predictor(built, 2, N, "fp64")[".private_segment_fixed_size"] < 4 * (N + 1) * WIDTH["fp64"]


def test_predictor_2d_degree_9_deviation_form_sweep_in_registers(built):
    """A lane's 128 registers hold the pencil and the flux sums of a 2D node in the deviation form
    (2 x 4 x 10 values); what is spilled are the values formed once per cell or kernel besides
    them, fewer than 50 (57 with flux sums among them)."""
    assert predictor(built, 2, 9, "dev")[".vgpr_spill_count"] < 50


@pytest.mark.parametrize("real", ["d", "f"])
def test_corrector_of_large_cells_spills_nothing(built, real):
    """One cell after the other in a workgroup: nothing of a cell's index arithmetic is to be kept
    from cell to cell, and 256 registers hold the 20 values of a thread with their indices.  The
    projection's 19 x 10 entries (380 scalar registers) are not to be held and spilled either."""
    name = [k for k in built if k.startswith(f"_ZN3adg18k_corrector_detectILi3ELi9E{real}E")]
    assert len(name) == 1 and built[name[0]][".vgpr_spill_count"] == 0
    assert built[name[0]][".sgpr_spill_count"] < 380


def test_predictor_3d_degree_9_fp64_time_operator_not_held(built):
    """The time operator's 10 x 10 entries take 200 scalar registers, twice what a wave has: fewer
    spilled ones show that they are loaded row by row."""
    assert predictor(built, 3, 9, "fp64")[".sgpr_spill_count"] < 200
