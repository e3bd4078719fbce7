"""Register budgets of the built kernels, from the metadata of the code objects inside the library."""
import re
import struct

import pytest

from paper_2605_05607_amd import build

msgpack = pytest.importorskip("msgpack")


def code_objects(blob):
    """gfx950 code objects of the library's offload bundles (uncompressed bundles of one entry per target)."""
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob):
        at = m.start()
        n, = struct.unpack_from("<Q", blob, at + 24)
        if n > 16:
            continue  # the magic inside some string
        p = at + 32
        for _ in range(n):
            off, size, id_len = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + id_len]
            p += 24 + id_len
            if name.endswith(b"gfx950"):
                yield blob[at + off:at + off + size]


def kernels(elf):
    """Metadata of the code object's kernels: the note of type 32 (msgpack)."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        sh = shoff + i * shentsize
        if struct.unpack_from("<I", elf, sh + 4)[0] != 7:  # SHT_NOTE
            continue
        off, size = struct.unpack_from("<QQ", elf, sh + 24)
        p = off
        while p < off + size:
            namesz, descsz, kind = struct.unpack_from("<III", elf, p)
            desc = p + 12 + (namesz + 3) // 4 * 4
            if kind == 32:
                yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            p = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def table():
    with open(build.LIB, "rb") as fh:
        blob = fh.read()
    out = {k[".name"]: k for obj in code_objects(blob) for k in kernels(obj)}
    assert len(out) > 50
    return out


def test_backward_gemms_leave_room_beside_them(table):
    # A SIMD has 512 registers, allocated by eights: two waves of at most 248 leave one transpose wave (16) its place.
    # Instances <GATED, FP8, TRAIN, FAR = false, BESIDE = true>.
    gemms = [k for n, k in table.items() if re.search(r"gemm_bf16_kernelILb0ELb0ELb[01]ELb0ELb1E", n)]
    beside = [k for n, k in table.items() if re.search(r"gather_transpose_kernel|wgrad_blocks_kernel", n)]
    assert len(gemms) == 2 and len(beside) == 2
    for k in gemms:
        assert k[".vgpr_count"] <= 248 and k[".vgpr_spill_count"] == 0, k[".name"]
    transpose = next(k for k in beside if "transpose" in k[".name"])
    assert transpose[".vgpr_count"] <= 16
    # LDS of a CU: 160 KiB, 128 KiB of it requested by these GEMMs
    assert 128 * 1024 + 3 * transpose[".group_segment_fixed_size"] <= 160 * 1024


def test_gemm_kernels_do_not_spill(table):
    for name, k in table.items():
        if re.search(r"gemm|wgrad|router_logits", name):
            assert k[".vgpr_spill_count"] == 0, (name, k[".vgpr_spill_count"])
