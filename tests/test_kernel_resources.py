"""Registers and LDS of the built kernels, from the code objects' own metadata, where a launch plan counts on them."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2608_08097_amd", "liboasis.so")
SGPRS, VGPRS, LDS = 800, 512, 160 * 1024  # per SIMD, per SIMD lane, per CU


def _notes(elf):
    """Descriptors of the AMDGPU metadata notes of one code object."""
    off, (size, count) = struct.unpack_from("<Q", elf, 40)[0], struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        head = struct.unpack_from("<IIQQQQIIQQ", elf, off + i * size)
        if head[1] != 7:  # SHT_NOTE
            continue
        at, end = head[4], head[4] + head[5]
        while at + 12 <= end:
            name, desc, kind = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3) // 4 * 4
            if kind == 32:  # NT_AMDGPU_METADATA
                yield elf[at:at + desc]
            at += (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    """{demangled name: metadata} of every gfx950 kernel in the library."""
    msgpack = pytest.importorskip("msgpack")
    if not os.path.exists(LIB):
        from paper_2608_08097_amd.build_lib import build
        build()
    with open(LIB, "rb") as f:
        data = f.read()
    found, at, magic = [], 0, b"__CLANG_OFFLOAD_BUNDLE__"
    while (at := data.find(magic, at)) >= 0:
        pos = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, pos)
            if size and b"gfx950" in data[pos + 24:pos + 24 + n]:
                for note in _notes(data[at + off:at + off + size]):
                    found += msgpack.unpackb(note)["amdhsa.kernels"]
            pos += 24 + n
        at += len(magic)
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), capture_output=True, text=True,
                           check=True).stdout.split("\n")
    out = {re.sub(r"^void |oasis::|\(anonymous namespace\)::|\(.*", "", n): k for n, k in zip(names, found)}
    assert len(out) == len(found) > 20
    return out


def waves_per_simd(k):
    vgprs = -(-k[".vgpr_count"] // 8) * 8  # AGPRs included
    sgprs = -(-k[".sgpr_count"] // 16) * 16 + 16  # 16 for the trap handler
    return min(8, VGPRS // vgprs, SGPRS // sgprs)


def test_two_selections_share_a_cu(kernels):
    """512 rows of up to 16,384 blocks are one round of 1,024-thread workgroups, two per CU."""
    for keys in (4, 8, 16):
        k = kernels[f"topk_kernel<1024, {keys}>"]
        assert waves_per_simd(k) == 8, (keys, k[".sgpr_count"], k[".vgpr_count"])
        assert 2 * k[".group_segment_fixed_size"] <= LDS
    k = kernels["topk_kernel<512, 4>"]  # four rows of up to 2,048 blocks
    assert waves_per_simd(k) == 8 and 4 * k[".group_segment_fixed_size"] <= LDS


def test_many_row_attention_and_staging_exclude_each_other(kernels):
    """What the plan of a pipelined step counts on: two teams and a staging workgroup do not share a CU, two of the
    one-team form do, and so do a workgroup of up to two row tiles and a staging one."""
    stage = {n: k[".group_segment_fixed_size"] for n, k in kernels.items() if n.startswith("stage_kernel<")}
    for n, k in kernels.items():
        lds = k[".group_segment_fixed_size"]
        if m := re.match(r"attn_split_rows_kernel<(\d), (\d)", n):
            assert (lds + min(stage.values()) > LDS) if m[2] == "2" else (2 * lds <= LDS), n
        elif n.startswith("attn_split_kernel<"):
            assert lds + stage["stage_kernel<16, 1>"] <= LDS and lds + stage["stage_kernel<32, 1>"] <= LDS, n
