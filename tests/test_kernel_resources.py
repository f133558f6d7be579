"""The built library's kernels keep their values in registers (read from the code objects' own metadata)."""
import struct

import msgpack
import pytest

import paper_2609_26300_amd as P
from paper_2609_26300_amd import binding as B


def _kernels(path):
    """The metadata records of every gfx950 kernel in a shared library built by this repository."""
    data = open(path, "rb").read()
    out = []
    at = data.find(b"\x7fELF", 1)
    while at > 0:
        if struct.unpack_from("<H", data, at + 18)[0] == 224:  # EM_AMDGPU
            shoff, = struct.unpack_from("<Q", data, at + 40)
            shentsize, shnum = struct.unpack_from("<HH", data, at + 58)
            for i in range(shnum):
                kind, = struct.unpack_from("<I", data, at + shoff + i * shentsize + 4)
                off, size = struct.unpack_from("<QQ", data, at + shoff + i * shentsize + 24)
                if kind != 7:  # SHT_NOTE
                    continue
                p, end = at + off, at + off + size
                while p < end:
                    nsz, dsz, what = struct.unpack_from("<III", data, p)
                    desc = p + 12 + (nsz + 3) // 4 * 4
                    if what == 32:  # NT_AMDGPU_METADATA
                        out += msgpack.unpackb(data[desc:desc + dsz], strict_map_key=False)["amdhsa.kernels"]
                    p = desc + (dsz + 3) // 4 * 4
        at = data.find(b"\x7fELF", at + 4)
    return out


@pytest.fixture(scope="module")
def kernels():
    P.library()
    ks = _kernels(B.LIB_PATH)
    assert len(ks) > 100
    return ks


def test_kernels_do_not_spill(kernels):
    """No kernel keeps values in scratch memory. (The small wave build holds two words there for the recomputation
    after its loop, which no ordinary input reaches.) A streaming-shape kernel that spilled 368 bytes took
    1.4 to 1.5 times as long."""
    spilled = {k[".name"]: k[".private_segment_fixed_size"] for k in kernels if k[".private_segment_fixed_size"] > 0}
    allowed = {n: b for n, b in spilled.items() if "build_stats_wave_kernelILi" in n and b <= 8}
    assert spilled == allowed


def test_scoring_of_few_groups_keeps_its_residency(kernels):
    """The chunk scoring of up to 32 variance groups holds at least four waves per SIMD (128 registers), as without the
    variances in flight; only the kernel of more groups takes more."""
    few = [k[".vgpr_count"] for k in kernels
           if "score_chunks_kernelILi" in k[".name"] and k[".name"].split("EEEv")[0].endswith(("ELi1", "ELi4"))]
    assert len(few) == 2 * 2 * 4 * 2 * 3  # (groups kept per lane, head sizes, query heads, step or call, slots)
    assert max(few) <= 128


def test_scoring_call_keeps_its_lds(kernels):
    """The scoring call's chunk workgroups (no append) hold no partial sums of a summary: eight fit the 160 KB of a
    compute unit."""
    lds = [k[".group_segment_fixed_size"] for k in kernels
           if "score_chunks_kernelILi" in k[".name"] and "ELb0E" in k[".name"]]
    assert lds and max(lds) * 8 <= 160 * 1024
