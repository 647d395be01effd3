"""What the compiler gave the kernels of the built library: registers and scratch, from the metadata notes of its
gfx950 code objects.  A kernel that spills without saying so, or whose registers cost it a wave on every SIMD, shows
in no result and in few timings."""
import re
import struct
import subprocess

import msgpack
import pytest

from paper_1812_11214_amd import binding, build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def notes(elf):
    """Descriptors of the AMDGPU metadata notes (type 32) of an ELF image."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        head = shoff + i * size
        if struct.unpack_from("<I", elf, head + 4)[0] != 7:  # SHT_NOTE
            continue
        at, length = struct.unpack_from("<QQ", elf, head + 24)
        end = at + length
        while at < end:
            name, desc, kind = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3) // 4 * 4
            if kind == 32:
                yield elf[at:at + desc]
            at += (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    """{name without namespaces and arguments: metadata} of every kernel."""
    binding.lib()
    blob, at, found = open(build.LIB, "rb").read(), 0, {}
    while (at := blob.find(MAGIC, at)) >= 0:
        entries, = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(entries if entries < 16 else 0):
            offset, size, chars = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + chars]
            p += 24 + chars
            if b"gfx950" in triple and size:
                for desc in notes(blob[at + offset:at + offset + size]):
                    found.update({k[".name"]: k for k in msgpack.unpackb(desc)["amdhsa.kernels"]})
        at += len(MAGIC)
    assert found
    names = subprocess.run(["c++filt"], input="\n".join(found), text=True, capture_output=True, check=True).stdout
    short = [re.search(r"(k\w+(?:<.*>)?)\(", n.replace("(anonymous namespace)::", "")) for n in names.split("\n")[:len(found)]]
    assert all(short), names
    return {m.group(1): k for m, k in zip(short, found.values())}


def test_plain_row_transforms_keep_their_waves(kernels):
    """k_row_fwd_reg shares its body with the planar rows, whose runs need more registers: 512 / registers waves."""
    for name, most in (("<16, 1>", 64), ("<16, 2>", 72), ("<16, 4>", 72), ("<16, 8>", 72), ("<16, 16>", 88),
                       ("<32, 16>", 144)):
        assert kernels["k_row_fwd_reg" + name][".vgpr_count"] <= most, name


# Kernels that keep part of a lane's state in scratch memory, and the bytes a lane.  Each says so at its launch
# bounds or is measured as the faster one with it.
SCRATCH = {
    "k_node_half<1, 1, false, false, 8>": 32,
    "k_node_half<1, 1, false, false, 16>": 216,
    "k_node_half<2, 1, false, true, 4>": 56,
    "k_node_half<4, 1, false, true, 4>": 56,
    "k_line_nodes<true, true>": 20,
    "k_plane_nodes<128, 128, true>": 56,
    "k_node_modback<128, 128, false, true>": 40,
    "k_node_modback<128, 128, true, true>": 44,
    "k_rows1d_reg<16, 16, false>": 12,
    "k_rows1d_reg<16, 16, true>": 8,
    "k_rows1d_adj<16, 4>": 12,
    "k3_slab_fwd_mulacc<128, 128>": 16,
    "k3_slab_fwd_mulacc<64, 256>": 8,
}


def test_no_other_kernel_uses_scratch(kernels):
    used = {name: k[".private_segment_fixed_size"] for name, k in kernels.items() if k[".private_segment_fixed_size"]}
    assert set(used) <= set(SCRATCH), used
    assert all(size <= SCRATCH[name] for name, size in used.items()), used
