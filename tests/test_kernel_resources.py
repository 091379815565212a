"""Registers and memory of the walk kernels, from the metadata of the built library: the words that a step
takes from its packet's stream stay in registers (no scratch, and no LDS beyond the census sums), where the
walks are bound by instruction issue and a word through memory is a dependent store and load per step."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1709_10187_amd", "librddmc.so")
NT_AMDGPU_METADATA = 32


def _code_objects(blob):
    """The gfx950 ELF files of every offload bundle in the library."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        n = struct.unpack_from("<Q", blob, at + 24)[0]
        p = at + 32
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", blob, p)
            if size and b"gfx950" in blob[p + 24:p + 24 + ln]:
                yield blob[at + off:at + off + size]
            p += 24 + ln
        at = blob.find(magic, at + 24)


def _kernels():
    """{demangled name without arguments: metadata} of the library's kernels."""
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    out = {}
    with open(LIB, "rb") as f:
        blob = f.read()
    for elf in _code_objects(blob):
        table = struct.unpack_from("<Q", elf, 40)[0]
        entry, count = struct.unpack_from("<HH", elf, 58)
        for i in range(count):
            h = table + i * entry
            if struct.unpack_from("<I", elf, h + 4)[0] != 7:   # SHT_NOTE
                continue
            p, size = struct.unpack_from("<QQ", elf, h + 24)
            end = p + size
            while p < end:
                ns, ds, kind = struct.unpack_from("<III", elf, p)
                d = p + 12 + ((ns + 3) & ~3)
                if kind == NT_AMDGPU_METADATA:
                    for k in msgpack.unpackb(elf[d:d + ds])["amdhsa.kernels"]:
                        out[k[".name"]] = k
                p = d + ((ds + 3) & ~3)
    names = list(out)
    plain = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True, check=True).stdout.split("\n")
    short = lambda s: s.split("(anonymous namespace)::")[1].split("(")[0]
    return {short(d): out[n] for n, d in zip(names, plain) if "(anonymous namespace)::" in d}


def _walks(prefix):
    got = {n: k for n, k in _kernels().items() if n.startswith(prefix)}
    assert got
    return got.items()


@pytest.mark.parametrize("prefix,lds", [("walk3d", 0), ("walk1dg", 0), ("walk1dh<", 32768), ("walk1dh_coop", 34816)])
def test_words_of_the_stream_stay_in_registers(prefix, lds):
    for name, k in _walks(prefix):
        census = name.startswith("walk1dh") and name.endswith("true>")   # path sums of census instantiations
        assert k[".group_segment_fixed_size"] <= (lds if census else 0), name
        # none but the few registers that a kernel held at four waves per SIMD spills
        held = k[".vgpr_count"] in (127, 128)
        assert k[".private_segment_fixed_size"] <= (48 if held else 0), name


def test_hybrid_walks_keep_their_waves_per_simd():
    """512 vector registers per SIMD lane, handed out in eights: four waves of the plain walks, three with
    weights or census estimators, two with both."""
    for name, k in _walks("walk1dh<"):
        sphere, single, weights, census = (v == "true" for v in re.findall("true|false", name))
        waves = 512 // (-(-k[".vgpr_count"] // 8) * 8)
        assert waves >= 4 - weights - census, name
