"""Register use of the built kernels, where their speed rests on it: read from the
code objects' metadata notes in the library (no GPU)."""
import struct

import pytest

import paper_2501_00692_amd as ssm

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"
PT_NOTE, NT_AMDGPU_METADATA = 4, 32


def _unpack(b, i=0):
    """The MessagePack object at b[i] (the types that the notes use) and the index after it."""
    t = b[i]
    if t < 0x80 or t >= 0xe0:
        return (t if t < 0x80 else t - 256), i + 1
    if t in (0xc0, 0xc2, 0xc3):
        return {0xc0: None, 0xc2: False, 0xc3: True}[t], i + 1
    if t in (0xcc, 0xcd, 0xce, 0xcf, 0xd0, 0xd1, 0xd2, 0xd3):
        n = 1 << (t & 3)
        return int.from_bytes(b[i + 1:i + 1 + n], "big", signed=t >= 0xd0), i + 1 + n
    if 0xa0 <= t < 0xc0 or t in (0xd9, 0xda, 0xdb):
        w = 0 if t < 0xc0 else 1 << (t - 0xd9)
        n = int.from_bytes(b[i + 1:i + 1 + w], "big") if w else t & 31
        return b[i + 1 + w:i + 1 + w + n].decode(), i + 1 + w + n
    w = 0 if t < 0xa0 else 2 << (t & 1)  # arrays and maps
    n = int.from_bytes(b[i + 1:i + 1 + w], "big") if w else t & 15
    i += 1 + w
    pairs = t < 0x90 or t in (0xde, 0xdf)
    items = []
    for _ in range(2 * n if pairs else n):
        v, i = _unpack(b, i)
        items.append(v)
    return (dict(zip(items[::2], items[1::2])) if pairs else items), i


def _kernels_of(elf):
    phoff, = struct.unpack_from("<Q", elf, 32)
    phentsize, phnum = struct.unpack_from("<HH", elf, 54)
    for k in range(phnum):
        kind, _, at, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + k * phentsize)
        end = at + size if kind == PT_NOTE else at
        while at < end:
            name, desc, tag = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3) // 4 * 4
            if tag == NT_AMDGPU_METADATA:
                yield from _unpack(elf[at:at + desc])[0]["amdhsa.kernels"]
            at += (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    """{mangled name: metadata} of every gfx950 kernel of the library."""
    data, out = ssm.LIB_PATH.read_bytes(), {}
    at = data.find(BUNDLE)
    while at >= 0:
        entries, = struct.unpack_from("<Q", data, at + 24)
        o = at + 32
        for _ in range(entries):
            off, size, n = struct.unpack_from("<QQQ", data, o)
            if b"gfx950" in data[o + 24:o + 24 + n]:
                out.update((k[".name"], k) for k in _kernels_of(data[at + off:at + off + size]))
            o += 24 + n
        at = data.find(BUNDLE, at + 24)
    assert out
    return out


def _pick(kernels, *parts):
    got = {n: k for n, k in kernels.items() if all(p in n for p in parts)}
    assert got, parts
    return got.items()


def test_chunk_aggregates_hold_four_waves(kernels):
    """The gradient's chunk aggregates with 16 states: 128 registers or fewer (four waves
    per SIMD) and no scratch, in all eight forms."""
    got = _pick(kernels, "12k_chunk_aggrI", "Lb1ELb1ELi8E")  # WANT_M, N16, SEG
    assert len(got) == 8
    for name, k in got:
        assert k[".vgpr_count"] <= 128 and k[".private_segment_fixed_size"] == 0, name


def test_gemm_keeps_its_accumulators(kernels):
    """The 256 x 256 kernels hold 256 accumulators in the AGPRs and everything else in the
    VGPRs: nothing in scratch, in any epilogue form."""
    got = [*_pick(kernels, "9k_gemm_ntI"), *_pick(kernels, "7k_gemm4I")]
    assert len(got) >= 4
    for name, k in got:
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, name


def test_pairs_hold_two_waves(kernels):
    """The pair kernel's products and sums of 8 steps by 8 states: two waves per SIMD and
    nothing in scratch, in all four forms."""
    got = _pick(kernels, "7k_pairsI")
    assert len(got) == 4
    for name, k in got:
        assert k[".vgpr_count"] <= 256 and k[".private_segment_fixed_size"] == 0, name
