"""Registers, scratch and code of the batch kernels in the built library, from the code objects' own metadata: what a
kernel of many tile bodies may cost over the kernels of its bodies alone."""
import os
import re
import struct
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2402_12274_amd", "libmdt.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
ALL, RELAY, COPY, CHUNK = 71, 16, 8, 4  # tile bodies, as in batch_kernel.h


def _code_objects(blob):
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob):
        at = m.start() + 24
        (n,) = struct.unpack_from("<Q", blob, at)
        at += 8
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", blob, at)
            triple = blob[at + 24:at + 24 + tlen]
            at += 24 + tlen
            if b"gfx950" in triple and size:
                yield blob[m.start() + off:m.start() + off + size]


@pytest.fixture(scope="module")
def kernels():
    """(policy, unpack, bodies) -> registers per lane, scratch bytes per lane, code bytes."""
    if not (os.path.exists(READELF) and os.path.exists(LIB)):
        pytest.skip("no built library or no readelf")
    out = {}
    with open(LIB, "rb") as f:
        blob = f.read()
    for obj in _code_objects(blob):
        with tempfile.NamedTemporaryFile() as f:
            f.write(obj)
            f.flush()
            notes = subprocess.check_output([READELF, "--notes", f.name], text=True)
            syms = subprocess.check_output([READELF, "-sW", f.name], text=True)
        size = {w[7]: int(w[2]) for w in (ln.split() for ln in syms.splitlines()) if len(w) >= 8 and w[3] == "FUNC"}
        for k in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.name:\s+(\S+)", k[k.index(".max_flat"):]).group(1)
            m = re.search(r"batch_kernelILi(\d)ELi(\d)ELi(\d+)E", name)
            if m:
                out[tuple(map(int, m.groups()))] = (int(re.search(r"\.vgpr_count:\s+(\d+)", k).group(1)),
                                                    int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", k).group(1)),
                                                    size[name])
    assert out
    return out


def _waves(registers):
    """Waves per SIMD: 512 registers per lane, handed out in eights, and at most eight waves."""
    return min(8, 512 // ((registers + 7) // 8 * 8))


@pytest.mark.parametrize("policy", [0, 1, 2])
def test_unpack_kernels_keep_their_waves(kernels, policy):
    # a tile's four packed loads per lane are all there is to overlap, so latency is hidden by waves: six for the chunk
    # body, five and more with every other body beside it
    assert _waves(kernels[policy, 1, CHUNK][0]) >= 6
    assert _waves(kernels[policy, 1, ALL][0]) >= 5
    assert kernels[policy, 1, CHUNK][1] == kernels[policy, 1, ALL][1] == 0


@pytest.mark.parametrize("policy", [0, 1, 2])
def test_pack_kernels_keep_their_waves(kernels, policy):
    assert _waves(kernels[policy, 0, CHUNK][0]) >= 6
    assert _waves(kernels[policy, 0, CHUNK | 32][0]) >= 6  # gathers through the caches
    assert _waves(kernels[policy, 0, ALL][0]) >= 5
    assert kernels[policy, 0, CHUNK][1] == kernels[policy, 0, ALL][1] == 0


@pytest.mark.parametrize("policy", [0, 1, 2])
def test_kernels_hold_each_body_once(kernels, policy):
    # relays add the unpack of every body to the packs, copies one gather and one scatter per kind: each at most about the
    # packs' size, and a third more for register spills
    packs = kernels[policy, 0, ALL][2]
    assert kernels[policy, 0, COPY][2] <= packs and kernels[policy, 0, COPY][1] == 0
    assert kernels[policy, 0, ALL | COPY][2] <= 3 * packs
    assert kernels[policy, 0, ALL | COPY | RELAY][2] <= 4 * packs
    assert _waves(kernels[policy, 0, ALL | COPY | RELAY][0]) >= 4
