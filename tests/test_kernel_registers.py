"""Registers of the built kernels against the lines between numbers of waves per SIMD that their launch rules count on."""
import re
import struct

import pytest

from paper_2602_04361_amd import sparvar as sv

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The gfx950 code objects of a library: one bundle per source, each with a table of (offset, size, target)."""
    at = data.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, pos - 8)[0]):
            offset, size, n = struct.unpack_from("<QQQ", data, pos)
            if b"gfx950" in data[pos + 24:pos + 24 + n]:
                yield data[at + offset:at + offset + size]
            pos += 24 + n
        at = data.find(MAGIC, pos)


def registers(elf):
    """Mangled kernel name -> VGPRs a wave is given (kernel descriptor, first resource word, units of 8)."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    entsize, num = struct.unpack_from("<HH", elf, 58)
    heads = [struct.unpack_from("<IIQQQQIIQQ", elf, shoff + i * entsize) for i in range(num)]
    out = {}
    for _, kind, _, _, offset, size, link, _, _, ent in heads:
        if kind != 11:  # dynamic symbols
            continue
        for i in range(0, size, ent):
            name, _, _, _, value, _ = struct.unpack_from("<IBBHQQ", elf, offset + i)
            start = heads[link][4] + name
            text = elf[start:elf.index(b"\0", start)].decode()
            if not text.endswith(".kd"):
                continue
            _, _, _, addr, base, _, _, _, _, _ = next(h for h in heads if h[1] == 1 and h[3] <= value < h[3] + h[5])
            out[text[:-3]] = ((struct.unpack_from("<I", elf, base + value - addr + 48)[0] & 63) + 1) * 8
    return out


@pytest.fixture(scope="module")
def vgprs():
    with open(sv.LIB_PATH, "rb") as f:
        data = f.read()
    found = {}
    for elf in code_objects(data):
        found.update(registers(elf))
    assert len(found) > 100
    return found


# 512 registers a SIMD lane: 128 give four waves, 168 three. Between the two: held to three waves and no more
@pytest.mark.parametrize("kernel,least,most", [
    (r"pooled_scores_kernelILi128ELi1ELi4E", 0, 128), (r"pooled_scores_kernelILi128ELi4ELi1E", 0, 128),
    (r"pooled_scores_kernelILi128ELi2ELi4E", 0, 128), (r"attn_bf16_kernelILi64ELi2ELi32ELi2E\w*9SparseSrc\w*Li1EE", 129, 168),
    (r"attn_bf16_kernelILi64ELi2ELi32ELi2E\w*8DenseSrc\w*Li1EE", 0, 128), (r"attn_bf16_kernelILi128ELi4ELi32ELi2E\w*8DenseSrc\w*Li1EE", 0, 168),
    (r"attn_bf16_kernelILi128ELi4ELi32ELi2E\w*8TokenSrc\w*Li1EE", 0, 168), (r"attn_bf16_kernelILi128ELi4ELi32ELi2E\w*11BlockRowSrc\w*Li1EE", 0, 168)])
def test_waves_per_simd(vgprs, kernel, least, most):
    got = {n: v for n, v in vgprs.items() if re.search(kernel, n)}
    assert len(got) == 1, sorted(got)
    assert least <= next(iter(got.values())) <= most, got
