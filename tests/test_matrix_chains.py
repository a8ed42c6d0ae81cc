"""Distance between matrix products of two shapes that accumulate on each
other, in the built library's machine code (CPU).

The hardware does not forward a 16 x 16 x 32 product's result to a 16 x 16 x
16 one (or the other way round), and the compiler inserts no wait between
them.  Each such pair therefore has three other products between, or a wait of
at least twelve states (s_nop) of its own; whatever else happens to stand there
does not count."""
import os
import re
import struct
import subprocess

import pytest

from paper_2403_18466_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 code objects of the library's offload bundles."""
    data = open(path, "rb").read()
    start = data.find(MAGIC)
    while start >= 0:
        n, = struct.unpack_from("<Q", data, start + len(MAGIC))
        at = start + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + idlen]
            at += 24 + idlen
            if b"gfx950" in name and size:
                yield data[start + off:start + off + size]
        start = data.find(MAGIC, start + 1)


def registers(operand):
    m = re.match(r"([va])\[(\d+):(\d+)\]$", operand)
    if m:
        return [(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)]
    m = re.match(r"([va])(\d+)$", operand)
    return [(m[1], int(m[2]))] if m else []


def crossings(lines):
    """(kernel, first shape, second shape, products between, longest s_nop
    between) of every product that accumulates on one of another shape."""
    kernel, last, products, nops = "", {}, 0, []
    for line in lines:
        m = re.match(r"(?:[0-9a-f]+ )?<(_Z\w+)>:", line)
        if m:
            kernel, last, products, nops = m[1], {}, 0, []
            continue
        words = line.split("//")[0].split(None, 1)
        if not words:
            continue
        op = words[0]
        args = [a.strip() for a in words[1].split(",")] if len(words) > 1 else []
        if op.startswith("v_mfma"):
            for r in registers(args[3].split()[0]):
                if r in last and last[r][0] != op:
                    shape, at = last[r]
                    waits = [n for p, n in nops if p > at]
                    yield kernel, shape, op, products - at - 1, max(waits, default=0)
                    break
            for r in registers(args[0]):
                last[r] = op, products
            products += 1
        elif op == "s_nop":
            nops.append((products, int(args[0], 0) + 1))
        elif args and re.match(r"(v_|ds_read|buffer_load|global_load)", op):
            for r in registers(args[0]):
                last.pop(r, None)


def test_products_of_two_shapes_keep_their_distance(tmp_path):
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(build.hipcc())))
    objdump = os.path.join(rocm, "llvm", "bin", "llvm-objdump")
    if not os.path.exists(objdump):
        pytest.skip("llvm-objdump not found")
    if not os.path.exists(build.LIB):
        build.build()
    seen, close = set(), []
    for i, code in enumerate(code_objects(build.LIB)):
        path = tmp_path / f"{i}.co"
        path.write_bytes(code)
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", "--no-leading-addr", str(path)],
                              check=True, capture_output=True, text=True).stdout
        for c in crossings(text.splitlines()):
            seen.add(c[0])
            if c[3] < 3 and c[4] < 12:
                close.append(c)
    # (the 16-bit instances of the wide network's two step kernels have them)
    assert sum("wide_step_kernel" in k for k in seen) == 4
    assert sum("wide_step16_kernel" in k for k in seen) == 4
    assert not close, close
