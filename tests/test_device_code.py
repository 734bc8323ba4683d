"""The built library's own device code (gfx950), disassembled: where kernels issue matrix products as inline assembly, the
compiler counts none of the wait states between a product and the instructions around it, so they are counted here."""
import os
import re
import struct
import subprocess

import pytest

from paper_2412_17246_amd import build as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
READ_AFTER_PRODUCT = 11     # wait states from a 4-pass product to the first other use of its result
PRODUCT_AFTER_WRITE = 2     # from a vector instruction's write to a product that reads it


def _code_objects(path):
    """The gfx950 code objects bundled in the library, one per source file."""
    data = open(path, "rb").read()
    for at in (m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data)):
        pos = at + 24
        (entries,) = struct.unpack_from("<Q", data, pos)
        pos += 8
        for _ in range(entries):
            offset, size, idlen = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if b"gfx950" in target:
                yield data[at + offset:at + offset + size]


def _kernels(tmp_path, name):
    """{symbol: [instruction text]} of the kernels whose symbol contains `name`, in address order."""
    found = {}
    for i, blob in enumerate(_code_objects(B.LIB)):
        if name.encode() not in blob:
            continue
        obj = tmp_path / ("code%d.o" % i)
        obj.write_bytes(blob)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(obj)], capture_output=True, text=True, check=True).stdout
        current = None
        for line in text.splitlines():
            label = re.match(r"[0-9a-f]+ <(.*)>:", line)
            if label:
                current = found.setdefault(label[1], []) if name in label[1] else None
            elif current is not None and line.strip():
                current.append(line.split("//")[0].strip())
    return found


def _registers(operand):
    """{('a' | 'v', number)} of one operand such as v12 or a[4:7]."""
    m = re.fullmatch(r"([av])(?:(\d+)|\[(\d+):(\d+)\])", operand.strip())
    if not m:
        return set()
    lo, hi = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
    return {(m[1], r) for r in range(lo, hi + 1)}


def _operands(instruction):
    return [_registers(o) for o in instruction.split(None, 1)[1].split(",")] if " " in instruction else []


def _states(instruction):
    return int(instruction.split()[1], 0) + 1 if instruction.startswith("s_nop") else 1


@pytest.mark.skipif(not os.path.exists(OBJDUMP) or not os.path.exists(B.LIB), reason="needs the built library and llvm-objdump")
def test_large_tile_products_are_settled_before_their_results_are_used(tmp_path):
    kernels = _kernels(tmp_path, "gemm_big_kernel")
    kernels = {k: v for k, v in kernels.items() if any(x.startswith("v_mfma") for x in v)}
    assert len(kernels) == 6                            # three epilogues, whole and split tiles
    for name, code in kernels.items():
        products = [i for i, x in enumerate(code) if x.startswith("v_mfma")]
        results = set().union(*(_operands(code[i])[0] for i in products))
        assert len(results) == 256, name
        # behind the loop: the wait comes before anything that touches an accumulator
        waited = 0
        for x in code[products[-1] + 1:]:
            if waited >= READ_AFTER_PRODUCT:
                break
            assert not results & set().union(set(), *_operands(x)), (name, x)
            waited += _states(x) if x.startswith("s_nop") else 0
        # inside it: no other instruction near a product touches its result, none before it has just written an operand
        for i in products:
            ops = _operands(code[i])
            states = 0
            for x in code[i + 1:]:
                if states >= READ_AFTER_PRODUCT:
                    break
                if not x.startswith("v_mfma"):
                    assert not ops[0] & set().union(set(), *_operands(x)), (name, code[i], x)
                states += _states(x)
            states = 0
            for x in reversed(code[:i]):
                if states >= PRODUCT_AFTER_WRITE:
                    break
                if x.startswith("v_") and not x.startswith("v_mfma"):
                    assert not _operands(x)[0] & set().union(*ops), (name, x, code[i])
                states += _states(x)
