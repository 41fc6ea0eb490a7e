"""The compiled device code of the library, on the CPU: registers and the masks of lanes.

Held below the registers it needs (a launch bound of more waves per SIMD), a kernel here came out wrong: the
compiler's register allocator split live ranges and put copies of loop-invariant coefficients at the head of a block
in front of the instruction that gives the block its lanes back,

    s_cbranch_execz L                      ; over the "then" side of an if
    ...
    L: v_mov_b64_e32 v[28:29], v[164:165]  ; with the lanes of the "then" side, or none
       s_andn2_saveexec_b64 s[92:93], ...  ; only now the lanes of the "else" side

so that lanes of the other side went on with whatever v[28:29] held (the FP64 smoothing step of degree 5 on
Gauss-Legendre nodes at three waves per SIMD: wrong V-cycles that varied from run to run).  The tests read the built
library's own code objects: no such block in any kernel, and no spilled vector registers in the operator kernels.
"""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2510_21213_amd", "libdgpoisson.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")


def code_objects(path):
    """The AMDGPU ELF images inside a shared library (offset, length, bytes of the whole file)."""
    data = open(path, "rb").read()
    at = data.find(b"\x7fELF\x02\x01", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            shoff, = struct.unpack_from("<Q", data, at + 40)
            size, num = struct.unpack_from("<HH", data, at + 58)
            yield data, at, shoff + size * num
        at = data.find(b"\x7fELF\x02\x01", at + 4)


def kernel_metadata(path):
    msgpack = pytest.importorskip("msgpack")
    for data, at, _ in code_objects(path):
        shoff, = struct.unpack_from("<Q", data, at + 40)
        size, num = struct.unpack_from("<HH", data, at + 58)
        for k in range(num):
            head = at + shoff + k * size
            if struct.unpack_from("<I", data, head + 4)[0] != SHT_NOTE:
                continue
            off, length = struct.unpack_from("<QQ", data, head + 24)
            p, end = at + off, at + off + length
            while p < end:
                nlen, dlen, kind = struct.unpack_from("<III", data, p)
                desc = p + 12 + (nlen + 3) // 4 * 4
                if kind == NT_AMDGPU_METADATA:
                    yield from msgpack.unpackb(data[desc:desc + dlen], raw=False)["amdhsa.kernels"]
                p = desc + (dlen + 3) // 4 * 4


LINE = re.compile(r"^\t(\S+)(.*?)\s*// ([0-9A-F]+): ([0-9A-F]{8})")
RESTORE = re.compile(r"s_(or_saveexec|andn2_saveexec|orn2_saveexec)_b64|s_(or|xor)_b64 exec, exec")
BLOCK_END = re.compile(r"s_(cbranch|branch|endpgm|setpc|barrier|and_saveexec|mov_b64 exec)")


def early_copies(lines):
    """Vector instructions between the target of an s_cbranch_execz, or a loop's end (s_cbranch_execnz
    backwards), and the
    instruction that restores the lanes there: (function, address, instruction)."""
    code, func, found = [], "", []

    def check():
        targets = {a + 4 + 4 * (w & 0xffff if not w & 0x8000 else (w & 0xffff) - 0x10000)
                   for a, w, t in code if t.startswith("s_cbranch_execz")}
        targets |= {a + 4 for a, w, t in code if t.startswith("s_cbranch_execnz") and w & 0x8000}
        pending = None
        for a, _, t in code:
            if a in targets:
                pending = []
            if pending is None:
                continue
            if RESTORE.match(t):
                found.extend((func, x, y) for x, y in pending)
                pending = None
            elif BLOCK_END.match(t):
                pending = None
            elif re.match(r"(v_(?!readlane|writelane|readfirstlane|nop)|scratch_load|ds_read|buffer_load|global_load)", t):
                pending.append((a, t))

    for line in lines:
        m = LINE.match(line)
        if m:
            code.append((int(m.group(3), 16), int(m.group(4), 16), (m.group(1) + m.group(2)).strip()))
        elif line.endswith(">:\n") and "<" in line:
            check()
            code, func = [], line[line.index("<") + 1:-3]
    check()
    return found


def disassembly(image, tmp_path):
    path = tmp_path / "object"
    path.write_bytes(image)
    p = subprocess.Popen([OBJDUMP, "-d", "--mcpu=gfx950", str(path)], stdout=subprocess.PIPE, text=True)
    yield from p.stdout
    assert p.wait() == 0


def test_the_pattern_is_found():
    """The block of the docstring, the same one compiled soundly, and a nested if whose inner join is a plain branch's
    target."""
    def text(*ins):
        return ["0000000000001000 <k>:\n"] + ["\t%s  // %012X: %s\n" % (t, 0x1000 + 4 * i, w)
                                              for i, (t, w) in enumerate(ins)]
    bad = text(("s_cbranch_execz 1", "BF880001"), ("v_add_f64 v[0:1], v[0:1], v[2:3]", "00000000"),
               ("v_mov_b64_e32 v[28:29], v[164:165]", "00000000"),
               ("s_andn2_saveexec_b64 s[92:93], s[92:93]", "00000000"), ("s_endpgm", "BF810000"))
    good = text(("s_cbranch_execz 1", "BF880001"), ("v_add_f64 v[0:1], v[0:1], v[2:3]", "00000000"),
                ("s_andn2_saveexec_b64 s[92:93], s[92:93]", "00000000"),
                ("v_mov_b64_e32 v[28:29], v[164:165]", "00000000"), ("s_endpgm", "BF810000"))
    inner = text(("s_cbranch_vccnz 1", "BF870001"), ("v_add_f64 v[0:1], v[0:1], v[2:3]", "00000000"),
                 ("v_mov_b64_e32 v[28:29], v[164:165]", "00000000"), ("s_or_b64 exec, exec, s[4:5]", "00000000"))
    assert [x[2] for x in early_copies(bad)] == ["v_mov_b64_e32 v[28:29], v[164:165]"]
    assert early_copies(good) == [] and early_copies(inner) == []


@pytest.mark.slow
def test_no_vector_instruction_before_a_block_has_its_lanes(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    objects = 0
    for data, at, length in code_objects(LIB):
        assert early_copies(disassembly(data[at:at + length], tmp_path)) == []
        objects += 1
    assert objects >= 5


def test_operator_kernels_spill_no_vector_registers():
    kernels = list(kernel_metadata(LIB))
    checked = [k for k in kernels if re.search(r"k_(slab|oct_op|quad|project|conv|brick|prolong|restrict|update|dot)", k[".name"])]
    assert len(checked) > 300
    bad = {k[".name"]: k[".vgpr_spill_count"] for k in checked if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]}
    assert not bad
