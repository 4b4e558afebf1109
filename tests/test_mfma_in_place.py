"""The kernels that issue matrix instructions as inline assembly, on accumulators that stay in their accumulation registers, as they
are compiled: the compiler inserts no wait states around an instruction it cannot see, so the code has to hold them.  Read from the
built library's own code objects, by control flow: an accumulator is touched by other instructions only behind the two `s_nop 15` that
outlast the longest of them, no vector instruction writes an operand within two wait states of its use, and nothing is spilled
(a spill would read an accumulator wherever the register allocator likes).  Nor do the float attention kernels spill, which hold the
operands of two products at once."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2505_24544_amd import build

LLVM = "/opt/rocm/llvm/bin/"
KERNELS = ("attn_bwd_dkv_bf16_kernel", "gemm_bf16_kernel", "gemm_bf16_ksplit_kernel")
COUNT = 2 + 12 + 12                              # instantiations
FLOAT_KERNELS = ("attn_fwd_f32_kernel", "attn_bwd_f32_kernel")      # four widths, whole and ragged, each
pytestmark = pytest.mark.skipif(not os.path.exists(LLVM + "llvm-objdump"), reason="no llvm-objdump")


def _out(*cmd, cwd=None):
    return subprocess.run(cmd, cwd=cwd, check=True, capture_output=True, text=True).stdout


def _regs(text):
    """Vector and accumulation registers that an operand names, as a bit set (accumulation registers from bit 512 on)."""
    bits = 0
    for kind, one, first, last in re.findall(r"\b([av])(?:(\d+)\b|\[(\d+):(\d+)\])", text):
        first, last = int(one or first), int(one or last)
        bits |= ((1 << (last - first + 1)) - 1) << (first + (512 if kind == "a" else 0))
    return bits


ACC = ((1 << 512) - 1) << 512


class Ins:
    def __init__(self, addr, text):
        self.addr, self.text = addr, text
        self.op, _, rest = text.partition(" ")
        ops = [_regs(o) for o in rest.split(",")]
        self.mfma = self.op.startswith("v_mfma")
        self.dst = ops[0]
        self.read = ops[1] | ops[2] if self.mfma else 0          # the two operands
        self.any = 0
        for o in ops:
            self.any |= o
        self.states = int(rest, 0) + 1 if self.op == "s_nop" else 1
        self.next = []


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    """({name: instructions with their successors} of KERNELS, {name: spilled registers} of every kernel)."""
    if not os.path.exists(build.OUT):
        build.build(verbose=False)
    tmp = str(tmp_path_factory.mktemp("co"))
    shutil.copy(build.OUT, os.path.join(tmp, "lib.so"))
    _out(LLVM + "llvm-objdump", "--offloading", "lib.so", cwd=tmp)
    found, spilled = {}, {}
    for f in sorted(os.listdir(tmp)):
        if not f.endswith("gfx950"):
            continue
        notes = _out(LLVM + "llvm-readelf", "--notes", f, cwd=tmp)
        here = dict(re.findall(r"\.name:\s+(_Z\S+)\n(?:(?!\.name).*\n)*?\s+\.vgpr_spill_count: (\d+)", notes))
        spilled.update((n, int(s)) for n, s in here.items())
        if not any(k in n for n in here for k in KERNELS):
            continue
        name, code = None, []
        for line in _out(LLVM + "llvm-objdump", "-d", "--mcpu=gfx950", f, cwd=tmp).splitlines():
            m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if m:
                name = m[1] if any(k in m[1] for k in KERNELS) and m[1] in here else None
                if name:
                    found[name] = code = []
            elif name and (m := re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+): [0-9A-F ]+?(?: <.*\+0x([0-9a-f]+)>)?\s*$", line)):
                code.append(Ins(int(m[2], 16), m[1]))
                code[-1].to = int(m[3], 16) if m[3] else None
    for code in found.values():
        at = {i.addr - code[0].addr: n for n, i in enumerate(code)}
        for n, i in enumerate(code):
            if i.op.startswith(("s_cbranch", "s_branch")):
                i.next.append(at[i.to])
            if n + 1 < len(code) and i.op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
                i.next.append(n + 1)
    return found, spilled


@pytest.fixture(scope="module")
def kernels(library):
    return library[0]


def test_every_kernel_is_there(kernels):
    assert len(kernels) == COUNT, sorted(kernels)
    for name, code in kernels.items():
        assert any(i.mfma and i.dst & ACC for i in code), name


def test_accumulators_are_read_behind_the_wait(kernels):
    wrong = []
    for name, code in kernels.items():
        undrained = [None] * len(code)           # accumulators that may be in flight ahead of an instruction
        undrained[0], todo = 0, [0]
        while todo:
            n = todo.pop()
            i, state = code[n], undrained[n]
            if i.mfma:
                state |= i.dst & ACC
            elif i.op == "s_nop" and i.states == 16 and n and code[n - 1].op == "s_nop" and code[n - 1].states == 16:
                state = 0
            for m in i.next:
                if undrained[m] is None or state & ~undrained[m]:
                    undrained[m] = state | (undrained[m] or 0)
                    todo.append(m)
        for i, state in zip(code, undrained):
            if state and state & (i.read if i.mfma else i.any):
                wrong.append((name, hex(i.addr), i.text))
    assert not wrong, (len(wrong), wrong[:5])


def test_operands_are_written_in_time(kernels):
    wrong = []
    for name, code in kernels.items():
        for n, i in enumerate(code):
            if not i.op.startswith("v_") or i.mfma or not i.dst:
                continue
            todo = [(m, 0) for m in i.next]
            while todo:
                m, states = todo.pop()
                j = code[m]
                if states >= 2:
                    continue
                if j.mfma and j.dst & ACC and i.dst & (j.read | j.dst):
                    wrong.append((name, hex(i.addr), i.text, j.text))
                todo += [(k, states + j.states) for k in j.next]
    assert not wrong, (len(wrong), wrong[:5])


def test_nothing_is_spilled(library):
    spilled = {n: s for n, s in library[1].items() if any(k in n for k in KERNELS + FLOAT_KERNELS)}
    assert len(spilled) == COUNT + 16
    assert {n: s for n, s in spilled.items() if s} == {}
