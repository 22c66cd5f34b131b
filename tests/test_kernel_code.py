"""What the pipelined dK/dV kernel asks of register allocation, read from the AMD assembly of the built library (CPU only).

Its S and dP products are inline assembly, whose latency the compiler does not see: nothing but the order of the instructions keeps
an operand in place until an MFMA has read it and a result untouched until it is there."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2502_00340_amd import binding as Bn

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
KERNEL = re.compile(r"^[0-9a-f]+ <(\S*attn_dkv_kernel\S*)>:")
REACH = 120         # instructions that a walk goes on for


def _regs(operand):
    """VGPRs and AGPRs that an operand names."""
    return {(m[1], r) for m in re.finditer(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+))", operand)
            for r in range(int(m[2] or m[4]), int(m[3] or m[4]) + 1)}


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{name: [(offset, opcode, operands, branch target)]}"""
    if not os.path.exists(Bn.LIB_PATH):
        from paper_2502_00340_amd import build
        build.build_library(verbose=False)
    tmp = tmp_path_factory.mktemp("code")
    shutil.copy(Bn.LIB_PATH, tmp / "lib.so")                    # the code objects are written beside it
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp, check=True, capture_output=True)
    out = {}
    for f in sorted(tmp.glob("*gfx950")):
        code, base = None, 0
        for line in subprocess.run([OBJDUMP, "-d", f.name], cwd=tmp, check=True, capture_output=True, text=True).stdout.splitlines():
            if line and not line[0].isspace():
                m = KERNEL.match(line)
                code, base = (out.setdefault(m[1], []), int(line.split()[0], 16)) if m else (None, 0)
            elif code is not None and "//" in line:
                text, note = line.split("//", 1)
                op, _, rest = text.strip().partition(" ")
                m = re.search(r"\+0x([0-9a-f]+)>", note)
                code.append((int(note.split(":")[0], 16) - base, op, rest.split(","), int(m[1], 16) if m else None))
    assert len(out) == 4, sorted(out)                           # d = 64 and 128, with and without rotary tables
    return out


def _mfmas_before(code, at, start, hit):
    """Fewest MFMAs that start after instruction `start` and before the first one that `hit` says yes to, over all paths."""
    best, todo, seen = REACH, [(start + 1, 0, 0)], {}
    while todo:
        i, mfmas, steps = todo.pop()
        while i < len(code) and steps < REACH and mfmas < best and seen.get(i, REACH) > mfmas:
            seen[i] = mfmas
            _, op, ops, target = code[i]
            if op == "s_endpgm":
                break
            if hit(op, ops):
                best = mfmas
                break
            mfmas += op.startswith("v_mfma")
            steps += 1
            if target is not None and op != "s_branch":
                todo.append((at[target], mfmas, steps))
            i = at[target] if op == "s_branch" else i + 1
    return best


def test_registers_of_mfmas_that_the_compiler_does_not_wait_for(kernels):
    """MFMAs of a wave start one after the other, so an operand C has been read once the next one has started, and a result is there
    once the one after that has."""
    for name, code in kernels.items():
        at = {c[0]: i for i, c in enumerate(code)}
        found = 0
        for i, (off, op, ops, _) in enumerate(code):
            if not op.startswith("v_mfma") or not ops[0].strip().startswith("v"):
                continue                    # accumulators in AGPRs are the compiler's
            found += 1
            d, c = _regs(ops[0]), _regs(ops[3])

            def overwrites(op, ops):        # the first operand is the result, of all but MFMAs (behind this one anyway) and these
                return not op.startswith(("v_mfma", "buffer_", "global_store", "ds_write", "s_")) and bool(_regs(ops[0]) & c)

            def touches(op, ops):
                return bool(set().union(*map(_regs, ops[1:3] if op.startswith("v_mfma") else ops)) & d)
            assert c <= d or _mfmas_before(code, at, i, overwrites) >= 1, (name, hex(off), op, ops, "C overwritten")
            assert _mfmas_before(code, at, i, touches) >= 2, (name, hex(off), op, ops, "result touched")
        assert found >= 64, (name, found)


def test_loops_around_mfmas_are_uniform(kernels):
    """A loop that the compiler takes for a divergent one counts in vector registers, beside every MFMA, and masks lanes."""
    for name, code in kernels.items():
        at = {c[0]: i for i, c in enumerate(code)}
        first = next(i for i, c in enumerate(code) if c[1].startswith("v_mfma"))
        loops = [(at[target], i) for i, (_, _, _, target) in enumerate(code) if target is not None and at[target] < i]
        loops = [(a, b) for a, b in loops if first < a and sum(c[1].startswith("v_mfma") for c in code[a:b]) >= 32]
        assert len(loops) >= 2, name            # the steps of a head with and without the mask
        for a, b in loops:
            assert not code[b][1].startswith("s_cbranch_exec"), (name, hex(code[a][0]), hex(code[b][0]), code[b][1])
