"""Wait states that the CDNA4 instruction set asks of the program, in the compiled kernels.  The compiler inserts them between
instructions that it knows; inline assembly it does not look into, and which registers it puts beside such a piece of assembly
changes with every build, so the code as built is walked: every path of at most so many states behind the instruction that
writes a register.

  m0 written                        -> load to LDS                               1 state between
  scalar register written by vector -> vector memory instruction that reads it   5
  vector register written by vector -> matrix product that reads it              2
  result of a 16 x 16 x 32 product  -> anything but a product that accumulates   8 (4 passes; what the compiler keeps for its own)
                                       onto the same registers

And, from the same code objects: the pipelined attention kernels keep every vector register (a reload waits for all loads before it, the
tiles in flight too).

Needs the LLVM tools of ROCm and the built library, and no GPU."""
import os
import re
import subprocess

import pytest

from paper_2603_01281_amd import build

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
READELF = os.path.join(os.path.dirname(OBJDUMP), "llvm-readelf")
KINDS = {"v": 0, "a": 1 << 9, "s": 1 << 10}
NAMED = {"m0": {KINDS["s"] + 200}, "vcc": {KINDS["s"] + 106, KINDS["s"] + 107}, "vcc_lo": {KINDS["s"] + 106}, "vcc_hi": {KINDS["s"] + 107},
         "exec": {KINDS["s"] + 126, KINDS["s"] + 127}}
M0 = NAMED["m0"]
OPERAND = re.compile(r"\b([vas])(?:\[(\d+):(\d+)\]|(\d+))|\b(m0|vcc_lo|vcc_hi|vcc|exec)\b")
NO_RESULT = ("ds_write", "global_store", "scratch_store", "global_load_lds", "s_barrier", "s_waitcnt", "s_nop", "s_setprio", "s_cmp", "s_bitcmp",
             "s_cbranch", "s_branch", "s_endpgm", "ds_or_b32")
VECTOR_SCALARS = ("v_cmp", "v_readlane", "v_readfirstlane", "v_mad_u64_u32", "v_mad_i64_i32", "v_div_scale")


def registers(text):
    out = set()
    for kind, lo, hi, one, name in OPERAND.findall(text):
        if name:
            out |= NAMED[name]
        else:
            first = int(lo or one)
            out |= set(range(KINDS[kind] + first, KINDS[kind] + int(hi or one) + 1))
    return out


class Instruction:
    __slots__ = ("line", "op", "reads", "writes", "states", "target", "falls", "parts")

    def __init__(self, line, text):
        self.line = text
        op, _, rest = text.partition(" ")
        self.op = op
        parts = [p.strip() for p in re.split(r",(?![^\[]*\])", rest)] if rest.strip() else []
        self.parts = [registers(p) for p in parts]
        self.states = int(parts[0], 0) + 1 if op == "s_nop" else 1
        self.target, self.falls = None, op not in ("s_branch", "s_endpgm", "s_setpc_b64")
        results = 0 if op.startswith(NO_RESULT) else 1
        if op.startswith(("v_mad_u64_u32", "v_mad_i64_i32", "v_div_scale", "v_permlane16_swap", "v_permlane32_swap")) or "_co_u32" in op:
            results = 2                                   # a carry, or both operands
        self.writes = set().union(*self.parts[:results])
        self.reads = set().union(*self.parts[results:])
        if "swap" in op or op.startswith(("v_fmac", "v_dot2c", "v_writelane")):
            self.reads |= self.parts[0]
        if "saveexec" in op or op.startswith("v_cmpx"):
            self.writes |= NAMED["exec"]


def kernels(path):
    """(name, instructions) of every function of a code object."""
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", path], check=True, capture_output=True, text=True).stdout
    name, body, found = None, [], []
    for line in text.splitlines():
        m = re.match(r"^([0-9a-f]+) <(\S+)>:$", line)
        if m:
            if body:
                found.append((name, body))
            name, body = m.group(2), []
            start = int(m.group(1), 16)
            continue
        m = re.match(r"^\s+(\S.*?)\s*// ([0-9A-F]+):", line)
        if m and name:
            t = re.search(r"<[^>+]*(?:\+0x([0-9a-f]+))?>\s*$", line)
            body.append((int(m.group(2), 16) - start, m.group(1), int(t.group(1) or "0", 16) if t else None))
    if body:
        found.append((name, body))
    for name, body in found:
        at = {offset: i for i, (offset, _, _) in enumerate(body)}
        out = []
        for i, (offset, text, target) in enumerate(body):
            ins = Instruction(offset, text)
            if ins.op.startswith(("s_cbranch", "s_branch")):
                assert target in at, f"{name}: {text}"
                ins.target = at[target]
            out.append(ins)
        yield name, out


def walk(code, k, limit, visit):
    """Calls visit(instruction, states since k) on every path behind code[k]; a path ends at `limit` states or where visit says so."""
    least, todo = {}, [(k, 0)]
    while todo:
        i, passed = todo.pop()
        ins = code[i]
        after = [ins.target] if ins.target is not None else []
        if ins.falls and i + 1 < len(code):
            after.append(i + 1)
        for j in after:
            if passed >= limit or least.get(j, limit) <= passed:
                continue
            least[j] = passed
            if not visit(code[j], passed):
                todo.append((j, passed + code[j].states))


def vector_memory(op):
    return op.startswith(("global_", "buffer_", "scratch_", "flat_"))


def violations(code):
    found = []
    for k, ins in enumerate(code):
        def flag(kind, other, passed):
            found.append(f"{kind}: {ins.line}  ->  {other.line}  ({passed} states between)")

        if ins.writes & M0:
            def visit(other, passed):
                if "_lds_" in other.op or other.op.endswith("_lds"):
                    flag("m0", other, passed)
                return bool(other.writes & M0)
            walk(code, k, 1, visit)
        if ins.op.startswith(VECTOR_SCALARS) or "_co_u32" in ins.op:
            scalars = {r for r in ins.writes if r >= KINDS["s"]}
            if scalars:
                def visit(other, passed):
                    if vector_memory(other.op) and other.reads & scalars:
                        flag("scalar base", other, passed)
                    return other.op.startswith("s_") and scalars <= other.writes
                walk(code, k, 5, visit)
        if ins.op.startswith("v_mfma_f32_16x16x32_bf16"):
            d = ins.parts[0]

            def visit(other, passed):
                if other.op.startswith("v_mfma"):
                    if other.parts[3] == d and not (other.parts[1] | other.parts[2]) & d:
                        return True                       # the accumulator of the next one: the hardware waits
                    if (other.reads | other.writes) & d:
                        flag("result in a product", other, passed)
                elif (other.reads | other.writes) & d:
                    flag("result", other, passed)
                return False
            walk(code, k, 8, visit)
        elif ins.op.startswith("v_") and not ins.op.startswith("v_mfma"):
            vectors = {r for r in ins.writes if r < KINDS["s"]}
            if vectors:
                def visit(other, passed):
                    if other.op.startswith("v_mfma") and other.reads & vectors:
                        flag("operand", other, passed)
                    return False
                walk(code, k, 2, visit)
    return found


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(build.LIB):
        build.build()
    folder = tmp_path_factory.mktemp("code")
    os.symlink(build.LIB, folder / "libseka.so")
    subprocess.run([OBJDUMP, "--offloading", "libseka.so"], cwd=folder, check=True, capture_output=True)
    objects = sorted(str(p) for p in folder.iterdir() if p.name.endswith("gfx950"))
    assert objects
    return objects


def assemble(*lines):
    return [Instruction(i, l) for i, l in enumerate(lines)]


@pytest.mark.parametrize("lines,kind", [
    (("s_mov_b32 m0, s4", "global_load_lds_dwordx4 v1, s[2:3]"), "m0"),
    (("s_mov_b32 m0, s4", "s_nop 0", "global_load_lds_dwordx4 v1, s[2:3]"), None),
    (("v_readlane_b32 s3, v9, 5", "s_mov_b32 m0, s4", "s_nop 2", "global_load_lds_dwordx4 v1, s[2:3]"), "scalar base"),
    (("v_readlane_b32 s3, v9, 5", "s_mov_b32 m0, s4", "s_mov_b64 s[6:7], s[2:3]", "global_load_lds_dwordx4 v1, s[6:7]"), None),
    (("v_readlane_b32 s3, v9, 5", "s_nop 4", "global_load_dword v1, v2, s[2:3]"), None),
    (("v_mov_b32_e32 v5, v1", "s_nop 0", "v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3]"), "operand"),
    (("v_mov_b32_e32 v5, v1", "s_nop 1", "v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3]"), None),
    (("v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3]", "s_nop 6", "v_mul_f32_e32 v9, v3, v3"), "result"),
    (("v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3]", "s_nop 7", "v_mul_f32_e32 v9, v3, v3"), None),
    (("v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3]", "v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3]"), None),
    (("v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], 0", "v_mfma_f32_16x16x32_bf16 v[12:15], v[0:3], v[8:11], v[12:15]"), "result in a product")])
def test_the_walk_sees_what_it_looks_for(lines, kind):
    found = violations(assemble(*lines))
    assert [f.split(":")[0] for f in found] == ([kind] if kind else [])


def test_compiled_kernels_keep_them(code_objects):
    bad, seen = [], 0
    for path in code_objects:
        for name, code in kernels(path):
            seen += sum(i.op.startswith("v_mfma_f32_16x16x32_bf16") for i in code)
            found = violations(code)
            if found:
                bad.append(f"{name}: {len(found)}\n  " + "\n  ".join(found[:4]))
    assert seen > 1000, "the products of the attention kernels"
    assert not bad, "\n".join(bad)


def test_pipelined_kernels_spill_no_vector_registers(code_objects):
    spills = {}
    for path in code_objects:
        notes = subprocess.run([READELF, "--notes", path], check=True, capture_output=True, text=True).stdout
        kernel = ""
        for key, value in re.findall(r"\.(symbol|vgpr_spill_count):\s+(\S+)", notes):
            if key == "symbol":
                kernel = value
            elif "attention_bf16_pipe_kernel" in kernel:
                spills[kernel] = int(value)
    assert len(spills) == 32, sorted(spills)
    assert not any(spills.values()), {k: v for k, v in spills.items() if v}
