"""The wait states of the matrix instructions in the library as built.

The four-wavefront GEMM loops issue theirs through inline assembly, and the compiler puts no wait
states around those: the source has to, and where registers are assigned or moved differently by
another compiler the distances can change.  So the machine code is read back (no GPU needed): along
every path, between an instruction that writes a register and one that needs the result, lie the
wait states that the CDNA ISA documents ask for (`s_nop n` counts n + 1, any other instruction 1).
"""
import collections
import functools
import re
import shutil
import subprocess

import pytest

import paper_2210_17223_amd as moe
from paper_2210_17223_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

# passes (of four cycles) of the matrix instructions in use, and whether they are of the reduced-
# precision kind, whose results take longer to be visible
MATRIX = {"16x16x32": (4, True), "32x32x16": (8, True), "16x16x4": (8, False)}
VALU_TO_MATRIX, VALU_SGPR_TO_MEMORY = 2, 5


def visible_after(mnemonic):
    """Wait states until a matrix instruction's result can be read or overwritten by others."""
    for shape, (passes, reduced) in MATRIX.items():
        if "_" + shape + "_" in mnemonic or mnemonic.endswith("_" + shape):
            return passes + 4 if reduced else passes + 2
    raise AssertionError("matrix instruction without an entry: " + mnemonic)


Inst = collections.namedtuple("Inst", "name reads writes states preds text")
_REG = re.compile(r"(?<![\w.])([vas])(?:(\d+)|\[(\d+):(\d+)\])(?![\w.])")


@functools.lru_cache(maxsize=None)
def registers(operand):
    out = set()
    for kind, one, lo, hi in _REG.findall(operand):
        lo, hi = (int(one), int(one)) if one else (int(lo), int(hi))
        out.update((kind, r) for r in range(lo, hi + 1))
    return frozenset(out)


def functions(asm):
    """{symbol: [Inst]} of the kernels with matrix instructions in a disassembly with addresses."""
    out, name = {}, None
    for line in asm.splitlines():
        head = re.match(r"([0-9a-f]+) <(\S+)>:$", line)
        if head:
            name, base = head[2], int(head[1], 16)
            out[name] = (base, [])
        elif name and line.startswith("\t") and "//" in line:
            out[name][1].append(line)
    return {n: parse(base, lines) for n, (base, lines) in out.items() if any("v_mfma" in l for l in lines)}


def parse(base, lines):
    insts, at, jumps = [], {}, []
    falls = True
    for i, line in enumerate(lines):
        code, _, note = line.strip().partition("//")
        name, _, args = code.strip().partition(" ")
        ops = [o.strip() for o in re.split(r",(?![^\[]*\])", args)] if args else []
        at[int(note.split(":")[0], 16)] = i
        dest = 0 if name.startswith(("ds_write", "ds_bpermute", "buffer_store", "global_store", "flat_store",
                                     "global_atomic", "s_cbranch", "s_branch", "s_cmp", "s_waitcnt", "s_nop")) else 1
        if name.startswith("buffer_load") and " lds" in " " + args:
            dest = 0
        if name.startswith("v_swap"):
            dest = 2
        if "_co_" in name or name.startswith("v_div_scale"):
            dest = 2
        writes = set().union(*map(registers, ops[:dest])) if dest else set()
        reads = set().union(*map(registers, ops[dest:])) if ops[dest:] else set()
        if dest == 2 and name.startswith("v_swap"):
            reads = writes
        if name.startswith(("v_fmac", "v_pk_fmac", "v_dot2c")):
            reads = reads | writes
        states = int(ops[0], 0) + 1 if name == "s_nop" else 1
        insts.append(Inst(name, reads, writes, states, [i - 1] if falls and i else [], code.strip()))
        if name.startswith(("s_branch", "s_cbranch")):
            jumps.append((i, int(re.search(r"\+0x([0-9a-f]+)>", note)[1], 16) + base if "+0x" in note else base))
        falls = name not in ("s_branch", "s_endpgm", "s_setpc_b64")
    for i, target in jumps:
        insts[at[target]].preds.append(i)
    return insts


def is_matrix(inst):
    return inst.name.startswith("v_mfma")


def needed(writer, reader):
    """Wait states between two instructions of which the second touches what the first writes."""
    raw = writer.writes & reader.reads
    if is_matrix(writer):
        if is_matrix(reader):
            d, a, b, c = (registers(o.strip()) for o in reader.text.split(" ", 1)[1].split(",", 3))
            if writer.writes & (a | b):
                return visible_after(writer.name)
            if writer.writes & c and writer.writes != c:
                return visible_after(writer.name) - 2
            return 0
        return visible_after(writer.name) if raw or writer.writes & reader.writes else 0
    if writer.name.startswith("v_"):
        if is_matrix(reader) and raw:
            return VALU_TO_MATRIX
        if reader.name.startswith(("buffer_", "global_", "flat_")) and any(k == "s" for k, _ in raw):
            return VALU_SGPR_TO_MEMORY
    return 0


LONGEST = 12


def hazards(insts):
    """[(writer, reader)] that are too close on some path."""
    found = []
    for i, reader in enumerate(insts):
        if reader.name.startswith("s_"):
            continue
        memory = reader.name.startswith(("buffer_", "global_", "flat_"))
        stack, seen = [(p, 0) for p in reader.preds], {}
        while stack:
            j, states = stack.pop()
            if states >= LONGEST or seen.get(j, LONGEST) <= states:
                continue
            seen[j] = states
            writer = insts[j]
            if (is_matrix(writer) or is_matrix(reader) or memory) and writer.name.startswith("v_") \
                    and needed(writer, reader) > states:
                found.append((writer.text, reader.text))
            stack.extend((p, states + writer.states) for p in writer.preds)
    return found


def listing(*code):
    return parse(0x1000, [f"\t{c.split('@')[0]} // {0x1000 + 4 * i:012X}: 00000000" +
                          (f" <f+{c.split('@')[1]}>" if "@" in c else "") for i, c in enumerate(code)])


MFMA = "v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[4:7], a[0:3]"


@pytest.mark.parametrize("code,bad", [
    (["v_mov_b32_e32 v4, v9", MFMA], 1),
    (["v_accvgpr_write_b32 a1, v9", "s_nop 0", MFMA], 1),
    (["v_accvgpr_write_b32 a1, v9", "s_nop 1", MFMA], 0),
    (["v_mov_b32_e32 v12, v9", MFMA], 0),
    ([MFMA, "v_accvgpr_read_b32 v0, a3"], 1),
    ([MFMA, "s_nop 7", "v_accvgpr_read_b32 v0, a3"], 0),
    ([MFMA, "s_nop 6", "v_accvgpr_write_b32 a2, v0"], 1),
    ([MFMA, MFMA, MFMA], 0),
    ([MFMA, "v_mfma_f32_16x16x32_bf16 a[2:5], v[8:11], v[4:7], a[2:5]"], 1),
    ([MFMA, "ds_write_b128 v0, a[0:3]"], 1),
    (["v_readfirstlane_b32 s4, v0", "s_nop 3", "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"], 1),
    (["v_readfirstlane_b32 s4, v0", "s_nop 4", "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"], 0),
    ([MFMA, "v_mov_b32_e32 v4, v9", "s_cbranch_scc1 65533 @0x0", "s_endpgm"], 1),       # round the loop
    ([MFMA, "v_mov_b32_e32 v4, v9", "s_nop 0", "s_cbranch_scc1 65532 @0x0", "s_endpgm"], 0),
])
def test_the_check_sees_planted_hazards(code, bad):
    assert len(hazards(listing(*code))) == bad


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    moe.lib()                                       # (built if it is not there)
    if shutil.which(OBJDUMP) is None:
        pytest.skip("no llvm-objdump")
    where = tmp_path_factory.mktemp("code")
    shutil.copy(moe.lib_path(), where / "libmoe.so")
    subprocess.run([OBJDUMP, "--offloading", "libmoe.so"], cwd=where, check=True, capture_output=True)
    out = {}
    for f in sorted(where.glob("*gfx950")):
        asm = subprocess.run([OBJDUMP, "-d", str(f)], check=True, capture_output=True, text=True).stdout
        out.update(functions(asm))
    return out


def test_no_matrix_instruction_of_the_library_is_too_close(library):
    assert sum("w4_kernel" in n for n in library) >= 20 and len(library) >= 100
    bad = {n: h for n, f in library.items() if (h := hazards(f))}
    assert not bad, "\n".join(f"{n}: {len(h)}, e.g. {h[0][0]} -> {h[0][1]}" for n, h in bad.items())


LOADS = """
#include <hip/hip_runtime.h>
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
namespace {
#include "gemm_w4.h"
}
__global__ void loads(const char *p, int n, uint32_t at)
{
    __shared__ char lds[4096];
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), 0, n, 0x00020000);
    auto *dst = (__attribute__((address_space(3))) void *)lds;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst, 4, threadIdx.x * 4, 0, 0, 0);
    load_to_lds(rs, threadIdx.x * 16, at, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst, 4, threadIdx.x * 4, 0, 256, 0);
}
"""


def test_a_load_to_lds_tells_the_compiler_that_m0_changes(tmp_path):
    """The compiler's own loads to LDS keep their destination in M0 from one to the next: between
    them `load_to_lds` takes M0 for its own, so the second has to set it again."""
    (tmp_path / "loads.hip").write_text(LOADS)
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-Wall")]
    subprocess.run([build.HIPCC, *flags, "-w", "--cuda-device-only", "-S", "loads.hip", "-o", "loads.asm"],
                   cwd=tmp_path, check=True, capture_output=True)
    code = [l.split(";")[0].strip() for l in (tmp_path / "loads.asm").read_text().splitlines()]
    loads = [i for i, l in enumerate(code) if l.startswith("buffer_load") and l.endswith(" lds")]
    assert len(loads) == 3
    for before, load in zip([0] + loads, loads):
        assert any(re.match(r"s_\w+ m0,", l) for l in code[before:load]), code[before:load + 1]
