"""Wait states that gfx950 leaves to the program, looked for in assembly made by the compiler.

A few results of vector instructions may not be read by the next instructions: the compiler puts other instructions or
s_nop between the two, but it does not look into inline assembly.  violations() reads the text of a build and reports every
pair that stands too close and of which one instruction at least is inline assembly."""
import re
from typing import NamedTuple

# wait states between the instruction that writes and the one that reads
SCALAR_TO_VECTOR = 2        # a scalar register (or vcc) written by a vector instruction, read by a vector instruction
SCALAR_TO_MEMORY = 5        # the same, read as an address by a memory instruction
SCALAR_TO_LANE = 4          # the same, read as the lane of v_readlane / v_writelane
VECTOR_TO_DPP = 2           # a vector register, read across lanes (DPP)
VECTOR_TO_LANE = 1          # a vector register, read by v_readlane / v_readfirstlane
TRANSCENDENTAL = 1          # a vector register written by v_rcp and the like, read by another kind of vector instruction
EXEC_TO_DPP = 5             # the execution mask written by a vector comparison, then DPP
EXEC_TO_LANE = 4            # the same, then v_readlane / v_readfirstlane / v_writelane
WINDOW = 5

_TWO_RESULTS = ("v_add_co_", "v_addc_co_", "v_sub_co_", "v_subb_co_", "v_subrev_co_", "v_subbrev_co_", "v_div_scale_",
                "v_mad_u64_u32", "v_mad_i64_i32")
_TRANSCENDENTAL = ("v_rcp_", "v_rsq_", "v_sqrt_", "v_log_", "v_exp_", "v_sin_", "v_cos_")
_LANE = ("v_readlane_", "v_readfirstlane_", "v_writelane_")
_REGISTER = re.compile(r"\b([vsa])(?:(\d+)\b|\[(\d+):(\d+)\])|\b(vcc|exec)(?:_lo|_hi)?\b")


class Instruction(NamedTuple):
    line: int
    text: str
    name: str
    operands: list
    inline: bool


def _registers(operand):
    out = set()
    for kind, one, first, last, special in _REGISTER.findall(operand):
        if special:
            out.add(special)
        elif one:
            out.add(f"{kind}{one}")
        else:
            out.update(f"{kind}{n}" for n in range(int(first), int(last) + 1))
    return out


def _is_dpp(i):
    return "_dpp" in i.name or any(w in i.text for w in ("quad_perm", "row_shl", "row_shr", "row_ror", "row_bcast", "wave_", "row_mirror"))


def _written(i):
    """registers that a vector or scalar instruction writes"""
    if not i.operands or i.name.startswith(("v_nop", "s_nop", "s_cmp", "s_bitcmp", "s_branch", "s_cbranch", "s_waitcnt", "s_set")):
        return set()
    if not i.name.startswith(("v_", "s_")):
        return set()
    out = _registers(i.operands[0])
    if i.name.startswith(_TWO_RESULTS):
        out |= _registers(i.operands[1])
    if i.name.startswith("v_cmpx"):
        out.add("exec")
    return out


def _read(i):
    skip = 2 if i.name.startswith(_TWO_RESULTS) else 1
    if i.name.startswith(("global_store", "flat_store", "buffer_store", "scratch_store")):
        skip = 0
    out = set()
    for o in i.operands[skip:]:
        out |= _registers(o)
    if i.name.startswith("v_div_fmas"):
        out.add("vcc")
    return out


def _is_scalar(register):
    return register == "vcc" or register[0] == "s"


def needed(writer, reader, overwritten=frozenset()):
    """wait states that must lie between the two instructions, 0 if none; overwritten: registers that others between the
    two have written"""
    if not writer.name.startswith("v_"):
        return 0
    written, need = _written(writer) - overwritten, 0
    if reader.name.startswith("v_"):
        read = _read(reader)
        if reader.name.startswith(("v_readlane_", "v_writelane_")) and written & _registers(reader.operands[2]):
            need = max(need, SCALAR_TO_LANE)
        if any(_is_scalar(r) for r in written & read):
            need = max(need, SCALAR_TO_VECTOR)
        vectors = {r for r in written & read if r[0] == "v" and r != "vcc"}
        if vectors and _is_dpp(reader):
            need = max(need, VECTOR_TO_DPP)
        if vectors and reader.name.startswith(_LANE[:2]):
            need = max(need, VECTOR_TO_LANE)
        if vectors and writer.name.startswith(_TRANSCENDENTAL) and not reader.name.startswith(_TRANSCENDENTAL):
            need = max(need, TRANSCENDENTAL)
        if "exec" in written:
            need = max(need, EXEC_TO_DPP if _is_dpp(reader) else (EXEC_TO_LANE if reader.name.startswith(_LANE) else 0))
    elif reader.name.startswith(("global_", "flat_", "buffer_", "scratch_")):
        if any(_is_scalar(r) for r in written & _read(reader)):
            need = SCALAR_TO_MEMORY
    return need


def instructions(assembly):
    """The instructions of a text in order, None where a function starts.  (Labels and branches are passed over: what stands
    in front of a reader is taken to run in front of it.)"""
    inline = False
    for number, line in enumerate(assembly.splitlines(), 1):
        if "#ASMSTART" in line or "#ASMEND" in line:
            inline = "#ASMSTART" in line
            continue
        text = line.split(";")[0].split("//")[0].strip()
        if text.startswith((".globl", ".section")):
            yield None
        if not re.match(r"[a-z]+_[a-z0-9_]+(\s|$)", text):
            continue
        name, _, rest = re.sub(r"\s+", " ", text).partition(" ")
        operands = [o.strip() for o in rest.split(",")] if rest else []
        yield Instruction(number, text, name, operands, inline)


def violations(assembly, compiler_made=False):
    """(states needed, states found, writer, reader) of every pair that stands too close; with compiler_made also pairs in
    which the compiler has seen both."""
    found, recent = [], []          # recent: (instruction, wait states it counts)
    for i in instructions(assembly):
        if i is None:
            recent = []
            continue
        states, overwritten = 0, set()
        for writer, counts in reversed(recent):
            if states < WINDOW and (compiler_made or writer.inline or i.inline):
                need = needed(writer, i, overwritten)
                if states < need:
                    found.append((need, states, writer, i))
            overwritten |= _written(writer)
            states += counts
            if states >= WINDOW:
                break
        recent.append((i, 1 + int(i.operands[0], 0) if i.name == "s_nop" else 1))
        del recent[:-WINDOW]
    return found
