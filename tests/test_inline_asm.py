"""What the compiler does not do inside an asm statement, checked over the kernels' sources: the wait states that the hardware leaves to
the program, and operands that must not share a register."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_05207_amd", "csrc")
LITERAL = re.compile(r'"((?:[^"\\]|\\.)*)"')


def split_operands(text):
    """The template and the operand lists of what stands between the brackets of an asm statement: colons outside of literals part them."""
    parts, depth = [""], False
    for c in text:
        depth ^= c == '"'
        if c == ":" and not depth:
            parts.append("")
        else:
            parts[-1] += c
    return parts


def statements():
    out = []
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        src = re.sub(r"//[^\n]*", "", open(path).read())
        macros = {m.group(1): (m.group(2), m.group(3)) for m in re.finditer(r"#define (\w+)\((\w+)\) ((?:[^\n\\]|\\.)*)", src) if '"' in m.group(3)}
        for m in re.finditer(r"\basm(?: volatile)?\((.*?)\);", src, re.S):
            parts = split_operands(m.group(1))

            def expand(call):
                arg, body = macros[call.group(1)]
                return re.sub(r"#" + arg + r"\b", '"' + call.group(2) + '"', body)

            template = re.sub(r"\b(\w+)\((\d+)\)", expand, parts[0])
            text = "".join(LITERAL.findall(template)).replace("\\n", "\n").replace("\\t", "")
            lines = [x.strip() for x in text.split("\n") if x.strip() and not x.strip().startswith(";")]
            out.append((os.path.basename(path) + ":" + str(src[: m.start()].count("\n") + 1), lines, [LITERAL.findall(p) for p in parts[1:]]))
    return out


STATEMENTS = statements()


def test_they_are_found():
    assert any(len(lines) > 30 for _, lines, _ in STATEMENTS)            # the rank of sixteen keys


@pytest.mark.parametrize("where,lines,operands", [s for s in STATEMENTS if s[1]], ids=lambda x: x if isinstance(x, str) else "")
def test_wait_states(where, lines, operands):
    """Two states between a vector instruction that writes a carry and one that reads it, between one that writes a register and a
    row operation on it (gfx940 and later)."""
    since = {"vcc": 9}                                                    # states since the register was last written
    since.update({f"%{k}": 0 for k in range(9)})                          # an operand may have been written just before
    for line in lines:
        name, _, rest = line.partition(" ")
        if name == "s_nop":
            since = {r: n + 1 + int(rest) for r, n in since.items()}
            continue
        ops = [x.strip().split()[0] for x in rest.split(",")]
        reads = ops[1:] if "_co_" not in name else ops[2:]
        if "vcc" in reads:
            assert since["vcc"] >= 2, f"{where}: {line}"
        if "_dpp" in name:
            assert since[reads[0]] >= 2, f"{where}: {line}"
        since = {r: n + 1 for r, n in since.items()}
        since[ops[0]] = 0
        if "_co_" in name:
            since["vcc"] = 0


@pytest.mark.parametrize("where,lines,operands", [s for s in STATEMENTS if s[1]], ids=lambda x: x if isinstance(x, str) else "")
def test_early_clobbers(where, lines, operands):
    """An output that is written before the last line that reads an input has a register of its own (&): without it a read-write operand may
    share one with an input that the compiler knows to be equal."""
    outputs = [c for c in operands[0]] if operands else []
    inputs = [f"%{len(outputs) + k}" for k in range(len(operands[1]) if len(operands) > 1 else 0)]
    reads = [n for n, line in enumerate(lines) if any(re.search(re.escape(i) + r"\b", line) for i in inputs)]
    for k, constraint in enumerate(outputs):
        writes = [n for n, line in enumerate(lines) if re.match(rf"\w+ %{k}\b", line)]
        if writes and reads and writes[0] < reads[-1]:
            assert "&" in constraint, f"{where}: operand {k} is {constraint!r}"


@pytest.mark.parametrize("where,lines,operands", [s for s in STATEMENTS if s[1]], ids=lambda x: x if isinstance(x, str) else "")
def test_scalar_operands_may_be_fresh(where, lines, operands):
    """A scalar register that a vector instruction has just written (a lane read, a reload of a spilled scalar) is to be waited for by who
    reads it in a vector instruction: an asm statement that takes one starts with the two states."""
    takes = any(c.lstrip("+=&") in ("s", "sgpr") for c in sum(operands[1:2], []))
    assert not takes or re.match(r"s_nop [1-9]", lines[0]), where


def test_dynamic_lds_is_aligned_for_vectors():
    """LDS sized at the launch begins behind a kernel's static LDS, wherever that ends, unless its declaration asks for more: kernels read it in vectors."""
    found = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip"))):
        for line in open(path).read().split("\n"):
            if "extern __shared__" in line:
                found += 1
                assert "__align__(16)" in line, f"{os.path.basename(path)}: {line.strip()}"
    assert found >= 2
