"""The inline assembler statements of the kernels' sources: what the compiler is
free to place around one, or to give its operands, cannot change its result."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2602_19699_amd", "csrc")


def _closing(text, at):
    """Index past the parenthesis that closes the one at `at` (string literals skipped)."""
    depth, i = 0, at
    while True:
        c = text[i]
        if c == '"':
            i = re.compile(r'"(?:[^"\\]|\\.)*"').match(text, i).end()
            continue
        depth += c == "("
        depth -= c == ")"
        i += 1
        if depth == 0:
            return i


def _statements():
    """(file, line, text) of every asm statement, with the file's macros
    written out: object-like and function-like ones by their bodies."""
    out = []
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        joined = text.replace("\\\n", "  ")
        macros = dict(re.findall(r"#define (\w+)(?:\([^)]*\))? +([^\n]*)", joined))
        for m in re.finditer(r"\basm\s*(?:volatile\s*)?\(", text):
            s = text[m.end() - 1:_closing(text, m.end() - 1)]
            for _ in range(20):  # macros in macros
                t = re.sub(r"\b(CBIC_\w+)\b", lambda k: f" {macros.get(k.group(1), '')} ", s)
                if t == s:
                    break
                s = t
            out.append((os.path.basename(path), text[:m.start()].count("\n") + 1, s))
    return out


STATEMENTS = _statements()
DPP = [s for s in STATEMENTS if "row_newbcast" in s[2]]


def test_statements_are_found():
    assert len(STATEMENTS) > 5 and len(DPP) > 2


@pytest.mark.parametrize("name,line,text", DPP, ids=[f"{n}:{i}" for i, (n, _, _) in enumerate(DPP)])
def test_dpp_reads_wait_in_their_own_statement(name, line, text):
    # a vector write of a register needs two wait states before a DPP read of
    # it, which the compiler does not insert inside a statement; the wait of
    # another statement does not cover a copy or reload placed between them
    assert re.match(r'\(\s*"s_nop 1\\n', text), f"{name}:{line} reads by DPP without waiting first"


def _outputs(text):
    """The output part of a statement: between its first and second colon outside literals."""
    bare = re.sub(r'"((?:[^"\\]|\\.)*)"', lambda m: '"' + m.group(1).replace(":", ";") + '"', text)
    return bare.split(":")[1]


@pytest.mark.parametrize("name,line,text", DPP, ids=[f"{n}:{i}" for i, (n, _, _) in enumerate(DPP)])
def test_accumulators_share_no_register_with_an_input(name, line, text):
    # these statements write accumulators before they have read the last input:
    # without the early-clobber mark an input whose value the compiler knows to
    # equal an accumulator's could be given the accumulator's register
    outs = re.findall(r'"([^"]*)"\s*\(', _outputs(text))
    assert outs and all(o == "+&v" for o in outs), f"{name}:{line} {outs}"
