"""Hand-written DPP blocks of the kernels, read as text (no GPU).  A DPP read needs two wait states after the vector write of
its register.  At the head of a block the compiler may have placed a copy right before, so every block that reads through DPP
starts with `s_nop 1`, and so must any other that follows it on the same registers; inside a block they are counted here."""
import os
import re
import subprocess

import pytest

from paper_2602_08810_amd import build

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_08810_amd", "csrc")
FILES = sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".hpp")) and f != "valu_probe.hip")


def _blocks(text):
    """(line, body) of every asm statement; strings are taken whole, so parentheses inside them do not count."""
    text = re.sub(r"//[^\n]*", "", text)
    for m in re.finditer(r"\basm\b\s*(?:volatile)?\s*\(", text):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = text[i]
            if c == '"' and text[i - 1] != "\\":
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            i += 1
        yield text.count("\n", 0, m.start()) + 1, text[m.end():i - 1]


def _dpp_macros():
    text = "".join(open(os.path.join(CSRC, f)).read() for f in FILES).replace("\\\n", " ")
    defs = dict(re.findall(r"#define (LRNNX_\w+)(?:\([^)]*\))?([^\n]*)", text))
    names = {n for n, body in defs.items() if "_dpp" in body}
    while True:                                            # macros made of such macros
        more = {n for n, body in defs.items() if any(re.search(rf"\b{k}\b", body) for k in names)} - names
        if not more:
            return names
        names |= more


@pytest.mark.parametrize("name", FILES)
def test_dpp_blocks_start_with_wait_states(name):
    macros = _dpp_macros()
    for line, body in _blocks(open(os.path.join(CSRC, name)).read()):
        if "_dpp" in body or any(re.search(rf"\b{m}\b", body) for m in macros):
            assert re.match(r'\s*"s_nop [1-9]', body), f"{name}:{line}: a DPP block without s_nop 1 at its head"


def _instructions(body):
    """The instructions of an asm statement after preprocessing: its string literals up to the first colon outside them."""
    text, i = "", 0
    while i < len(body) and body[i] != ":":
        if body[i] == '"':
            j = i + 1
            while body[j] != '"':
                j += 2 if body[j] == "\\" else 1
            text += body[i + 1:j]
            i = j
        i += 1
    return [s.strip() for s in text.replace("\\t", " ").split("\\n") if s.strip()]


def _hazards(instructions):
    """(reader, wait states since the write) of every DPP read that comes fewer than two wait states after the vector write of its
    register; an instruction is one wait state, s_nop K is K + 1."""
    now, written, bad = 0, {}, []
    for ins in instructions:
        op, *rest = ins.split(None, 1)
        if op == "s_nop":
            now += int(rest[0]) + 1
            continue
        regs = re.findall(r"%\d+", rest[0]) if rest else []
        if "_dpp" in op and regs[1] in written and now - written[regs[1]] < 2:       # (the first source is the one read through DPP)
            bad.append((ins, now - written[regs[1]]))
        now += 1
        if op.startswith("v_"):
            written[regs[0]] = now
    return bad


def test_hazards_are_seen():
    write, read = "v_mul_f32 %0, %1, %1", "v_add_f32_dpp %2, %0, %1 row_shr:1"
    assert _hazards([write, read]) and _hazards([write, "s_nop 0", read]) and _hazards([write, "v_mov_b32 %3, %1", read])
    assert not _hazards([write, "s_nop 1", read]) and not _hazards([write, "s_nop 0", "v_mov_b32 %3, %1", read])
    assert not _hazards([write, "v_add_f32_dpp %2, %1, %0 row_shr:1"])               # not the operand that is moved between lanes


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
@pytest.mark.parametrize("name,scans", [("selective_fwd.hip", 6), ("selective_bwd.hip", 3), ("selective_cplx_fwd.hip", 2), ("selective_cplx_bwd.hip", 1)])
def test_dpp_reads_inside_blocks_wait(name, scans):
    """Every block as the compiler gets it, its macros expanded."""
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-E", "-P", os.path.join(CSRC, name)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    own = r.stdout[r.stdout.index("namespace lrnnx {"):]
    blocks = [b for b in (_instructions(body) for _, body in _blocks(own)) if any("_dpp" in i for i in b)]
    assert sum(len(b) > 3 for b in blocks) == scans, "all of the file's scans"
    for b in blocks:
        assert not _hazards(b), f"{name}: {_hazards(b)} in\n" + "\n".join(b)
