"""Hand-written DPP blocks of the kernels, read as text (no GPU).  A DPP read needs two wait states after the vector write of
its register; inside a block the author counts them, at its head the compiler may have placed a copy right before, so
every block that reads through DPP starts with `s_nop 1`, and so must any other that follows it on the same registers."""
import os
import re

import pytest

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
