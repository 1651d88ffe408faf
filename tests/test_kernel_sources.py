"""CPU test of the inline assembly in the kernel sources: the compiler inserts no
wait states inside a block or between it and the instructions around it, so a
block of DPP operations has to begin and end with its own (two states between a
vector write and a DPP read, one between a vector write and a lane read)."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1107_2619_amd", "csrc")


def _blocks(text):
    """Template of every asm statement (strings and macro calls up to the operands)."""
    text = re.sub(r"//[^\n]*", "", text)
    for m in re.finditer(r"\basm\s+(?:volatile\s*)?\(", text):
        depth, k, quoted = 1, m.end(), False
        while depth and not (depth == 1 and not quoted and text[k] == ":"):
            if text[k] == '"' and text[k - 1] != "\\":
                quoted = not quoted
            elif not quoted:
                depth += {"(": 1, ")": -1}.get(text[k], 0)
            k += 1
        yield text[m.end():k].strip()


def test_dpp_blocks_wait_at_both_ends():
    found = 0
    for path in glob.glob(os.path.join(CSRC, "*.h*")):
        with open(path) as f:
            text = f.read()
        for body in _blocks(text):
            if "dpp" not in body.lower():
                continue
            found += 1
            assert re.match(r'"s_nop [1-7]\\n', body), (path, body[:60])
            assert re.search(r'"s_nop [0-7](\\n(\\t)?)?"$', body), (path, body[-60:])
    assert found >= 2
