"""What the compiler is not told it cannot respect: inline assembly in the kernels' sources."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_13581_amd", "csrc")


def _asm_statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        text = open(path).read()
        for m in re.finditer(r"\basm\s+volatile\s*\(", text):
            depth, i = 1, m.end()
            while depth:
                depth += {"(": 1, ")": -1}.get(text[i], 0)
                i += 1
            yield os.path.basename(path), text[m.end():i - 1]


def test_assembly_that_writes_m0_says_so():
    """The compiler keeps values of its own in m0 (dynamic register indexes, LDS offsets of its own copies): a statement that
    writes it lists it as clobbered."""
    seen = 0
    for path, body in _asm_statements():
        code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', body.split("::")[0]))
        if re.search(r"s_mov\w* m0\b", code):
            seen += 1
            assert '"m0"' in body.rsplit(":", 1)[1], (path, body)
    assert seen >= 1
