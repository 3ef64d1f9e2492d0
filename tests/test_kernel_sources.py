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


def test_shared_arrays_read_as_vectors_are_aligned():
    """An LDS array of scalars is only as aligned as its element type says, unless it says more: one that a kernel accesses through
    a pointer to a vector type says __align__(16)."""
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip"))):
        for kernel in re.split(r"\b__global__\b", open(path).read())[1:]:
            vectors = set(re.findall(r"\*\((?:const )?(?:u?int[24]|float[24]|u32x4\w*|f32x4\w*|floatx4\w*) \*\)&(\w+)\[", kernel))
            for aligned, names in re.findall(r"__shared__ (__align__\(16\) )?(?:float|int|u?int16_t|u?int32_t) ([^;]+);", kernel):
                for name in re.findall(r"(\w+)(?:\[[^\]]*\])+", names):
                    if name in vectors:
                        seen += 1
                        assert aligned, (os.path.basename(path), name)
    assert seen >= 7
