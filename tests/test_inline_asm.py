"""What hand-written instructions tell the compiler about the registers they change."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_13473_amd", "csrc")


def _asm_statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        text = open(path).read() if os.path.isfile(path) else ""
        text = re.sub(r"//[^\n]*", "", text)
        for m in re.finditer(r"\basm\s*(?:volatile\s*)?\((.*?)\)\s*;", text, flags=re.S):
            yield os.path.basename(path), m.group(1)


def test_asm_that_writes_m0_says_so():
    """m0 is a register that the compiler may hold a value in: a statement that moves into it and does not
    list it as clobbered may destroy that value."""
    writers = [(f, s) for f, s in _asm_statements() if re.search(r"\bs_\w+\s+m0\b", s)]
    assert writers
    for f, s in writers:
        clobbers = s.rsplit(":", 1)[1]
        assert '"m0"' in clobbers, f"{f}: {s}"
