"""What the HIP sources must not hold, checked on their text."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_37988_amd", "csrc")


def test_no_instruction_in_inline_assembly():
    """Lane swaps and DPP reads need two wait states after a vector write of their operand, and an MFMA's
    accumulator must not be written while it is in flight: the compiler counts these only for
    instructions it sees, so no asm statement holds one (an empty asm that only hides a value is fine)."""
    found = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            src = re.sub(r"//[^\n]*", "", f.read())
        for m in re.finditer(r"\basm\b\s*(?:volatile\s*)?\(\s*((?:\"[^\"]*\"\s*)+)", src):
            found += 1
            text = "".join(re.findall(r"\"([^\"]*)\"", m.group(1)))
            assert not text.strip(), f"{os.path.basename(path)}: asm({text!r})"
    assert found > 0  # the empty ones: the pattern still finds asm statements
