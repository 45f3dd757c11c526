"""Memory instructions in asm blocks read scalar registers, which a vector instruction (v_readlane of a spilled register, say) may
have written just before: the hardware wants five wait states in between, and the compiler does not look into asm blocks for them.
Every block has to hold them itself."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2406_04984_amd", "csrc")


def _states(text):
    """wait states that the instructions of `text` take: one each, s_nop N takes N + 1"""
    ops = [o.strip() for o in text.split("\n") if o.strip()]
    return sum(int(o.split()[1]) + 1 if o.startswith("s_nop") else 1 for o in ops)


def test_scalar_operands_of_memory_instructions():
    seen = 0
    for path in glob.glob(os.path.join(CSRC, "*")):
        for block in re.findall(r'\basm volatile\(\s*((?:"[^"]*"\s*)+)', open(path).read()):
            text = "".join(re.findall(r'"([^"]*)"', block)).replace("\\n", "\n").replace("\\t", " ")
            at = re.search(r"\b(buffer|global|flat|scratch)_\w+", text)
            if at:
                seen += 1
                assert _states(text[:at.start()]) >= 5, (os.path.basename(path), text)
    assert seen
