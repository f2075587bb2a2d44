"""Wait states inside the hand-written LDS copies: nobody inserts them in inline assembly.

The LDS address travels in M0, whose scalar write needs one wait state before the copy reads it, and a copy with
a scalar base address may read registers that a vector instruction has just written: five wait states."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_12457_amd", "csrc")


def _copies():
    """(file, instructions before the first copy, whether it has a scalar base) of every asm block with an LDS copy."""
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith((".hip", ".h")):
            continue
        for block in re.findall(r"asm volatile\(\s*((?:\"[^\"]*\"\s*)+)", open(os.path.join(CSRC, name)).read()):
            lines = "".join(re.findall(r"\"([^\"]*)\"", block)).replace("\\t", "").split("\\n")
            at = [i for i, l in enumerate(lines) if l.startswith("global_load_lds")]
            if at:
                yield name, lines[:at[0]], not re.search(r",\s*off\b", lines[at[0]])


def test_lds_copies_wait_for_their_scalar_operands():
    found = list(_copies())
    assert len(found) >= 3 and any(scalar for _, _, scalar in found)
    for name, before, scalar_base in found:
        states = [int(l.split()[1]) + 1 if l.startswith("s_nop") else 1 for l in before]
        m0 = max(i for i, l in enumerate(before) if l.startswith("s_mov_b32 m0"))
        assert sum(states[m0 + 1:]) >= 1, (name, before)
        if scalar_base:
            assert sum(states) >= 5, (name, before)
