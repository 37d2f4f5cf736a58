"""Inline assembly that copies to LDS through m0 (CPU, source check).

The compiler must know that m0 changes (it may hold a value there for a copy of
its own), so a statement that sets it has it as an input and output operand.
The compiler does not see the statement's buffer load as one either and adds
none of the wait states the load may need: five between a vector instruction
that writes a scalar register (a spilled one read back with v_readlane) and
the vector memory instruction that reads it."""
import glob
import os
import re

from paper_2506_20686_amd import build as hipbuild


def statements():
    for path in sorted(glob.glob(os.path.join(hipbuild.CSRC, "*"))):
        if os.path.isfile(path):
            for s in re.findall(r"asm volatile\((.*?)\);", open(path).read(), flags=re.S):
                if re.search(r"\bm0\b|\blds\b", s):
                    yield os.path.basename(path), s


def wait_states(code):
    """Wait states before the first buffer load of an asm template."""
    n = 0
    for line in re.split(r"\\n\\t|\\n", code):
        op = line.split()
        if op[0].startswith("buffer_load"):
            return n
        n += int(op[1]) + 1 if op[0] == "s_nop" else 1
    raise AssertionError("no buffer load in " + code)


def test_m0_statements():
    found = list(statements())
    assert found
    for name, s in found:
        template, operands = s.split(":", 1)
        code = "".join(re.findall(r'"([^"]*)"', template))
        assert '"+{m0}"(' in operands, (name, s)
        assert wait_states(code) >= 5, (name, s)
