"""The global -> LDS copies written in inline assembly take their LDS address from register m0, where the compiler
keeps values of its own: it has to be an operand of the statement, set by the compiler, and never written inside."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_14423_amd", "csrc")


def _copies():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        for stmt in re.findall(r"asm volatile\((.*?)\);", open(path).read(), re.S):
            if "load_lds" in stmt or re.search(r"\bm0\b", stmt):
                yield os.path.basename(path), stmt


def test_m0_is_an_operand():
    copies = list(_copies())
    assert len(copies) >= 4
    for name, stmt in copies:
        assert '"{m0}"' in stmt and not re.search(r"\bm0\s*,", stmt), (name, stmt)


def test_wait_state_behind_the_write_of_m0():
    """One wait state between a scalar write of m0 and a copy that uses it: the compiler inserts it for its own
    instructions, not for one inside a statement."""
    for name, stmt in _copies():
        assert re.match(r'"s_nop 0\\n\\tglobal_load_lds_dword', stmt.strip()), (name, stmt)
