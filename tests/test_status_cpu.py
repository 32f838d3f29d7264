"""A step of a solve that fails must not end as success: the solve steps'
status is used wherever they are called."""
import os
import re

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1505_04340_amd", "csrc",
                   "slr_api.hip")
STEPS = ("block_sweep", "deep_sweep", "csweep", "c2sweep", "c1solve", "c_lower", "c_upper", "bsolve", "bsolve_first",
         "bsolve_et", "run_bsolve", "apply_dd", "ws_ensure", "perm_ws")


def test_no_status_is_dropped():
    with open(SRC) as f:
        text = re.sub(r"//[^\n]*", "", f.read())
    seen = set()
    for m in re.finditer(r"(?<![\w>.:])(%s)(<[^>;]*>)?\(" % "|".join(STEPS), text):
        before = text[:m.start()].rstrip()
        seen.add(m.group(1))
        # a definition, or a use of the value: never a statement of its own or a cast to void
        assert not before.endswith((";", "{", "}", "else", ")")), text[m.start() - 60:m.start() + 60]
    assert seen == set(STEPS), set(STEPS) - seen
