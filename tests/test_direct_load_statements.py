"""The inline assembly of the direct global -> LDS loads, read from the sources.  The compiler keeps no distance between what it
schedules before such a statement and the loads inside: each has to see to its own.  A scalar register that a vector instruction
has written may be read by a load five wait states later, one that a scalar instruction has written at once; M0 one later."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2210_09603_amd", "csrc")


def statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        for m in re.finditer(r"asm volatile\((.*?)\);", open(path).read(), re.S):
            text = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', m.group(1).split("\n        :")[0].split('" :')[0] + '"'))
            if "global_load_lds" in text:
                yield os.path.basename(path), [i.strip() for i in re.split(r"\\n\\t|\\n", text) if i.strip()]


def wait_states(instruction):
    return int(instruction.split()[1]) + 1 if instruction.startswith("s_nop") else 1


def test_direct_loads_keep_their_distance():
    seen = 0
    for where, code in statements():
        for i, load in enumerate(code):
            if not load.startswith("global_load_lds"):
                continue
            base = load.split(",")[1].strip()
            own = any(re.match(r"s_mov_b64 %s," % re.escape(base), c) for c in code[:i])
            assert own or sum(map(wait_states, code[:i])) >= 5, (where, code)
            m0 = max(j for j in range(i) if re.match(r"s_\w+ m0,", code[j]))
            assert sum(map(wait_states, code[m0 + 1:i])) >= 1, (where, code)
            seen += 1
    assert seen >= 3
