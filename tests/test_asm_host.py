"""What the inline assembly of csrc/ owes the compiler, on the host."""
import os
import re

from paper_2508_00960_amd.build import CSRC


def asm_statements():
    """[(file, text of the statement)] of every inline assembly statement in csrc/"""
    out = []
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".h", ".hip")):
            with open(os.path.join(CSRC, name)) as f:
                out += [(name, m.group(0)) for m in re.finditer(r"asm\s+volatile\s*\(.*?\)\s*;", f.read(), re.S)]
    return out


def test_statements_that_write_m0_say_so():
    writes = [(name, text) for name, text in asm_statements() if re.search(r"s_\w+ m0,", text)]
    assert writes
    for name, text in writes:
        assert '"m0"' in text.rsplit(":", 1)[1], f"{name}: {text}"
