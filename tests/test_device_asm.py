"""No machine instruction in the device sources is written as inline assembly:
the compiler does not look inside such a statement, so it would not insert the
wait states that gfx950 needs between a lane read that restores a spilled scalar
register and a vector instruction that reads it (two of them).  Register
constraints with an empty text are not instructions and are allowed."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2310_00317_amd", "csrc")


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*"))),
                         ids=os.path.basename)
def test_inline_assembly_holds_no_instruction(path):
    with open(path) as f:
        text = f.read().replace('\\"', '"')   # the generated kernels' text is in literals
    texts = re.findall(r'\basm\b\s*(?:volatile|goto)?\s*\(\s*"([^"]*)"', text)
    assert len(texts) == len(re.findall(r'\basm\b\s*(?:volatile|goto)?\s*\(', text))
    assert "__asm" not in text
    assert not [t for t in texts if t.strip()]
