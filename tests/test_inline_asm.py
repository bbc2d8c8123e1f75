"""Source check of the hand-written assembly (no GPU needed): registers that a statement writes without an output operand
have to be on its clobber list, or the compiler may keep something of its own there."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_29233_amd", "csrc")
STATEMENT = re.compile(r"asm volatile\s*\((.*?)\);", re.S)


def statements(directory):
    for path in sorted(glob.glob(os.path.join(directory, "*.h")) + glob.glob(os.path.join(directory, "*.hip"))):
        for m in STATEMENT.finditer(open(path).read()):
            yield os.path.basename(path), m.group(1)


@pytest.mark.parametrize("written,name", [(r"s_mov_b32 m0,", '"m0"'), (r"s_cmp_", '"scc"'), (r"load_lds|ds_write", '"memory"')])
def test_what_assembly_writes_is_declared(written, name):
    found = [(f, text) for f, text in statements(CSRC) if re.search(written, text)]
    assert found, "no statement of this kind is left: drop its row"
    for f, text in found:
        assert name in text.rsplit(":", 1)[1], (f, text)
