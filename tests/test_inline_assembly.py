"""What the kernels' inline assembly has to tell the compiler, read from the sources (CPU).

The compiler moves, copies and spills values between two statements as it likes, so each has to name what it needs.
"""
import glob
import os
import re

import paper_2510_07651_amd

SOURCES = sorted(glob.glob(os.path.join(os.path.dirname(paper_2510_07651_amd.__file__), "csrc", "*.h*")))


def _statements():
    for path in SOURCES:
        text = open(path).read()
        for m in re.finditer(r"asm volatile\((.*?)\);", text, re.S):
            yield "%s:%d" % (os.path.basename(path), text[:m.start()].count("\n") + 1), m.group(1)


def test_transfers_to_lds_name_their_address_register():
    """m0 holds a transfer's LDS address: an operand of the statement, not what an earlier one happens to have left there."""
    transfers = [(at, asm) for at, asm in _statements() if "load_lds" in asm]
    assert len(transfers) >= 3
    assert all('"{m0}"(' in asm and "s_nop 0" in asm for _, asm in transfers), transfers


def test_no_statement_writes_m0():
    assert not [at for at, asm in _statements() if re.search(r"s_mov_b32 m0", asm)]


def test_no_load_returns_before_its_wait():
    """A load in assembly hands out registers that are not filled yet: only the compiler's own loads may."""
    assert not [at for at, asm in _statements() if re.search(r"\b(ds_read|global_load_dword|buffer_load)", asm)]
