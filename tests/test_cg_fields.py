"""The CG steps that many workgroups finish for themselves never read what their own launch writes.

A workgroup may start after workgroup 0 of the same launch has written its
results, and the wavefronts of one workgroup may see different values; so the
fields of CgCtl that a body reads and those it assigns must not meet.
"""
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def body(text, name):
    at = text.index("{", text.index(f"void {name}("))
    depth, end = 0, at
    while True:
        depth += {"{": 1, "}": -1}.get(text[end], 0)
        end += 1
        if depth == 0:
            return re.sub(r"//.*", "", text[at:end])


@pytest.mark.parametrize("name", ["cg_update_body", "cg_direction_body"])
def test_reads_and_writes_do_not_meet(name):
    text = open(os.path.join(ROOT, "paper_1309_5609_amd", "csrc", "dst_cg.h")).read()
    code = body(text, name)
    written = set(re.findall(r"ctl->(\w+)\s*=(?!=)", code))
    read = set(re.findall(r"ctl->(\w+)", re.sub(r"ctl->\w+\s*=(?!=)", "", code)))
    assert written and read
    assert not written & read, written & read
