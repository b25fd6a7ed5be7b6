"""Conventions of the kernel sources that no result shows when they are broken."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1403_5524_amd", "csrc")


def _source(name):
    with open(os.path.join(CSRC, name)) as f:
        return f.read()


def _body(text, start):
    """The braces' content from the first one after ``start``."""
    a = text.index("{", start)
    depth = 0
    for b in range(a, len(text)):
        depth += {"{": 1, "}": -1}.get(text[b], 0)
        if depth == 0:
            return text[a + 1:b]
    raise ValueError("unbalanced")


def test_group_decision_is_not_contracted():
    """Two kernels of two units make it and must agree to the last bit."""
    text = _source("polesum_group.h")
    body = _body(text, text.index("pg_decide("))
    assert body.lstrip().startswith("#pragma clang fp contract(off)")
    for unit in ("polesum.hip", "polesum_group.hip"):
        assert "pg_decide(" in _source(unit)
