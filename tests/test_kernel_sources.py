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


TEAM_UNITS = ("team.h", "match_core.h", "outer.hip")


def _strip(text):
    return re.sub(r"//[^\n]*", "", text)


def _parens(text, start):
    """What stands in the parentheses opened just before ``start``, its end."""
    depth, b = 1, start
    while depth:
        depth += {"(": 1, ")": -1}.get(text[b], 0)
        b += 1
    return text[start:b - 1], b


def _functions(text):
    """(name, parameters, body) of the team routines and the kernels."""
    for m in re.finditer(r"\b(team_\w+|\w+_kernel)\(", text):
        params, b = _parens(text, m.end())
        if text[b:].lstrip().startswith("{"):
            yield m.group(1), params, _body(text, b)


@pytest.mark.parametrize("unit", TEAM_UNITS)
def test_team_sizes_are_scalar(unit):
    """Routines with barriers take their sizes through uni(): a size in a vector
    register turns a branch around a barrier into a mask, and the compiler has
    reloaded spilled registers under such a mask while it was empty.  Members of
    the symmetry are loaded anew where they are named, so in a condition they go
    through uni() there."""
    seen = 0
    for name, params, body in _functions(_strip(_source(unit))):
        if "team_" not in body:  # no barrier
            continue
        if name.startswith("team_"):
            for p in re.findall(r"\bint (\w+)(?:\s*=\s*\w+)?\s*(?:,|$)", params):
                assert "%s = uni(%s);" % (p, p) in body, (name, p)
                seen += 1
        for m in re.finditer(r"\b(?:if|while|for) (?:constexpr )?\(", body):
            cond = _parens(body, m.end())[0]
            bare = re.sub(r"uni\([^()]*(?:\([^()]*\)[^()]*)*\)", "", cond)
            assert not re.search(r"\bS\.\w+", bare), (name, cond)
            seen += 1
    assert seen
