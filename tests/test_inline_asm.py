"""Operands of inline asm blocks of several instructions."""
import os
import re

import pytest

import paper_2510_19262_amd as rs

CSRC = os.path.join(os.path.dirname(os.path.abspath(rs.__file__)), "csrc")


def _asm_statements(text):
    """Bodies of the asm statements of a source, comments removed."""
    text = re.sub(r"//[^\n]*", "", text)
    for m in re.finditer(r"\basm\s*(?:volatile\s*)?\(", text):
        depth, i = 1, m.end()
        while depth:
            if text[i] == '"':
                i = text.index('"', i + 1)
            depth += {"(": 1, ")": -1}.get(text[i], 0)
            i += 1
        yield text[m.end():i - 1]


@pytest.mark.parametrize("name", sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".h"))))
def test_operands_written_before_the_last_instruction_are_early_clobber(name):
    # without '&' the compiler may give such an operand the register of an input that a later instruction still reads
    with open(os.path.join(CSRC, name)) as f:
        for body in _asm_statements(f.read()):
            template, _, operands = body.partition(":")
            while template.count('"') % 2:                     # a colon inside the template
                more, _, operands = operands.partition(":")
                template += ":" + more
            if template.count("\\n") == 0:
                continue
            for constraint in re.findall(r'"([=+][^"]*)"', operands):
                assert "&" in constraint, f"{name}: {constraint} in {body.strip()[:80]}"
