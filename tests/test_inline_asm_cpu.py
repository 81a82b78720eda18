"""Inline assembly in the kernels: m0, which the compiler reserves and takes no clobber of,
is saved before the code that writes it and put back after it."""
import glob
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1609_00958_amd", "csrc")
SOURCES = sorted(os.path.basename(f) for f in glob.glob(os.path.join(CSRC, "*"))
                 if f.endswith((".hip", ".h")))


def _functions(text):
    """Name and body of every function whose assembly writes m0."""
    for m in re.finditer(r"asm volatile\([^;]*?\bs_\w+ m0\b", text):
        head = text.rfind("__device__", 0, m.start())
        name = re.search(r"(\w+)\(", text[head:]).group(1)
        yield name, m.start()


@pytest.mark.parametrize("source", SOURCES)
def test_m0_is_put_back(source):
    with open(os.path.join(CSRC, source)) as f:
        text = f.read()
    writers = {name for name, _ in _functions(text)} - {"restore_m0"}
    for name in writers:
        calls = [m.start() for m in re.finditer(r"\b%s\(" % name, text)]
        uses = [c for c in calls if "__device__" not in text[text.rfind("\n", 0, c):c]]
        assert uses
        for c in uses:
            # the nearest of the two before the call saves, the nearest after it restores
            assert text.rfind("= save_m0()", 0, c) > text.rfind("restore_m0(m0)", 0, c)
            after, save = text.find("restore_m0(m0)", c), text.find("= save_m0()", c)
            assert after >= 0 and (save < 0 or after < save)


def test_the_check_sees_the_writers():
    names = set()
    for source in SOURCES:
        with open(os.path.join(CSRC, source)) as f:
            names |= {name for name, _ in _functions(f.read())}
    assert "load_to_lds" in names
