"""The short square root and reciprocal that the polar factor, the draws and the
walk's ranks use, over every float of their ranges, and the squared limits of the
membership tests for every bound (tests/native/short_forms_check.hip)."""
import os
import subprocess

import pytest

from paper_2403_09990_amd import build as B

pytestmark = pytest.mark.gpu

EXE = os.path.join(B.ROOT, "tests", "native", "short_forms_check")


def test_short_forms_are_correctly_rounded():
    if not os.path.exists(EXE):
        B.build_tool(EXE + ".hip", EXE)
    r = subprocess.run([EXE], capture_output=True, text=True, timeout=60)
    print(r.stdout, r.stderr)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok")
