"""The library exports what its headers declare and nothing else."""
import os
import re
import shutil
import subprocess

import pytest

import paper_1902_01981_amd as cr

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADERS = [os.path.join("include", "codedreduce.h"), os.path.join("paper_1902_01981_amd", "csrc", "testing.h")]


@pytest.mark.skipif(shutil.which("nm") is None, reason="needs nm")
def test_nothing_undeclared():
    cr.load_library()
    declared = set()
    for header in HEADERS:
        with open(os.path.join(ROOT, header)) as f:
            declared |= set(re.findall(r"^(?:int|void|const char \*)\s*\**(cr_\w+)\(", f.read(), flags=re.M))
    listed = subprocess.run(["nm", "-D", "--defined-only", cr.LIB_PATH], check=True, capture_output=True, text=True).stdout
    assert {line.split()[-1] for line in listed.splitlines()} == declared
