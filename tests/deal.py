"""The rule by which decode attention deals its rows out, asked of the header that the library is built from
(tests/host/attend_deal_check.cpp, compiled with g++), so that a test can say which kernel its case runs."""
import functools
import os
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host", "attend_deal_check.cpp")
INC = os.path.join(ROOT, "paper_2601_07891_amd", "csrc")


@functools.lru_cache(None)
def checker():
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = os.path.join(tempfile.mkdtemp(prefix="deal"), "attend_deal_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fwrapv", "-I", INC, SRC, "-o", exe], check=True)
    return exe


def form(heads, group, max_rows, window, store_rows):
    """"plain n" or "streamed n": n splits of each head; "list n" or "block n": one list for n wavefronts."""
    args = [str(int(x)) for x in (heads, group, max_rows, window, store_rows)]
    return subprocess.run([checker(), *args], check=True, capture_output=True, text=True).stdout.strip()
