"""How decode attention deals its rows out (paper_2601_07891_amd/csrc/attend_deal.h):
tests/host/attend_deal_check.cpp, compiled here with g++ from the header that the kernels use.  CPU only."""
import subprocess

from tests.deal import program


def test_parts_stay_inside_the_list_whatever_the_lengths_say():
    r = subprocess.run([program("attend_deal_check")], capture_output=True, text=True)
    assert r.returncode == 0 and " 0 faults" in r.stdout, r.stdout


def test_a_list_longer_than_its_sum_can_hold_is_caught():
    # the planted mistake: lists are made however much the store could hold
    r = subprocess.run([program("attend_deal_check"), "--plant"], capture_output=True, text=True)
    assert r.returncode == 1 and "part outside the list" in r.stdout
