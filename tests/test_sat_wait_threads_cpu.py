"""The grid-wide wait of hb_sat2d as the kernel compiles it (csrc/sat_wait.hpp), run with threads as workgroups: one and two groups, fewer running at
a time than there are, wait limits from none to plenty, the words cleared by workgroup 0 or by whoever looks first, six launches in
a row on the same words.  Every workgroup ends, every region is finished and none before those it reads, and nothing of the
launch's number is left.  Where a second launch writes to the same words, every workgroup still ends."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("sat_wait") / "sat_wait_threads")
    subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", "-I", os.path.join(HERE, "..", "paper_2512_02371_amd", "csrc"),
                    os.path.join(HERE, "sat_wait_threads.cpp"), "-o", exe], check=True)
    return exe


def run(program, *args):
    r = subprocess.run([program] + [str(a) for a in args], stdout=subprocess.PIPE, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout


@pytest.mark.parametrize("claim_polls", [0, 3, 64])
@pytest.mark.parametrize("nwg,first,slots,wait_limit", [
    (2, 2, 2, 10000), (2, 2, 2, 1), (2, 1, 1, 0), (8, 4, 3, 0), (8, 4, 8, 2), (12, 12, 12, 3), (3, 2, 3, 50), (17, 17, 4, 0), (40, 20, 7, 3), (40, 24, 7, 0), (97, 49, 5, 1), (97, 97, 97, 10000), (200, 100, 16, 2),
    (64, 32, 64, 0), (64, 32, 64, 10000), (160, 152, 30, 5), (33, 8, 33, 1)])
def test_every_workgroup_ends_and_every_region_is_finished(program, nwg, first, slots, wait_limit, claim_polls):
    for seed in range(20 if nwg <= 16 else 3):            # the rare orders show with few workgroups
        run(program, "launches", nwg, first, slots, wait_limit, claim_polls, seed)


@pytest.mark.parametrize("nwg,first", [(8, 8), (12, 6)])
def test_words_that_something_else_writes_do_not_hold_a_workgroup(program, nwg, first):
    run(program, "words", nwg, first, nwg, 100, 64, 1)
