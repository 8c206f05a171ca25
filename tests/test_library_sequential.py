"""The evaluation stream of programs compiled node by node
(gp_eval_sequential.h: user functions, user losses, long and deep programs),
on the CPU: its words stay within the program's
room and, run by a plain interpreter, give the prefix list's own value.  A
call's instructions with their reloads once took more than the room of its
node (a one-argument function x0 + c on a stack twelve deep: 64 word pairs
for every 63 of room), so that runs of some 1,200 such calls wrote into the
next program."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("seq") / "sequential_check")
    subprocess.run(["g++", "-O2", "-g", "-std=c++17", "-ffp-contract=off",
                    "-Wno-unknown-pragmas", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2110_11226_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "sequential_check.cpp")], check=True)
    return exe


@pytest.mark.parametrize("args", [("chains",), ("random", "4000"), ("malformed", "4000")])
def test_streams_stay_in_their_room_and_give_the_programs_value(checker, args):
    r = subprocess.run([checker, *args], capture_output=True, text=True)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-2000:])
    assert int(r.stdout.split()[0]) > 500
