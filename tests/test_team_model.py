"""The bitset traversal's teams (paper §IV-A, §IV-C) as a CPU model under ThreadSanitizer: threads
play wavefronts that hand sub-trees over inside their team (claims of idle bits, mailboxes, the
count of held sub-trees, the meeting before the team looks for work) and donate up to four nodes at
once to the worklist. Invariants checked by the model: no node lost, none taken twice, counters back
at zero, every slot free for its next lap, no mail left; by ThreadSanitizer: no data race on boxes,
worklist slots and what a team's first wavefront passes on. Planted protocol mistakes show the
checks bite."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "worklist_model", "team_model.cpp")
ENV = dict(os.environ, TSAN_OPTIONS="halt_on_error=0 exitcode=66")


def build(tmp, mutation=0):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is not installed")
    out = os.path.join(tmp, f"team_model_{mutation}")
    subprocess.run([gxx, "-O1", "-g", "-std=c++17", "-pthread", "-fsanitize=thread",
                    f"-DVC_MODEL_MUTATION={mutation}", SRC, "-o", out],
                   check=True, capture_output=True, timeout=300)
    return out


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    return build(str(tmp_path_factory.mktemp("tm")))


def run(binary, *args):
    return subprocess.run([binary, *map(str, args)], capture_output=True, text=True, timeout=300,
                          env=ENV)


# teams, wavefronts per team, ring capacity, donation threshold, instances, tree depth, stack, seed
CASES = [
    (2, 4, 64, 8, 1, 18, 20, 1),
    (1, 8, 64, 4, 3, 17, 20, 2),        # one team: handovers, and donations to itself
    (4, 4, 128, 40, 5, 17, 20, 3),
    (2, 16, 256, 64, 4, 18, 20, 5),     # the largest team
    (6, 1, 64, 16, 4, 17, 20, 6),       # workgroups of one wavefront: donations only
    (3, 4, 64, 0, 8, 16, 20, 8),        # threshold 0: handovers only
    (3, 2, 4096, 4000, 4, 17, 1, 4),    # rings of one entry: always full
    (2, 8, 4096, 4000, 6, 17, 3, 5),
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}x{c[1]}_thr{c[3]}_stack{c[6]}" for c in CASES])
def test_teams_lose_nothing_and_have_no_data_race(model, case):
    r = run(model, *case)
    assert "ThreadSanitizer" not in r.stderr, r.stderr[-2000:]
    assert r.returncode == 0, r.stderr
    assert r.stdout.startswith("ok ")
    handed, donated = int(r.stdout.split()[3]), int(r.stdout.split()[6])
    assert (handed > 0) == (case[1] > 1) and (donated > 0 or case[3] == 0 or case[0] == 1), r.stdout


def test_handover_that_is_not_counted_is_caught(tmp_path):
    r = run(build(str(tmp_path), 1), 2, 8, 128, 16, 3, 17, 20, 1)
    assert r.returncode == 1 and "below zero" in r.stderr


@pytest.mark.parametrize("mutation", [2, 3], ids=["relaxed_mail", "relaxed_claim"])
def test_relaxed_handover_is_a_data_race(tmp_path, mutation):
    """A mail flag set with a relaxed store (the box is read before it is written), or an idle bit
    claimed with a relaxed operation (the box is written before its last content has been read)."""
    r = run(build(str(tmp_path), mutation), 2, 8, 128, 16, 3, 17, 20, 1)
    assert "ThreadSanitizer: data race" in r.stderr
