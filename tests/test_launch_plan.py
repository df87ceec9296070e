"""The launch plans (csrc/launch_plan.h), asked on the host: which workgroup shape and order a size gets."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
FOLDED, LONGEST_FIRST = 0, 1


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_query")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", os.path.join(HERE, "plan_query.cpp"), "-o", exe], check=True)

    def ask(questions):
        text = "".join(" ".join(map(str, q)) + "\n" for q in questions)
        res = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60)
        return [tuple(x if x == "pair" else int(x) for x in line.split()) for line in res.stdout.splitlines()]

    return ask


def test_only_256_row_workgroups_work_pairs_of_tiles(plans):
    # the second sweep of a pair runs downwards over every key tile: waves that split the keys would step past tile 0
    assert plans([("order", rows, FOLDED) for rows in (32, 64, 128, 256)]) == [(LONGEST_FIRST,)] * 3 + [(FOLDED,)]
    sizes = [(int(1.13 ** n), heads) for n in range(1, 115) for heads in (1, 2, 3, 5, 8, 24, 64, 100, 256)]
    for rows, order in plans([("fwd", S, h) for S, h in sizes]):
        assert rows in (32, 64, 128, 256) and (order == LONGEST_FIRST or rows == 256)
    for plan in plans([("bwd", S, h) for S, h in sizes]):
        if plan[0] != "pair":
            assert plan[0] in (32, 64, 128, 256)
            continue
        for rows, order in (plan[1:3], plan[3:5]):
            assert order == LONGEST_FIRST or rows == 256
