"""The launch plans (csrc/launch_plan.h), asked on the host: which workgroup shape and order a size gets."""
import os
import subprocess

import pytest

import shape_cases as shapes
from shape_cases import FOLDED, LONGEST_FIRST

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_query")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", os.path.join(HERE, "plan_query.cpp"), "-o", exe], check=True)

    def ask(questions):
        text = "".join(" ".join(map(str, q)) + "\n" for q in questions)
        res = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60)
        return [tuple(map(int, line.split())) for line in res.stdout.splitlines()]

    return ask


def test_only_256_row_workgroups_work_pairs_of_tiles(plans):
    # the second sweep of a pair runs downwards over every key tile: waves that split the keys would step past tile 0
    assert plans([("order", rows, FOLDED) for rows in (32, 64, 128, 256)]) == [(LONGEST_FIRST,)] * 3 + [(FOLDED,)]
    sizes = [(int(1.13 ** n), heads) for n in range(1, 115) for heads in (1, 2, 3, 5, 8, 24, 64, 100, 256)]
    for rows, order in plans([("fwd", S, h) for S, h in sizes]):
        assert rows in (32, 64, 128, 256) and (order == LONGEST_FIRST or rows == 256)
    for rows, joint, k_order, q_order in plans([("bwd", S, h) for S, h in sizes]):
        assert rows in (32, 64, 128, 256)
        assert k_order == q_order == LONGEST_FIRST or (rows == 256 and not joint)


# the sizes at which a joint launch was measured slower than a pair of folded ones by more than the runs differ
@pytest.mark.parametrize("S,heads", [(4096, 256), (8192, 64), (8192, 128), (8192, 256), (16384, 64), (32768, 32), (50000, 5), (65536, 10),
                                     (131072, 3), (131072, 5), (262144, 5)])
def test_backward_of_many_heads_keeps_the_folded_order(plans, S, heads):
    assert plans([("bwd", S, heads)]) == [(256, 0, FOLDED, FOLDED)]


@pytest.mark.parametrize("S,heads", [(50000, 5), (200000, 5), (400000, 5), (25000, 10), (131072, 5), (4096, 96)])
def test_forward_of_five_heads_keeps_the_folded_order(plans, S, heads):
    assert plans([("fwd", S, heads)]) == [(256, FOLDED)]


@pytest.mark.parametrize("S,heads", [(65536, 5), (81920, 5), (98304, 5), (40000, 10), (150000, 4), (400000, 4), (250000, 2)])
def test_forward_between_whole_rounds_stays_longest_first(plans, S, heads):
    assert plans([("fwd", S, heads)]) == [(256, LONGEST_FIRST)]


# and faster
@pytest.mark.parametrize("S,heads", [(2048, 96), (3000, 48), (4096, 48), (6000, 32), (12288, 16), (16384, 10), (25000, 8), (32768, 5), (50000, 4),
                                     (50000, 8), (65536, 5), (150000, 3)])
def test_backward_between_whole_rounds_stays_joint(plans, S, heads):
    rows, joint, k_order, q_order = plans([("bwd", S, heads)])[0]
    assert (rows, joint) == (256, 1) or (rows, k_order) == (256, LONGEST_FIRST)


@pytest.mark.parametrize("tiles,heads", [(1, 1), (2, 3), (5, 40), (31, 8), (32, 6), (63, 4), (64, 4), (65, 4), (256, 1), (512, 1), (7000, 2)])
def test_joint_order_works_every_tile_once_and_longest_first(plans, tiles, heads):
    for keys, queries in ((tiles, tiles), (tiles, 0), (0, tiles)):
        order = plans([("joint", keys, queries, heads)])[0]
        assert [r for r in order if r >= 0] == list(range(keys))
        assert [-1 - r for r in order if r < 0] == list(range(queries))


# launches of one to two rounds of workgroups, where key tiles spread among the query tiles were measured slower, and one beyond
@pytest.mark.parametrize("tiles,heads", [(13, 16), (14, 12), (9, 24), (8, 32), (22, 6), (64, 4), (64, 2), (32, 8), (65, 4)])
def test_joint_launch_works_the_key_tiles_first(plans, tiles, heads):
    assert plans([("joint", tiles, tiles, heads)])[0] == tuple(range(tiles)) + tuple(-1 - r for r in range(tiles))


def test_division_by_a_launch_constant(plans):
    top = (1 << 32) - 1
    for d in (1, 2, 3, 5, 7, 40, 65535, 65536, 1000003, (1 << 26) - 1, (1 << 31) + 1, top):
        xs = sorted({x for m in (0, 1, 2, 1000, top // d) for x in (m * d - 1, m * d, m * d + 1) if 0 <= x <= top} | {top})
        assert plans([("divide", x, d) for x in xs]) == [divmod(x, d) for x in xs]


# fp32 at head dim 64: the sizes at which shared rows were measured slower than none by more than the runs differ
def test_fp32_rows_are_shared_only_where_that_is_not_slower(plans):
    forward = [(1700, 2), (2000, 2), (2500, 1), (3000, 1), (4000, 1), (5000, 2), (5000, 4), (10000, 1)]
    assert [p[0] for p in plans([("f32rows", S, h) for S, h in forward])] == [0] * len(forward)
    backward = [(6000, 2), (7000, 4), (8000, 1), (8000, 4), (10000, 3), (12000, 2), (16000, 1), (20000, 2), (30000, 1)]
    assert [p[1] for p in plans([("f32rows", S, h) for S, h in backward])] == [0] * len(backward)
    # and faster
    forward, backward = [(1500, 3), (2000, 3), (4000, 3), (3000, 4)], [(200, 64), (300, 64), (1024, 4), (2000, 3), (3000, 2), (5000, 1)]
    assert [p[0] for p in plans([("f32rows", S, h) for S, h in forward])] == [1] * len(forward)
    assert [p[1] for p in plans([("f32rows", S, h) for S, h in backward])] == [1] * len(backward)


def test_projection_buffers_stay_inside_the_matrix(plans):
    # every tile a workgroup may name: its own, and the ones behind its last, whose buffers are empty
    for begin, end, tile_rows in ((0, 1, 64), (0, 64, 64), (130, 40001, 256), (7, 5000, 192), (4096, 4100, 128)):
        tiles = (end - begin + tile_rows - 1) // tile_rows
        ask = [("window", begin, end, t, tile_rows, int(t < tiles)) for t in range(tiles + 300)]
        covered = 0
        for (first, rows), (_, _, _, t, _, live) in zip(plans(ask), ask):
            assert begin <= first < end and first + rows <= end and (rows > 0) == bool(live)
            if live:
                assert first == begin + t * tile_rows
                covered += rows
        assert covered == end - begin


def test_gpu_tests_get_the_shapes_they_are_written_for(plans):
    assert plans([("fwd", S, h) for S, h in shapes.FWD_64_EDGES]) == [(64, LONGEST_FIRST)] * len(shapes.FWD_64_EDGES)
    assert [p[0] for p in plans([("bwd", S, h) for S, h in shapes.BWD_32_EDGES])] == [32] * len(shapes.BWD_32_EDGES)
    assert plans([("fwd", S, h) for S, h, _ in shapes.FWD_SHAPES]) == list(shapes.FWD_SHAPES.values())
    for table in (shapes.BWD_SHAPES, shapes.BWD_LONG_SHAPES):
        assert plans([("bwd", S, h) for S, h in table]) == list(table.values())
    assert plans([("lin", S - begin, K, N) for S, K, N, begin in shapes.LINEAR_SHAPES]) == list(shapes.LINEAR_SHAPES.values())
    # every shape that there is has its case
    assert {rows for rows, _ in shapes.FWD_SHAPES.values()} == {32, 64, 128, 256}
    assert set(shapes.LINEAR_SHAPES.values()) == {(64, 64), (128, 64), (128, 128), (192, 128), (256, 128), (256, 256)}


def test_the_edges_of_the_long_kernels_get_them(plans):
    for table, waves in ((shapes.FWD_LONG_EDGES, 8), (shapes.FWD_FOUR_WAVE_EDGES, 4), (shapes.FWD_LONG_SUMS, 4)):
        for (S, heads), order in table.items():
            assert plans([("fwd", S, heads), ("waves", S, heads)]) == [(256, order), (waves,)]
    for (S, heads), orders in shapes.BWD_LONG_EDGES.items():
        assert plans([("bwd", S, heads)]) == [(256, 0) + orders]
    assert plans([("bwd", S, h) for S, h in shapes.BWD_JOINT_EDGES]) == [(256, 1, LONGEST_FIRST, LONGEST_FIRST)] * len(shapes.BWD_JOINT_EDGES)
    assert plans([("bwdwaves", S, h) for S, h in shapes.BWD_JOINT_EDGES]) == [(4,)] * len(shapes.BWD_JOINT_EDGES)
    for (B, S, heads), orders in shapes.LONG_LAYOUTS.items():
        assert plans([("bwd", S, B * heads)]) == [(256, 0) + orders] and plans([("waves", S, B * heads)]) == [(4,)]
    assert plans([("waves", 3905, 128)]) == [(4,)]


# a sweep in four waves starts and ends later: where it was measured slower than one in eight
@pytest.mark.parametrize("S,heads", [(301, 193), (473, 163), (482, 227), (666, 122), (719, 177), (850, 92), (917, 256), (1074, 78), (1468, 161), (1600, 56),
                                     (1977, 50), (2444, 99), (2543, 99)])
def test_short_forward_sweeps_do_not_take_four_waves(plans, S, heads):
    assert plans([("waves", S, heads)]) == [(8,)]


# and faster, longest first for 128 rows, in launches of little more than a round
@pytest.mark.parametrize("S,heads", [(6000, 16), (8422, 12), (10116, 10), (12715, 8), (20000, 10), (25000, 4), (40000, 5), (50000, 2)])
def test_long_forward_sweeps_just_beyond_a_round_take_four_waves(plans, S, heads):
    assert plans([("fwd", S, heads), ("waves", S, heads)]) == [(256, LONGEST_FIRST), (4,)]


# joint launches of 256 rows: the sizes where four waves were measured slower than eight, and where they and not two launches were fastest
@pytest.mark.parametrize("S,heads,waves", [(961, 128, 8), (1442, 128, 8), (2115, 100, 8), (8577, 20, 4), (14528, 8, 4), (22690, 5, 4), (42591, 4, 4), (70000, 4, 4),
                                           (85099, 4, 4)])
def test_joint_backward_takes_the_faster_number_of_waves(plans, S, heads, waves):
    assert plans([("bwd", S, heads), ("bwdwaves", S, heads)]) == [(256, 1, LONGEST_FIRST, LONGEST_FIRST), (waves,)]


def test_fp32_launches_that_fill_the_chip_go_to_the_fp16_instructions(plans):
    cases = shapes.F32_SPLIT_EDGES + shapes.F32_SPLIT_ONE
    assert plans([("f32split", *c) for c in cases]) == [(1,)] * len(cases)
    # measured slower there forward, and faster
    slower = ((1990, 1, 64), (950, 4, 64), (527, 8, 64), (751, 40, 64), (1, 8454015, 64), (1945, 1, 128), (1436, 3, 128), (939, 4, 128), (1227, 5, 128), (135, 12, 128))
    faster = ((4501, 1, 64), (2969, 2, 64), (1959, 4, 64), (1251, 20, 64), (2355, 1, 128), (1262, 4, 128), (1228, 6, 128), (864, 8, 128), (899, 12, 128), (448, 40, 128))
    assert plans([("f32split", *c) for c in slower + faster]) == [(0,)] * len(slower) + [(1,)] * len(faster)
