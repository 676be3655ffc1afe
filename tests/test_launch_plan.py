"""How launches are laid out (csrc/lychee_plan.h), compiled for the host (no GPU needed)."""
import ctypes
import itertools
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_04541_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no C++ compiler")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("plan") / "plan.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                           os.path.join(ROOT, "tests", "c", "plan.cpp"), "-o", lib])
    dll = ctypes.CDLL(lib)
    dll.front_plan.argtypes = [ctypes.c_int32] * 6 + [ctypes.c_void_p]
    dll.list_row_entries.argtypes = [ctypes.c_int32] * 3
    return dll


def front_plan(plan, selects, copies, thresholds, gated, r_blocks, n_wg):
    out = (ctypes.c_int32 * 2)()
    plan.front_plan(selects, copies, thresholds, int(gated), r_blocks, n_wg, out)
    return out[0], out[1]


def gets_stuck(n_front, n_aside, n_wg, resident):
    """Workgroups start in index order as places come free.  One below n_front runs its units first; one below
    n_aside leaves then, every other one takes pieces that wait (the worst case) until all units are done."""
    started, waiting = 0, 0
    while started < n_wg:
        if waiting == resident and started < n_front:
            return True                 # every place is held by a workgroup that waits for one not started
        if waiting == resident:
            return False                # all units are done or running: the waiting ones go on
        started += 1
        if started > n_aside:
            waiting += 1
    return False


def gets_stuck_on_xcds(n_aside, n_tail, n_wg, resident, n_xcd):
    """The workgroups are dealt to the XCDs in turn, and every XCD starts its own in index order as its places come free,
    however far the others are.  Those below n_aside run their units and leave; the last n_tail wait until all
    pieces are done; the others have the pieces, which wait (the worst case) until all units are done."""
    queue = [list(range(x, n_wg, n_xcd)) for x in range(n_xcd)]
    held = [[] for _ in range(n_xcd)]
    units, pieces = n_aside, n_wg - n_aside - n_tail      # workgroups of each kind that have not ended
    while True:
        moved = False
        for x in range(n_xcd):
            while queue[x] and len(held[x]) < resident:
                held[x].append(queue[x].pop(0))
            for w in list(held[x]):
                if w < n_aside:
                    units -= 1
                elif w < n_wg - n_tail and units == 0:
                    pieces -= 1
                elif w < n_wg - n_tail or pieces:
                    continue
                held[x].remove(w)
                moved = True
        if not moved:
            return any(queue) or any(held)


def layers(rng):
    """What consecutive layers of a call bring: (selects, copies, thresholds, gated, blocks streamed)."""
    batch = rng.choice([1, 2, 3, 8, 64, 100, 256])
    kv = rng.choice([1, 2, 8, 64])
    prev_r, cur_r = rng.randint(0, kv), rng.randint(0, kv)
    blocks = sum((rng.choice([1, 64, 3001, 32768, 131072]) + 63) // 64 for _ in range(batch))
    selects, copies = rng.choice([(batch * prev_r, batch * (kv - prev_r)), (0, batch * kv), (0, 0)])
    thresholds = rng.choice([0, 4 * batch * cur_r])
    return selects, copies, thresholds, bool(selects + copies) and rng.random() < 0.7, cur_r * blocks


def test_no_piece_waits_for_a_workgroup_that_may_not_have_started(plan):
    rng = random.Random(5)
    cases = [(0, 800, 0, True, 0)] + [layers(rng) for _ in range(400)]   # (copies alone, every piece a gated gather)
    for case in cases:
        selects, copies, thresholds, gated, _ = case
        for n_wg in (1, 2, 7, 8, 9, 37, 256, 512, 513, 768):
            n_front, n_aside = front_plan(plan, *case, n_wg)
            assert 0 <= n_aside <= n_front <= n_wg
            assert n_front > 0 or selects + copies + thresholds == 0
            assert n_aside < n_wg            # somebody takes the pieces
            if not (gated or thresholds):
                continue
            for resident in {min(n_wg, r) for r in (7, 8, 100, 256, 512)}:
                assert not gets_stuck(n_front, n_aside, n_wg, resident), (case, n_wg, resident, n_front, n_aside)


def test_no_workgroup_waits_for_one_that_its_xcd_cannot_start(plan):
    """Units in front, pieces, and selects at the end of the grid that wait for all pieces, also where the XCDs hold far
    fewer workgroups than the grid has."""
    rng = random.Random(9)
    with_tail = 0
    for case in [layers(rng) for _ in range(60)]:
        _, _, thresholds, _, r_blocks = case
        for n_wg in (8, 37, 64, 512, 768):
            tail = plan.tail_selects(thresholds // 4, r_blocks, n_wg)
            with_tail += tail > 0
            _, n_aside = front_plan(plan, 0, case[1], thresholds, False, r_blocks, n_wg)
            assert n_aside + tail < n_wg and (n_aside > 0 or thresholds == 0)   # (what pieces wait for waits for nothing)
            for n_xcd, resident in ((8, 1), (8, 2), (8, 64), (1, 1), (1, 100)):
                assert not gets_stuck_on_xcds(n_aside, tail, n_wg, resident, n_xcd), (case, n_wg, n_xcd, resident)
    assert with_tail > 20


def test_copies_that_nothing_waits_for_are_done_on_the_way(plan):
    assert front_plan(plan, 0, 800, 0, False, 4096, 512) == (512, 0)
    assert front_plan(plan, 0, 5, 0, False, 4096, 512) == (5, 0)
    assert front_plan(plan, 0, 800, 0, True, 4096, 512) == (128, 128)    # gated: a quarter of the grid, to themselves


def test_a_block_granular_list_holds_every_block(plan):
    rng = random.Random(6)
    for _ in range(2000):
        k = rng.choice([1, 5, 204, 4096, 131072])
        n = int(2 ** rng.uniform(0, 24))
        for max_len in {n, n // 64 * 64 + 1, 64 * (k + 16384) + rng.choice([0, 1, 63, 64, 65]), 2000001, 1 << 24}:
            if 1 <= max_len <= 1 << 24:
                assert plan.list_row_entries(max_len, k, 1) >= (max_len + 63) // 64, (max_len, k)
                # lists of positions may overflow: their size, and with it the workspace's, is what it was
                assert plan.list_row_entries(max_len, k, 0) == min(max(4 * k, k + 16384, max_len // 64),
                                                                   (max_len + 63) // 64 * 64)


def test_front_units_do_not_outlast_half_of_the_streaming(plan):
    """Units run in turn (about 8 us each) on fewer workgroups than they could have only where that takes no
    longer than half of the streaming (5.5 ns a block of 64 rows), or where a sixteenth of the grid is in front."""
    rng = random.Random(7)
    for case in [(256, 256, 1024, True, 64 * 4 * 128)] + [layers(rng) for _ in range(400)]:
        units = sum(case[:3])
        for n_wg in (16, 37, 256, 512, 768):
            n_front, n_aside = front_plan(plan, *case, n_wg)
            if n_aside == 0 or n_front in (units, n_wg // 4):
                continue
            turns = -(-units // n_front)
            assert turns <= 1 + case[4] * 5.5e-3 / 2 / 8, (case, n_wg, n_front)


def test_gather_blocks_are_shorter_where_rows_fill_the_launch(plan):
    for r, g, max_len, n_wg, rows in ((6144, 0, 4096, 512, 64), (6144, 1, 4096, 512, 48), (0, 12, 768, 1, 64),
                                      (0, 13, 832, 1, 48), (2 ** 30, 2 ** 30, 1 << 24, 768, 48), (0, 0, 1, 512, 64),
                                      (0, 512, 114687, 512, 64), (0, 512, 114688, 512, 48)):
        assert plan.gather_block_rows(r, g, max_len, n_wg) == rows


def test_selects_at_the_end_of_the_grid_leave_the_pieces_their_workgroups(plan):
    for rows, r_blocks, n_wg, tail in ((8, 2 ** 30, 512, 8), (16, 8193, 512, 0), (16, 8192, 512, 16), (9, 2 ** 30, 512, 0),
                                       (32, 4096, 512, 32), (32, 4097, 512, 0), (33, 64, 512, 0), (1, 64, 63, 0),
                                       (1, 2 ** 30, 64, 1), (5, 5, 64, 0), (0, 0, 512, 0)):
        assert plan.tail_selects(rows, r_blocks, n_wg) == tail
        front, aside = front_plan(plan, 0, 8 * rows, 4 * rows, False, r_blocks, n_wg)
        assert n_wg - aside - tail >= n_wg // 2


def test_rules_select_apart_where_many_rows_end_a_short_streaming(plan):
    for rows, r_blocks, n_wg, apart in ((128, 64, 512, 0), (129, 129, 512, 1), (129, 16384, 512, 1), (129, 16385, 512, 0),
                                        (16384, 2 ** 30, 512, 0), (1, 1, 4, 0), (1, 1, 3, 1)):
        assert plan.rules_apart(rows, r_blocks, n_wg) == apart


def test_rules_select_behind_a_launch_whose_runs_hold_several_short_rows(plan):
    for r_blocks, n_wg, shortest, apart in ((188, 13, 6, 1), (156, 13, 6, 0), (157, 13, 6, 1), (942, 17, 70, 0), (0, 1, 6, 0),
                                            (2 ** 31 - 1, 768, 2 ** 18 + 5, 1), (2 * 768 * (2 ** 18 + 5), 768, 2 ** 18 + 5, 0)):
        assert plan.rows_in_turn(r_blocks, n_wg, shortest) == apart


def test_quotients_are_exact_over_their_whole_range(plan):
    """Around multiples of the divisor, where a rounded quotient goes wrong first, and at the top of the range, where the
    product of quotient and divisor passes 2^31; with reciprocals that are one unit in the last place off either way."""
    rng = random.Random(8)
    divisors = [1, 2, 3, 5, 7, 48, 64, 511, 512, 1000, 4097, 65535, 2 ** 20 + 1, 2 ** 23 - 1, 2 ** 24 - 1]
    divisors += [int(2 ** rng.uniform(0, 24)) for _ in range(150)]
    for b in divisors:
        top = 2 ** 31 - b - 1
        near = [0, b, 2 ** 22, 2 ** 24, 2 ** 30, top] + [int(2 ** rng.uniform(0, 31)) for _ in range(20)]
        for n in near:
            for a in (n - n % b - 1, n - n % b, n - n % b + 1, n - n % b + b - 1, n):
                if 0 <= a <= top:
                    for ulps in (-1, 0, 1):
                        assert plan.quot(a, b, ulps) == a // b, (a, b, ulps)


def test_one_unit_takes_a_threshold_where_the_launch_is_short_and_the_rest_fits_registers(plan):
    fits = 32 * 256
    for n, L, r_blocks, n_wg, margin, alone in ((2048, 32768, 1536, 512, 6.0, 1), (2048, 32768, 2560, 512, 6.0, 1),
                                                (2048, 32768, 2561, 512, 6.0, 0), (3900, 32768, 1536, 512, 6.0, 1),
                                                (4000, 32768, 1536, 512, 6.0, 0), (3900, 32768, 1536, 512, 60.0, 0),
                                                (1, 20000, 320, 64, 6.0, 1), (1, 20000, 321, 64, 6.0, 0),
                                                (1, 1 << 24, 0, 512, 6.0, 0)):
        got = plan.threshold_alone(n, L, r_blocks, n_wg, ctypes.c_float(margin), fits)
        assert got == alone, (n, L, r_blocks, n_wg, margin)
        if got:   # what reaches the threshold, for f of the n best among 512 sampled rows, with a tenth to spare
            f = n * 512 / L
            assert (f + margin * f ** 0.5 + 6) * L / 512 <= 0.9 * fits * (1 + 1e-5)


def test_merges_of_a_phased_step_are_dealt_evenly(plan):
    """Every head is merged once, however a KV head's heads are divided into retrieval and sparse ones; where workgroups
    take several units no unit is empty and every one has as many heads; one kind or one head a unit only where each
    has a workgroup of its own (or heads of many slots take up to three rounds)."""
    splits = set()
    for kv_heads, group, sparse, others, slots, n_wg in itertools.product(
            (1, 64, 128, 129, 255, 256, 257, 512, 513, 4096, 127 * 16 * 64), (1, 2, 3, 4), (0, 1), (0, 8), (4, 96, 97, 194), (1, 512, 768)):
        split = plan.merge_split(kv_heads, group, sparse, others, slots, n_wg)
        parts = plan.merge_parts(split, group)
        splits.add(split)
        for rmask in range(1 << group) if sparse else [(1 << group) - 1]:
            masks = [plan.merge_heads(split, part, rmask, group) for part in range(parts)]
            assert sum(masks) == (1 << group) - 1 and sum(bin(m).count("1") for m in masks) == group, (split, rmask, masks)
            if kv_heads * parts + others > n_wg:
                assert len({bin(m).count("1") for m in masks}) == 1, (split, rmask, masks)
        if kv_heads * parts + others > n_wg and parts > 1:
            assert slots > 96 and kv_heads * parts <= 3 * n_wg
        assert sparse or split != 1      # (a dense step's units of the sparse kind would all be empty)
    assert splits == {0, 1, 2}


def test_no_launch_has_the_generation_of_flags_that_nobody_has_written(plan):
    """Flags start at 0 and a threshold word that was not asked for is 0: across the wrap of the 32 bits too no
    generation is, and it differs from the one before it."""
    plan.first_generation.restype = plan.next_generation.restype = ctypes.c_uint32
    plan.next_generation.argtypes = [ctypes.c_uint32]
    assert plan.first_generation() != 0
    for start in (plan.first_generation(), 2 ** 31 - 2, 2 ** 32 - 3):
        gen = start
        for _ in range(6):
            after = plan.next_generation(gen)
            assert after not in (0, gen)
            gen = after
    with open(os.path.join(CSRC, "lychee_layer.hip")) as f:   # (what the launches do: the only store of the word)
        assert [line.strip() for line in f if "store_agent(A->gen," in line] == ["store_agent(A->gen, next_generation(gen));"]
