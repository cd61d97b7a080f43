"""How tree_verify_attn splits a call, host only: by its sizes alone, never by how large a workspace it is given."""
import random

import pytest

from paper_2505_22179_amd import binding as B

TICKETS, PARTIAL = 16384, 64 * 130 * 4   # bytes: the ticket area; one range of one row tile
HEADS = [(64, 8), (32, 8), (40, 8), (16, 2), (12, 2), (8, 8), (8, 1), (4, 4), (1, 1), (128, 16), (24, 3)]


def least_workspace(M, P, Hq, Hkv):
    """the least accepted workspace, by bisection over plans (the plan of an accepted call, refused below)"""
    def accepted(nbytes):
        try:
            B.tree_verify_attn_plan_describe(M, P, Hq, Hkv, 128, nbytes)
            return True
        except B.W4A16Error as e:
            assert e.code == -5
            return False
    if accepted(0):
        return TICKETS
    lo, hi = 0, B.tree_verify_attn_workspace_bytes(M, P, Hq, Hkv, 128)
    assert accepted(hi)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if accepted(mid) else (mid, hi)
    return hi


def calls():
    rng = random.Random(5)
    for Hq, Hkv in HEADS:
        for M in (1, 4, 8, 9, 16, 17, 27, 33, 34, 50, 60, 64):
            for P in [0, 31, 100, 300, 1000, 2048, 7699, 12031, 16000, 65536] + [rng.randint(1, 30000) for _ in range(6)]:
                yield M, P, Hq, Hkv


def test_a_larger_workspace_changes_nothing():
    moved = 0
    for M, P, Hq, Hkv in calls():
        stated = B.tree_verify_attn_workspace_bytes(M, P, Hq, Hkv, 128)
        plan = B.tree_verify_attn_plan_describe(M, P, Hq, Hkv, 128, stated)
        for nbytes in (stated + 256, 4 * stated, 1 << 40):
            assert B.tree_verify_attn_plan_describe(M, P, Hq, Hkv, 128, nbytes) == plan, (M, P, Hq, Hkv, nbytes)
        rows, tiles, ranges, fused, plain = plan
        assert 1 <= rows <= 64 and (tiles - 1) * rows < Hq // Hkv * M <= tiles * rows and 1 <= ranges <= min(32, (P + M + 31) // 32)
        assert fused in (0, 1) and (ranges > 1 or not fused)
        assert ranges == 1 or TICKETS + Hkv * tiles * ranges * PARTIAL <= stated
        moved += not plain
    assert moved > 500   # the rule is at work in this sweep


def test_a_smaller_workspace_gets_the_plain_split_or_is_refused():
    for M, P, Hq, Hkv in list(calls())[::7]:
        least = least_workspace(M, P, Hq, Hkv)
        plan = B.tree_verify_attn_plan_describe(M, P, Hq, Hkv, 128, least)
        preferred = B.tree_verify_attn_plan_describe(M, P, Hq, Hkv, 128, 1 << 40)
        assert plan == preferred or plan[4] == 1
        if least > TICKETS:
            assert plan[2] == 1 or TICKETS + Hkv * plan[1] * plan[2] * PARTIAL <= least
            with pytest.raises(B.W4A16Error):
                B.tree_verify_attn_plan_describe(M, P, Hq, Hkv, 128, least - 1)
        else:
            assert plan[2] == 1


def test_the_stated_size_serves_smaller_calls_and_never_shrank():
    for Hq, Hkv in HEADS:
        for M, P in ((64, 0), (60, 100), (33, 400), (64, 2048), (64, 20000)):
            stated = B.tree_verify_attn_workspace_bytes(M, P, Hq, Hkv, 128)
            assert stated >= TICKETS + Hq * min(16, (P + M + 31) // 32) * PARTIAL   # sixteen ranges per query head
            for m in (1, 7, M):
                for p in (0, P // 3, P):
                    assert B.tree_verify_attn_workspace_bytes(m, p, Hq, Hkv, 128) <= stated


@pytest.fixture
def knobs():
    yield B.w4a16_set_param
    for name in ("attn_pack", "attn_splits", "attn_fused_merge"):
        B.w4a16_set_param(name, 0)


@pytest.mark.parametrize("splits,merge", [(0, 0), (2, 0), (9, 2), (32, 2)])
@pytest.mark.parametrize("pack", [1, 2, 3, 4, 14])
def test_the_stated_size_serves_every_way_of_cutting_tiles(knobs, pack, splits, merge):
    """no more partial results than it holds, and a ticket for every tile that the last of its workgroups merges"""
    knobs("attn_pack", pack)
    knobs("attn_splits", splits)
    knobs("attn_fused_merge", merge)
    for M, P, Hq, Hkv in list(calls())[::3] + [(M, P, Hq, Hkv) for Hq, Hkv in ((4096, 512), (4096, 4096)) for M in (1, 33, 64) for P in (0, 300, 5000)]:
        stated = B.tree_verify_attn_workspace_bytes(M, P, Hq, Hkv, 128)
        rows, tiles, ranges, fused, _ = B.tree_verify_attn_plan_describe(M, P, Hq, Hkv, 128, stated)
        assert ranges == 1 or TICKETS + Hkv * tiles * ranges * PARTIAL <= stated, (M, P, Hq, Hkv)
        assert not fused or Hkv * tiles <= TICKETS // 4, (M, P, Hq, Hkv)
        assert 1 <= rows <= (32 if pack == 4 else 64) and (tiles - 1) * rows < Hq // Hkv * M <= tiles * rows


def test_describe_rejects_what_the_call_rejects():
    for args, code in (((0, 10, 8, 8, 128), -1), ((1, -1, 8, 8, 128), -1), ((65, 10, 8, 8, 128), -4), ((1, 10, 8, 8, 64), -4),
                       ((1, 10, 64, 4, 128), -4), ((1, 10, 64, 7, 128), -1)):
        with pytest.raises(B.W4A16Error) as e:
            B.tree_verify_attn_plan_describe(*args, 1 << 30)
        assert e.value.code == code, args
    assert B.load().tree_verify_attn_plan_describe(1, 10, 8, 8, 128, 1 << 30, None) == -2
