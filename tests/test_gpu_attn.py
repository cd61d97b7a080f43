"""GPU: tree_verify_attn through the C ABI against the fp64 oracle (paper section 2.1).
Tolerance: max |err| <= 1e-2 and relative Frobenius error <= 1e-3."""
import numpy as np
import pytest
import torch

from oracle import reference as R
from paper_2505_22179_amd import binding as B
from paper_2505_22179_amd import inputs as I
from tests.test_attn_plan_host import least_workspace

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(autouse=True)
def _reset_knobs():
    yield
    B.w4a16_set_param("attn_splits", 0)
    B.w4a16_set_param("attn_pack", 0)
    B.w4a16_set_param("attn_row_tiles", 0)
    B.w4a16_set_param("attn_fused_merge", 0)


def run_attn(a: I.AttnInputs, ws=None):
    q, k, v = (torch.from_numpy(t).to(DEV) for t in (a.q, a.k, a.v))
    mask = torch.from_numpy(a.mask).to(DEV)
    out = torch.full((a.M + 1, a.Hq, a.D), 77.0, dtype=torch.float16, device=DEV)
    if ws is None:
        ws = B.new_workspace(B.tree_verify_attn_workspace_bytes(a.M, a.P, a.Hq, a.Hkv, a.D))
    B.tree_verify_attn(q, k, v, mask, out, a.M, a.P, a.Hq, a.Hkv, a.D, a.scale, ws)
    torch.cuda.synchronize()
    o = out.cpu().numpy()
    assert (o[a.M:] == np.float16(77.0)).all()
    return o[:a.M]


def check(out16, ref64, what):
    err = np.abs(out16.astype(np.float64) - ref64)
    rel = np.linalg.norm(out16.astype(np.float64) - ref64) / np.linalg.norm(ref64)
    assert err.max() <= 1e-2, f"{what}: max abs {err.max():.3g}"
    assert rel <= 1e-3, f"{what}: rel fro {rel:.3g}"
    return float(err.max()), float(rel)


CASES = [
    # M, P, Hq, Hkv, tree
    (60, 2048, 64, 8, "random"),     # the tree-verify configuration
    (60, 2048, 64, 8, "chain"),
    (7, 2048, 64, 8, "chain"),       # sequence-draft verification
    (1, 2048, 64, 8, "identity"),    # plain decode
    (64, 100, 8, 8, "random"),
    (17, 0, 16, 4, "random"),        # no prefix: only the tree itself
    (1, 0, 8, 1, "identity"),        # a single key
    (33, 31, 8, 2, "identity"),
    (48, 5, 4, 1, "random"),
    (8, 1000, 64, 8, "random"),      # 8 rows x 8 heads of a KV group fill one 64-row tile exactly
    (5, 70, 24, 3, "random"),        # 40 of 64 tile rows in use, three KV heads
    (16, 333, 16, 4, "chain"),       # 4 heads x 16 rows
    (3, 2, 12, 2, "chain"),          # fewer keys than one step
    (12, 300, 32, 4, "random"),      # groups of 8 heads, two heads per 24-row tile
    (7, 129, 12, 2, "chain"),        # groups of 6 heads: three per 21-row tile (42 rows would need the tall tile)
    (8, 10001, 16, 2, "random"),     # long prefixes: many rounds per key range, a ragged last step
    (3, 65536, 8, 8, "chain"),
]


@pytest.mark.parametrize("M,P,Hq,Hkv,tree", CASES)
def test_attn_parity(M, P, Hq, Hkv, tree):
    print(f"attn parity M={M} P={P} Hq={Hq} Hkv={Hkv} {tree}", flush=True)
    depth = 6 if M > 6 else max(M - 1, 0)
    a = I.make_attn(8000 + M + P + Hq, M, P, Hq, Hkv, 128, tree=tree, depth=depth)
    ref64, _ = R.tree_verify_attn(a.q, a.k, a.v, a.mask, a.scale)
    for pack in ((0, 1, 2) if Hq > Hkv else (0,)):   # heads of a KV group sharing a tile (by size, never, whole group)
        B.w4a16_set_param("attn_pack", pack)
        for row_tiles in (0, 2, 4):   # by tile height; 32 rows per wavefront (one or two row groups); all 64
            B.w4a16_set_param("attn_row_tiles", row_tiles)
            for splits in (0, 1, 3, 6, 16):
                B.w4a16_set_param("attn_splits", splits)
                B.w4a16_set_param("attn_fused_merge", 2)   # the last workgroup of a tile merges its key ranges
                got = run_attn(a)
                stats = check(got, ref64, f"M={M} P={P} {tree} splits={splits} pack={pack} row_tiles={row_tiles}")
                B.w4a16_set_param("attn_fused_merge", 1)   # a second kernel does: the same arithmetic in the same order
                two = run_attn(a)
                assert np.array_equal(two.view(np.uint16), got.view(np.uint16)), (splits, pack, row_tiles)
                B.w4a16_set_param("attn_fused_merge", 0)   # chosen by size
                assert np.array_equal(run_attn(a).view(np.uint16), got.view(np.uint16)), (splits, pack, row_tiles)
    print("   ", stats, flush=True)


@pytest.mark.parametrize("M,P,Hq,Hkv", [(1, 1100, 8, 2), (17, 40, 8, 2), (27, 1100, 12, 2), (33, 0, 10, 2), (64, 1100, 10, 2), (13, 300, 64, 8)])
def test_even_tiles_and_many_ranges(M, P, Hq, Hkv):
    """tiles that end inside a head (the group's rows cut evenly), one and up to 32 key ranges, both merges: against
    the oracle, and the two merges bit for bit"""
    print(f"even tiles M={M} P={P} Hq={Hq} Hkv={Hkv}", flush=True)
    a = I.make_attn(8500 + M + P + Hq, M, P, Hq, Hkv, 128, depth=6 if M > 6 else max(M - 1, 0))
    ref64, _ = R.tree_verify_attn(a.q, a.k, a.v, a.mask, a.scale)
    for pack in (3, 0):
        for splits in (1, 3, 17, 32):
            for row_tiles in (0, 2):
                B.w4a16_set_param("attn_pack", pack)
                B.w4a16_set_param("attn_splits", splits)
                B.w4a16_set_param("attn_row_tiles", row_tiles)
                got = []
                for merge in (1, 2):
                    B.w4a16_set_param("attn_fused_merge", merge)
                    got.append(run_attn(a))
                    check(got[-1], ref64, f"pack={pack} splits={splits} row_tiles={row_tiles} merge={merge}")
                assert np.array_equal(got[0].view(np.uint16), got[1].view(np.uint16)), (pack, splits, row_tiles)


@pytest.mark.parametrize("M,P,Hq,Hkv,least_differs", [
    (13, 4100, 40, 8, False), (32, 90, 64, 8, False), (40, 16001, 32, 8, False),   # another split, which the plain one's space holds
    (1, 7699, 32, 8, True), (4, 16000, 8, 8, True), (4, 300, 40, 8, True), (34, 16000, 12, 2, True)])   # and does not hold
def test_plan_by_size(M, P, Hq, Hkv, least_differs):
    """calls whose split is not the plain one: it follows from the sizes alone, so the stated workspace and a much larger one
    give the same bits; a workspace that does not hold it gets the plain split"""
    stated = B.tree_verify_attn_workspace_bytes(M, P, Hq, Hkv, 128)
    least = least_workspace(M, P, Hq, Hkv)
    plans = [B.tree_verify_attn_plan_describe(M, P, Hq, Hkv, 128, n) for n in (least, stated, 4 * stated)]
    print(f"M={M} P={P} heads {Hq}/{Hkv}: {least} bytes {plans[0]}, {stated} bytes {plans[1]}", flush=True)
    assert plans[1][4] == 0 and plans[2] == plans[1] and (plans[0] != plans[1]) == least_differs and plans[0][4] == least_differs
    a = I.make_attn(8600 + M + P + Hq, M, P, Hq, Hkv, 128, depth=6 if M > 6 else max(M - 1, 0))
    ref64, _ = R.tree_verify_attn(a.q, a.k, a.v, a.mask, a.scale)
    got = run_attn(a)
    check(got, ref64, f"M={M} P={P} heads {Hq}/{Hkv}")
    assert np.array_equal(run_attn(a, B.new_workspace(4 * stated)).view(np.uint16), got.view(np.uint16)), "a larger workspace, other bits"
    check(run_attn(a, B.new_workspace(least)), ref64, f"M={M} P={P} heads {Hq}/{Hkv}, {least} of {stated} bytes")


def test_attn_determinism_and_workspace_reuse():
    a = I.make_attn(8100, 60, 2048, 64, 8, 128)
    ws = B.new_workspace(B.tree_verify_attn_workspace_bytes(a.M, a.P, a.Hq, a.Hkv, a.D))
    first = run_attn(a, ws)
    for _ in range(4):
        assert np.array_equal(run_attn(a, ws).view(np.uint16), first.view(np.uint16))
    # the fused merge leaves its tickets at zero: the same workspace serves calls of other shapes in between
    b = I.make_attn(8101, 8, 500, 64, 8, 128)
    ref_b, _ = R.tree_verify_attn(b.q, b.k, b.v, b.mask, b.scale)
    for _ in range(2):
        check(run_attn(b, ws), ref_b, "shared workspace, second shape")
        assert np.array_equal(run_attn(a, ws).view(np.uint16), first.view(np.uint16))


def test_masked_draft_keys_have_no_influence():
    a = I.make_attn(8200, 40, 300, 16, 2, 128)
    base = run_attn(a)
    j = 25
    a.k[a.P + j] += np.float16(2.0)
    a.v[a.P + j] -= np.float16(1.0)
    pert = run_attn(a)
    for i in range(a.M):
        same = np.array_equal(pert[i].view(np.uint16), base[i].view(np.uint16))
        assert same == (a.mask[i, j] == 0), i


@pytest.mark.parametrize("gain", [6.0, 24.0])
def test_peaked_softmax(gain):
    """queries scaled up so that a handful of keys carry each row (logit spread of tens): the running-maximum
    rescaling across key steps, key ranges and the merge has to hold where exp() spans its whole range"""
    a = I.make_attn(8300 + int(gain), 60, 700, 16, 2, 128)
    a.q = (a.q.astype(np.float32) * gain).astype(np.float16)
    ref64, _ = R.tree_verify_attn(a.q, a.k, a.v, a.mask, a.scale)
    for splits in (0, 1, 5):
        B.w4a16_set_param("attn_splits", splits)
        for row_tiles in (0, 2):
            B.w4a16_set_param("attn_row_tiles", row_tiles)
            check(run_attn(a), ref64, f"peaked softmax x{gain} splits={splits} row_tiles={row_tiles}")


@pytest.mark.parametrize("M,P,Hq,Hkv", [(32, 0, 8, 8), (31, 95, 8, 8), (1, 255, 8, 4), (33, 600, 8, 4), (60, 300, 16, 2), (64, 1025, 8, 2)])
def test_short_tiles(M, P, Hq, Hkv):
    """tiles of at most 32 rows, whose wavefronts walk the keys on their own: full and partial tiles that end inside a head, fewer key
    steps than wavefronts, exactly eight and nine of them, ranges shorter than a round, both merges"""
    a = I.make_attn(8360 + M + P, M, P, Hq, Hkv, 128)
    ref64, _ = R.tree_verify_attn(a.q, a.k, a.v, a.mask, a.scale)
    ws = B.new_workspace(16384 + 2 * Hq * 32 * 64 * 130 * 4)   # more tiles than heads, asked for below
    B.w4a16_set_param("attn_pack", 4)
    for splits in (1, 2, 3, 9):
        B.w4a16_set_param("attn_splits", splits)
        plan = B.tree_verify_attn_plan_describe(M, P, Hq, Hkv, 128, ws.numel() * ws.element_size())
        assert plan[0] <= 32 and plan[2] <= splits
        got = []
        for merge in (1, 2):
            B.w4a16_set_param("attn_fused_merge", merge)
            got.append(run_attn(a, ws))
            check(got[-1], ref64, f"M={M} P={P} heads {Hq}/{Hkv} splits={splits} merge={merge}")
        assert np.array_equal(got[0].view(np.uint16), got[1].view(np.uint16)), splits


@pytest.mark.parametrize("M,P,Hq,Hkv", [(64, 300, 8, 1), (60, 300, 16, 2), (33, 600, 8, 4)])
def test_short_tiles_in_the_stated_workspace(M, P, Hq, Hkv):
    """more tiles than query heads, with as many key ranges as the stated workspace holds"""
    a = I.make_attn(8370 + M + P, M, P, Hq, Hkv, 128)
    ref64, _ = R.tree_verify_attn(a.q, a.k, a.v, a.mask, a.scale)
    B.w4a16_set_param("attn_pack", 4)
    for splits in (0, 16):
        B.w4a16_set_param("attn_splits", splits)
        check(run_attn(a), ref64, f"M={M} P={P} heads {Hq}/{Hkv} splits={splits}")


@pytest.mark.parametrize("pack", [3, 4])
@pytest.mark.parametrize("M,P,Hq,Hkv", [(5, 700, 21, 7), (33, 900, 24, 3), (64, 300, 20, 5), (9, 1500, 6, 2), (40, 333, 5, 1), (17, 650, 33, 11)])
def test_grids_that_eight_does_not_divide(M, P, Hq, Hkv, pack):
    """every (row tile, key range) has its workgroup, however many of either there are"""
    a = I.make_attn(8380 + M + P, M, P, Hq, Hkv, 128)
    ref64, _ = R.tree_verify_attn(a.q, a.k, a.v, a.mask, a.scale)
    B.w4a16_set_param("attn_pack", pack)
    for splits, merge in ((1, 0), (3, 1), (3, 2), (7, 1), (9, 2), (0, 0)):
        B.w4a16_set_param("attn_splits", splits)
        B.w4a16_set_param("attn_fused_merge", merge)
        check(run_attn(a), ref64, f"M={M} P={P} heads {Hq}/{Hkv} pack={pack} splits={splits} merge={merge}")


@pytest.mark.parametrize("M,P,Hq,Hkv,ranges", [(28, 11477, 28, 4, 16), (39, 15370, 28, 4, 12), (49, 6524, 20, 5, 12)])
def test_few_key_value_heads_are_not_slow(M, P, Hq, Hkv, ranges):
    """the plan of the call against full tiles in as many ranges as fill a grid that eight divides: 1.4 to 1.7 times as long while XCDs read all keys
    wherever eight did not divide the grid"""
    a = I.make_attn(8390, M, 0, Hq, Hkv, 128)
    q, mask = torch.from_numpy(a.q).to(DEV), torch.from_numpy(a.mask).to(DEV)
    k, v = (torch.randn(P + M, Hkv, 128, device=DEV).to(torch.float16) for _ in range(2))
    out, ws = torch.empty_like(q), B.new_workspace(B.tree_verify_attn_workspace_bytes(M, P, Hq, Hkv, 128))

    def usec():
        best = 1e9
        for _ in range(5):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(50):
                B.tree_verify_attn(q, k, v, mask, out, M, P, Hq, Hkv, 128, a.scale, ws)
            end.record()
            end.synchronize()
            best = min(best, begin.elapsed_time(end) * 20)
        return best
    default = usec()
    B.w4a16_set_param("attn_pack", 3)
    B.w4a16_set_param("attn_splits", ranges)
    full = usec()
    print(f"attention M={M} P={P} heads {Hq}/{Hkv}: {default:.1f} us, full tiles {full:.1f}", flush=True)
    assert default <= 1.25 * full


@pytest.mark.parametrize("M", [20, 45])
@pytest.mark.parametrize("rise", [0.02, 0.3, -0.3])
def test_maxima_that_move_along_the_keys(M, rise):
    """scores that rise by `rise` powers of two from key to key, so that a row's maximum moves in every step; falling ones leave
    it in the first"""
    a = I.make_attn(8350, M, 700, 16, 2, 128)
    a.q[..., 0] = np.float16(4.0)
    a.k[..., 0] = (rise / (4.0 * a.scale * 1.4426950408889634) * np.arange(a.k.shape[0])).astype(np.float16)[:, None]
    ref64, _ = R.tree_verify_attn(a.q, a.k, a.v, a.mask, a.scale)
    for splits in (0, 1, 5):
        B.w4a16_set_param("attn_splits", splits)
        check(run_attn(a), ref64, f"M={M} rise={rise} splits={splits}")


def test_constant_values_come_back_exactly():
    """V = c for every key: any convex combination of it is c, whatever the weights"""
    a = I.make_attn(8400, 33, 515, 8, 2, 128)
    a.v[...] = np.float16(0.375)
    for splits in (0, 4):
        B.w4a16_set_param("attn_splits", splits)
        got = run_attn(a).astype(np.float32)
        assert np.abs(got - 0.375).max() <= 2.0 ** -11 * 0.375 * 2, np.abs(got - 0.375).max()
