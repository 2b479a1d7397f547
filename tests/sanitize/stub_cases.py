"""Planner cases for the sanitizer build (run by test_host_sanitized.py, with
REFCACHE_LIB naming a library whose kernel launchers are the checking stubs of
stub_launchers.cpp; skipped otherwise).  Every successful call hands its
schedule to a stub that aborts on a broken invariant; pointers are fake and
never dereferenced."""
import ctypes
import os
import random

import pytest

import paper_2608_21229_amd as rc
from oracle import masks as om
from tests.test_capi_host import FAKE, _full, _full_ws, _prefill, _step, random_layout

pytestmark = pytest.mark.skipif(not os.environ.get("REFCACHE_STUB"), reason="needs the stub-launcher build")


def stub(name):
    f = getattr(rc.lib(), name)
    f.restype = ctypes.c_long
    return f()


def launches():
    return stub("rc_stub_launches")


def _prefill_fp8(L, B=1, H=2, D=128):
    return rc.lib().rc_ref_kv_prefill_fp8(ctypes.byref(L.c), B, H, D, 0.1, FAKE, FAKE, FAKE, H * D, FAKE, None, FAKE,
                                          FAKE, FAKE, None)


@pytest.mark.parametrize("preset", ["paper", "perref", "isolated", "dense"])
def test_random_layouts_through_every_entry(preset):
    rng = random.Random(11)
    for _ in range(200):
        kinds, lens = random_layout(rng)
        L = rc.Layout(list(zip(kinds, lens)), preset)
        vis = om.PRESETS[preset](kinds)
        B, H = rng.choice([1, 2, 3]), rng.choice([1, 2, 5, 24, 64])
        D = rng.choice([64, 128])
        ts = H * D
        n0 = launches()
        assert _full(L, B=B, H=H, D=D, ts=ts, lse=FAKE) == rc.RC_OK
        assert launches() == n0 + (1 if sum(lens) else 0)
        assert stub("rc_stub_work_groups") == L.work_groups(rc.ENTRY_FULL, B, H, D)
        # with the last-round split's workspace: the attention launch, plus the
        # merge when it splits
        need = L.full_workspace_bytes(B, H, D)
        n0 = launches()
        assert _full_ws(L, B=B, H=H, D=D, ts=ts, lse=FAKE, ws=FAKE, wsb=need) == rc.RC_OK
        assert launches() == n0 + (1 if sum(lens) else 0) + (1 if need else 0)
        assert stub("rc_stub_work_groups") == L.work_groups(rc.ENTRY_FULL, B, H, D, rc.SPLITS_LAST_ROUND)
        if not om.is_cacheable(kinds, vis):
            assert _prefill(L, B=B, H=H, D=D, ts=ts) == rc.RC_ERR_MASK_NOT_CACHEABLE
            continue
        assert _prefill(L, B=B, H=H, D=D, ts=ts, lse=FAKE) == rc.RC_OK
        if L.rows(rc.ROWS_STATIC):
            assert stub("rc_stub_work_groups") == L.work_groups(rc.ENTRY_PREFILL, B, H, D)
            assert _prefill_fp8(L, B, H, D) == rc.RC_OK
            assert stub("rc_stub_work_groups") == L.work_groups(rc.ENTRY_PREFILL, B, H, D, fp8=True)
        for splits in (1, 2, 5, 0, rc.SPLITS_TAIL, rc.SPLITS_BALANCED, rc.SPLITS_LAST_ROUND):
            need = L.workspace_bytes(B, H, D, splits)
            st = _step(L, B=B, H=H, D=D, ts=ts, splits=splits, ws=FAKE if need else None, wsb=need, lse=FAKE)
            assert st == rc.RC_OK, (kinds, lens, splits, rc.lib().rc_last_error().decode())
            if L.rows(rc.ROWS_LIVE):
                assert stub("rc_stub_work_groups") == L.work_groups(rc.ENTRY_STEP, B, H, D, splits), splits


@pytest.mark.parametrize("segs,mask,runs", [
    ([(0, 64), (1, 64), (2, 256)] + [(3, 128)] * 20, "paper", 1),      # the anchors before them are not cached
    ([(0, 64), (1, 64), (2, 256)] + [(3, 128)] * 20, "perref", 1),
    ([(3, 100), (0, 8), (3, 50), (2, 64), (3, 7)], "paper", 2),        # anchors between the references
    ([(3, 100), (0, 8), (3, 50), (2, 64), (3, 7)], "perref", 1),
    ([(3, 1), (0, 1), (3, 1), (2, 5), (0, 1), (3, 1)], "isolated", 3),
])
def test_copy_table_has_one_run_per_stretch_of_rows(segs, mask, runs):
    L = rc.Layout(segs, mask)
    assert _prefill(L) == rc.RC_OK and stub("rc_stub_copy_runs") == runs
    assert _prefill_fp8(L) == rc.RC_OK and stub("rc_stub_copy_runs") == runs


HEAD = [(0, 64), (1, 64), (2, 256)]


@pytest.mark.parametrize("refs,mask,B,H,D,heads", [
    ([128] * 10, "perref", 2, 24, 64, 0),         # 36 heads would fit on the idle CUs: 17 MB, short windows
    ([128] * 10, "perref", 2, 24, 128, 0),
    ([1024] * 3, "perref", 1, 40, 64, 0),         # 14 of 40
    ([1519] * 3, "perref", 1, 24, 128, 0),        # 13 of 24: 57 MB
    ([4096] * 8, "perref", 1, 24, 128, 0),        # 1 of 24: 403 MB, but windows of three tile times
    ([128] * 20, "paper", 1, 24, 64, 0),          # 8 of 24: long windows, 16 MB
    ([1519] * 3, "perref", 2, 24, 128, 0),        # 13 of 48: 114 MB, but windows of 24 in launches of one round
    ([1519] * 3, "perref", 3, 40, 128, 50),       # windows of 24, two rounds a launch
    ([2304], "perref", 3, 40, 64, 54),            # one round a launch, windows of 36, 73 MB
    ([4096] * 5, "perref", 1, 24, 128, 12),       # 252 MB, windows of 64
    ([4096] * 5, "perref", 1, 40, 128, 38),
    ([4096] * 3, "perref", 1, 24, 128, 24),       # all of them
    ([100] * 3, "perref", 1, 24, 64, 24),         # all, however small
])
def test_amax_work_groups_take_all_heads_or_many(refs, mask, B, H, D, heads):
    """The FP8 prefill's attention launch takes the amax of every head, or of
    some where that shortens the amax launch, or of none."""
    assert _prefill_fp8(rc.Layout(HEAD + [(3, n) for n in refs], mask), B, H, D) == rc.RC_OK
    assert stub("rc_stub_amax_heads") == heads


@pytest.mark.parametrize("M,N,K,ld", [(1, 128, 64, 128), (300, 384, 192, 4096), (257, 256, 1 << 22, 1 << 22)])
def test_linear_operands_reach_the_launch(M, N, K, ld):
    n0 = launches()
    assert rc.lib().rc_linear(M, N, K, FAKE, max(ld, K), FAKE, FAKE, max(ld, N), FAKE, max(ld, N), None) == rc.RC_OK
    assert launches() == n0 + 1


def _linear_tile(M, N, K):
    assert rc.lib().rc_linear(M, N, K, FAKE, K, FAKE, None, 0, FAKE, N, None) == rc.RC_OK
    return stub("rc_stub_linear_tile")


@pytest.mark.parametrize("M,N,K,tile", [
    # rounds of few slices, where a round's fixed part counts: the small tiles
    # measured 5 to 16% slower than the ones chosen
    (4665, 3456, 64, 1), (2700, 4224, 64, 1), (16350, 640, 64, 1), (299, 12032, 1024, 1), (1016, 8320, 64, 1),
    (264, 11776, 64, 1), (547, 7040, 1536, 1), (539, 13952, 2560, 2),
    # one round of each tile
    (4096, 4096, 3072, 0), (1536, 3072, 3072, 1), (300, 9216, 320, 2), (150, 9216, 832, 3), (16, 3072, 3072, 4),
    (1, 128, 64, 4),
    # more than one round of 256 x 256: the rest in 64, 128 or 256-row parts, or whole
    (256 * 33, 2048, 64, 5), (256 * 40, 2048, 64, 6), (256 * 44, 2048, 64, 7), (256 * 49, 2048, 64, 0),
    (256 * 64, 2048, 64, 0),
])
def test_projection_tile(M, N, K, tile):
    assert _linear_tile(M, N, K) == tile


def test_projection_tile_costs_least():
    """The rule on its own: the fewest nanoseconds in rounds of 256 work-groups,
    each with a fixed part and one per 64-wide k slice."""
    tiles = [(256, 256, 5500, 1475), (256, 128, 3700, 806), (128, 128, 3200, 473), (64, 128, 2500, 380),
             (64, 64, 1800, 223)]
    rng = random.Random(8)
    for _ in range(400):
        M, N, K = rng.randint(1, 1 << rng.randint(1, 15)), 128 * rng.randint(1, 110), 64 * rng.randint(1, 64)
        got = _linear_tile(M, N, K)
        cost = {i: -(-(-(-M // bm) * (N // bn)) // 256) * (f + s * (K // 64))
                for i, (bm, bn, f, s) in enumerate(tiles) if N % bn == 0}
        if got < 5:
            assert cost[got] == min(cost.values()), (M, N, K)
        else:
            rest = -(-M // 256) * (N // 256) % 256
            assert N % 256 == 0 and rest * (8, 4, 2)[got - 5] <= 256 and (got == 5 or rest * (8, 4, 2)[got - 6] > 256)
