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
