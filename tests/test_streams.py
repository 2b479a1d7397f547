"""Calls on a stream of the caller's choice (``stream=``): what a call
allocates for itself stays allocated until that stream is done with it.

On the CPU every entry runs with torch's stream context, the allocations and
the launches recorded; on the GPU a call is queued behind a delay, its
workspace dropped on return, and the memory that the current stream can then
get is overwritten before the call's kernels run."""
import contextlib
import types

import pytest
import torch

import paper_2608_21229_amd as rc
from paper_2608_21229_amd import binding as rcb

SEGS = [(0, 8), (1, 40), (2, 100), (3, 700), (3, 300)]
B, H, D = 1, 2, 64


def rows(which):
    return rc.Layout(SEGS, "perref").rows(which)


def entries(dev):
    """name -> call(stream) that allocates everything it may."""
    g = torch.Generator(device=dev)
    g.manual_seed(5)

    def rn(*s):
        return torch.randn(s, generator=g, device=dev).to(torch.bfloat16)

    def qkv(n):
        return tuple(rn(B, n, H, D) for _ in range(3))

    L, Ld = rc.Layout(SEGS, "perref"), rc.Layout([(1, 512), (2, 4096), (3, 4096)], "dense")
    st, lv, nc = qkv(rows(rc.ROWS_STATIC)), qkv(rows(rc.ROWS_LIVE)), rows(rc.ROWS_CACHED)
    kc, vc = rn(B, H, nc, D), rn(B, H, nc, D)
    k8, v8 = (torch.randint(0, 120, (B, H, nc, D), generator=g, device=dev).to(torch.uint8) for _ in range(2))
    sc = torch.full((B, H, 2), 2.0 ** -4, device=dev)
    C = H * D
    wq, wo = ([rn(n, C) * C ** -0.5 for _ in range(2)] for n in (3 * C, C))
    ch = {c: rc.Chain(L, wq, wo, H, D, cache=c) for c in ("bf16", "fp8")}
    hs, hl, ha = (rn(B, rows(n), C) for n in (rc.ROWS_STATIC, rc.ROWS_LIVE, rc.ROWS_ALL))
    caches = {"bf16": [(kc, vc)] * 2, "fp8": [(k8, v8, sc)] * 2}
    Hd = 18  # 18 heads x 17 query tiles: more than one round, so the recompute takes a workspace
    full = tuple(rn(1, Ld.rows(rc.ROWS_ALL), Hd, D) for _ in range(3))
    assert Ld.full_workspace_bytes(1, Hd, D) > 0 and L.workspace_bytes(B, H, D, 3) > 0
    a = rn(70, 128)
    collected = []

    def flat(x):
        return [t for e in x for t in (e if isinstance(e, tuple) else (e,)) if t is not None]

    def collect_step(s):
        collected.clear()
        return [ch["bf16"].step(hl, caches["bf16"], splits=3, collect=collected, stream=s)] + collected

    return {
        "prefill": lambda s: flat(rc.ref_kv_prefill(L, *st, want_lse=True, stream=s)),
        "prefill_fp8": lambda s: flat(rc.ref_kv_prefill_fp8(L, *st, want_lse=True, stream=s)),
        "step": lambda s: flat(rc.step_masked_attention(L, *lv, kc, vc, splits=3, want_lse=True, stream=s)),
        "step_fp8": lambda s: flat(rc.step_masked_attention_fp8(L, *lv, k8, v8, sc, splits=3, want_lse=True, stream=s)),
        "full": lambda s: flat(rc.full_attention(Ld, *full, want_lse=True, stream=s)),
        "linear": lambda s: [rc.linear(a, wq[0], stream=s)],
        "chain_prefill": lambda s: flat(ch["bf16"].prefill(hs, stream=s)),
        "chain_prefill_fp8": lambda s: flat(ch["fp8"].prefill(hs, stream=s)),
        "chain_step": collect_step,
        "chain_step_fp8": lambda s: [ch["fp8"].step(hl, caches["fp8"], splits=3, stream=s)],
        "chain_full": lambda s: [ch["bf16"].full(ha, stream=s)],
    }


NAMES = ["prefill", "prefill_fp8", "step", "step_fp8", "full", "linear", "chain_prefill", "chain_prefill_fp8",
         "chain_step", "chain_step_fp8", "chain_full"]


@pytest.mark.parametrize("own", [True, False])
@pytest.mark.parametrize("name", NAMES)
def test_allocations_follow_the_stream(name, own, monkeypatch):
    """With a stream every allocation is made on it and every returned tensor
    marked as used on the stream that was current; without one neither."""
    call = entries("cpu")[name]
    current, made, marked = ["main"], [], []
    empty, clone = torch.empty, torch.Tensor.clone

    @contextlib.contextmanager
    def fake_stream(s):
        current.append(s)
        yield
        current.pop()

    def fake_empty(*a, **k):
        t = empty(*a, **k)
        made.append((t, current[-1]))
        return t

    def fake_clone(t):
        c = clone(t)
        made.append((c, current[-1]))
        return c

    class Side:
        cuda_stream = 77

    launched = []
    monkeypatch.setattr(torch.cuda, "Stream", Side)
    monkeypatch.setattr(torch.cuda, "stream", fake_stream)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda dev=None: current[-1])
    monkeypatch.setattr(torch, "empty", fake_empty)
    monkeypatch.setattr(torch.Tensor, "clone", fake_clone)
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: marked.append((t.data_ptr(), s)))
    monkeypatch.setattr(rcb, "_inputs", lambda q, k, v: q.device)
    monkeypatch.setattr(rcb, "_rows_view", lambda t, what: t.stride(0))
    monkeypatch.setattr(rcb, "_call", lambda fn, dev, stream, *a: launched.append(stream))
    side = Side() if own else None
    out = call(side)
    assert made and launched and all(s is side for s in launched)
    assert [s for _, s in made] == [side if own else "main"] * len(made)
    ours = {t.data_ptr() for t, _ in made}
    for t in out:
        assert t.data_ptr() in ours
        assert ((t.data_ptr(), "main") in marked) == own


def test_any_object_with_a_stream_handle(monkeypatch):
    """A stream need not be torch's: its handle is enough."""
    seen = []

    class Torch:
        pass

    monkeypatch.setattr(torch.cuda, "Stream", Torch)
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda h, device: ("external", h, str(device)))
    monkeypatch.setattr(torch.cuda, "stream", lambda s: seen.append(s))
    t = Torch()
    rcb._on(t, torch.device("cpu"))
    rcb._on(types.SimpleNamespace(cuda_stream=41), torch.device("cpu"))
    assert seen == [t, ("external", 41, "cpu")]


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_dropped_workspace_is_not_reused(name):
    """The same bits as on the current stream, with the call's own memory
    dropped before its kernels start and everything that the current stream
    can allocate then overwritten."""
    call = entries("cuda")[name]
    want = [t.clone() for t in call(None)]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    call(side)  # the side stream's pool holds what the call needs
    torch.cuda.synchronize()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)  # about 10 ms
    got = call(side)
    print(f"[case] {name} on a side stream", flush=True)
    junk = [torch.empty(n, dtype=torch.uint8, device="cuda").fill_(0xff)
            for n in (1 << p for p in range(10, 27)) for _ in range(4)]
    torch.cuda.synchronize()
    del junk
    assert len(got) == len(want)
    for a, b in zip(got, want):
        assert torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))
