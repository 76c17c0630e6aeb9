"""The Bi-CSR built on the device (graphs of at least 4096 edges) against a
plain numpy statement of what the loader makes: merged pairs, one slot per
direction of every adjacent pair, row slack, pair links, and the same errors
as the host builder, at the edges of its tiles and key widths."""
import numpy as np
import pytest

import oracle
import paper_2511_01235_amd as mf
from paper_2511_01235_amd import gen

INT_MAX = 2**31 - 1


@pytest.fixture(scope="module")
def device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"


def _edges(kind, n, m, seed):
    rng = gen.rng_for(seed)
    if kind == "random":
        u, v = rng.integers(0, n, m), rng.integers(0, n, m)
    elif kind == "star":        # one row with an entry for every other vertex
        u, v = np.zeros(m, np.int64), 1 + np.arange(m) % (n - 1)
        flip = rng.random(m) < 0.3
        u[flip], v[flip] = v[flip], u[flip].copy()
    elif kind == "few":         # a handful of pairs, repeated; most vertices have no edge
        u, v = rng.integers(0, 3, m), rng.integers(n - 3, n, m)
    same = u == v
    v[same] = (v[same] + 1) % n
    return u.astype(np.int32), v.astype(np.int32), rng.integers(0, 50, m).astype(np.int32)


def _expect(n, u, v, c):
    key, inv = np.unique(u.astype(np.int64) * n + v, return_inverse=True)
    cap = np.bincount(inv, weights=c).astype(np.int64)
    slots = np.unique(np.concatenate([key, (key % n) * n + key // n]))
    length = np.bincount(slots // n, minlength=n)
    slack = np.maximum(8, (length * 12 + 99) // 100)
    live = cap > 0
    return key[live], cap[live], slots.size, int((length + slack).sum()), int(live.sum())


@pytest.mark.gpu
@pytest.mark.parametrize("kind,n,m", [
    ("random", 300, 4095), ("random", 300, 4096), ("random", 300, 4097), ("random", 300, 8193),
    ("random", 4096, 10240), ("random", 4097, 10241),
    ("random", 65536, 30000), ("random", 65537, 30001), ("random", 1_000_003, 40_000),
    ("star", 70_001, 90_000), ("few", 5000, 8192), ("few", 6, 9000), ("random", 2, 8200)])
def test_device_build(device, kind, n, m):
    u, v, c = _edges(kind, n, m, 900 + n + m)
    print(f"[test] device build {kind} n={n} m={m}", flush=True)
    key, cap, slots, capacity, live = _expect(n, u, v, c)
    s, t = 0, n - 1
    with mf.MaxFlowGraph(n, u, v, c, s, t) as G:
        st = G.stats()
        assert (st["slots"], st["slot_capacity"]) == (slots, capacity)
        assert st["kernel_cycles"] == max(1, (live + n // 2) // n)
        eu, ev, ec = G.get_edges()
        assert np.array_equal(eu.astype(np.int64) * n + ev, key) and np.array_equal(ec, cap)
        assert {k: x for k, x in G.invariants().items() if x} == {}
        o = oracle.DynOracle(n, u, v, c, s, t)
        assert G.maxflow() == o.static()
        # every pair is found again where the rows say it is, and a new one beside them
        up = gen.random_batch(n, 500, 60, 7 + n, np.stack([u, v], 1))
        assert G.apply_batch(*up) == o.apply(*up)
        inv = G.invariants()
        assert not any(inv[k] for k in ("negative_residuals", "pair_sums", "pair_links", "excess_mismatches"))


def _bad(at, **edge):
    u, v, c = _edges("random", 1000, 9000, 1)
    for name, x in edge.items():
        {"u": u, "v": v, "c": c}[name][at] = x
    return u, v, c


BAD = [(0, dict(u=-1)), (4500, dict(v=1000)), (8999, dict(c=-1)), (8999, dict(u=5, v=5)), (17, dict(u=INT_MAX))]


@pytest.mark.parametrize("at,edge", BAD)
def test_large_load_rejects_invalid_edges(at, edge):
    """Also without a device: the edges are validated before it is missed."""
    with pytest.raises(mf.MFError) as ei:
        mf.MaxFlowGraph(1000, *_bad(at, **edge), 0, 999)
    assert ei.value.status == mf.MF_ERR_INVALID


@pytest.mark.gpu
@pytest.mark.parametrize("at,edge", BAD)
def test_device_build_rejects_invalid_edges(device, at, edge):
    test_large_load_rejects_invalid_edges(at, edge)


@pytest.mark.gpu
def test_device_build_capacity_sums(device):
    """A pair's two merged capacities may sum to INT32_MAX and not above."""
    u, v, c = _edges("random", 1000, 9000, 3)
    keep = ~(((u == 7) & (v == 9)) | ((u == 9) & (v == 7)))
    u, v, c = (np.concatenate([x[keep], e]).astype(np.int32) for x, e in
               ((u, [7, 9, 7]), (v, [9, 7, 9]), (c, [INT_MAX - 100, 60, 40])))
    with mf.MaxFlowGraph(1000, u, v, c, 0, 999) as G:
        eu, ev, ec = G.get_edges()
        assert ec[(eu == 7) & (ev == 9)] == INT_MAX - 60 and ec[(eu == 9) & (ev == 7)] == 60
    c[-1] = 41
    with pytest.raises(mf.MFError) as ei:
        mf.MaxFlowGraph(1000, u, v, c, 0, 999)
    assert ei.value.status == mf.MF_ERR_OVERFLOW


@pytest.mark.gpu
@pytest.mark.parametrize("hook", [False, True])
def test_load_where_scratch_and_slots_do_not_fit_together(device, hook):
    """The device builder needs 76 bytes per edge beside the slot arrays.  With
    room for either but not for both, the graph is built on the host instead,
    also where the handle's memory comes from a caller's allocator."""
    import torch
    opt = dict(allocator=mf.TorchAllocator(device=0, stream=torch.cuda.current_stream())) if hook else {}
    n, m, left = 500_000, 4_000_000, 480 << 20   # scratch 320 MB, slot arrays 240 MB, the whole handle 370 MB
    u, v, c = _edges("random", n, m, 4)
    _, _, slots, capacity, _ = _expect(n, u, v, c)
    with mf.MaxFlowGraph(n, u, v, c, 0, n - 1) as G:
        want = G.maxflow()
    torch.cuda.empty_cache()
    print(f"[test] load beside {left >> 20} MB of free memory", flush=True)
    held = []
    try:
        while torch.cuda.mem_get_info()[0] > left + (20 << 20):
            held.append(torch.empty(torch.cuda.mem_get_info()[0] - left, dtype=torch.uint8, device="cuda"))
        with mf.MaxFlowGraph(n, u, v, c, 0, n - 1, **opt) as G:
            st = G.stats()
            assert (st["slots"], st["slot_capacity"]) == (slots, capacity)
            held.clear()
            torch.cuda.empty_cache()
            assert G.maxflow() == want
    finally:
        held.clear()
        torch.cuda.empty_cache()


@pytest.mark.gpu
def test_load_waits_for_its_own_stream_only(device):
    """A load returns while another stream's work still runs."""
    import time
    import torch
    n, m = 2000, 20_000
    u, v, c = _edges("random", n, m, 5)
    mf.MaxFlowGraph(n, u, v, c, 0, n - 1).close()
    beside = []
    # two streams may share one of the hardware's queues, where a load waits
    # for whatever is ahead of it: a few streams are tried
    for attempt in range(6):
        other, ev = torch.cuda.Stream(), torch.cuda.Event()
        torch.cuda.synchronize()
        with torch.cuda.stream(other):
            torch.cuda._sleep(300_000_000)
            ev.record()
        t = time.perf_counter()
        G = mf.MaxFlowGraph(n, u, v, c, 0, n - 1)
        beside.append(not ev.query())
        print(f"[test] load beside a busy stream {1e3 * (time.perf_counter() - t):.1f} ms, beside it: {beside[-1]}",
              flush=True)
        torch.cuda.synchronize()
        G.close()
        if beside[-1]:
            break
    assert any(beside)


@pytest.mark.gpu
@pytest.mark.parametrize("what,status", [("invalid", mf.MF_ERR_INVALID), ("pair sum", mf.MF_ERR_OVERFLOW),
                                         ("good", mf.MF_ERR_OUT_OF_MEMORY)])
def test_edges_decide_the_error_before_memory_does(device, what, status):
    u, v, c = _bad(4500, c=-1) if what == "invalid" else _edges("random", 1000, 9000, 3)
    if what == "pair sum":
        u[10:12], v[10:12], c[10:12] = (7, 9), (9, 7), INT_MAX

    class Refuses:
        alloc_fn = mf.ALLOC_FN(lambda nbytes, ctx: None)
        free_fn = mf.FREE_FN(lambda ptr, ctx: None)

    with pytest.raises(mf.MFError) as ei:
        mf.MaxFlowGraph(1000, u, v, c, 0, 999, allocator=Refuses, device=0)
    assert ei.value.status == status
