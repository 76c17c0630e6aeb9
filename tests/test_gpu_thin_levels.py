"""BFS levels and push-relabel rounds that one workgroup runs from LDS lists,
and the cut's long rows, at the sizes where a list, a piece of a row or a
bitmap word ends: layered graphs whose levels have a given width and rows a
given length.  Heights against the oracle's, values and cuts exact."""
import numpy as np
import pytest

import oracle
import paper_2511_01235_amd as mf
from paper_2511_01235_amd import gen


def ring_layers(width, out, layers, seed):
    """s -> layers of `width` vertices -> t, vertex a to a .. a + out - 1 (mod
    width) of the next layer: rows of 2 * out slots between the layers."""
    rng = gen.rng_for(seed)
    a = np.arange(width)
    n = 2 + width * layers
    u, v = [np.zeros(width, np.int64)], [1 + a]
    for i in range(layers - 1):
        for d in range(min(out, width)):
            u.append(1 + i * width + a)
            v.append(1 + (i + 1) * width + (a + d) % width)
    u.append(1 + (layers - 1) * width + a)
    v.append(np.full(width, n - 1))
    u, v = np.concatenate(u), np.concatenate(v)
    c = rng.integers(1, 30, u.size)
    return gen.Graph(f"ring_{width}_{out}", n, u.astype(np.int32), v.astype(np.int32), c.astype(np.int32), 0, n - 1)


def fan(top, levels, seed):
    """s -> top vertices, each to two of a layer twice as wide, and so on; the
    last layer -> t: a round's list doubles from layer to layer."""
    rng = gen.rng_for(seed)
    u, v, c = [np.zeros(top, np.int64)], [1 + np.arange(top)], [np.full(top, 1 << (levels + 2))]
    first, width = 1, top
    for i in range(levels):
        a = np.arange(width)
        for d in (0, 1):
            u.append(first + a)
            v.append(first + width + 2 * a + d)
            c.append(rng.integers(1, (1 << (levels + 1 - i)) + 1, width))
        first, width = first + width, 2 * width
    n = first + width + 1
    u.append(first + np.arange(width))
    v.append(np.full(width, n - 1))
    c.append(rng.integers(1, 4, width))
    u, v, c = np.concatenate(u), np.concatenate(v), np.concatenate(c)
    return gen.Graph(f"fan_{top}_{levels}", n, u.astype(np.int32), v.astype(np.int32), c.astype(np.int32), 0, n - 1)


# rows of 4, 32, 34 and 40 slots: one piece, eight, nine and ten; 2047 to 2049
# and 4095 to 4097 pieces of a level; 8184 to 8200 slots; s and t rows of 255 to
# 257 slots (the cut's long ones from 257 on); one vertex wide, and a wave wide
GRAPHS = [("ring", 1, 1, 40), ("ring", 64, 2, 9), ("ring", 40, 16, 5), ("ring", 40, 17, 5), ("ring", 33, 20, 4),
          ("ring", 255, 2, 4), ("ring", 256, 2, 4), ("ring", 257, 2, 4), ("ring", 1023, 4, 4), ("ring", 1024, 4, 4),
          ("ring", 1025, 4, 4), ("ring", 2047, 2, 3), ("ring", 2049, 2, 3), ("ring", 4095, 1, 3), ("ring", 4096, 1, 3),
          ("ring", 4097, 1, 3), ("fan", 500, 4), ("fan", 2048, 2)]


def make(spec, seed):
    return ring_layers(*spec[1:], seed) if spec[0] == "ring" else fan(*spec[1:], seed)


@pytest.fixture(scope="module")
def device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"


@pytest.mark.gpu
@pytest.mark.parametrize("spec", GRAPHS, ids=lambda s: "_".join(map(str, s)))
def test_thin_levels_and_rounds(device, spec):
    g = make(spec, 63000)
    h_want, _ = oracle.DynOracle(g.n, g.src, g.dst, g.cap, g.s, g.t).initial_labels()
    o = oracle.DynOracle(g.n, g.src, g.dst, g.cap, g.s, g.t)
    want = o.static()
    batch = gen.BatchStream(g, 63100, inc_max=20, new_cap_max=20).next_batch(max(1, g.m // 50))
    after = o.apply(*batch)
    print(f"[test] thin levels {g.name} n={g.n}", flush=True)
    # one workgroup as far as it goes, and the defaults
    for opt in (dict(bfs_narrow_slots=8192, round_narrow=4096), {}):
        with mf.MaxFlowGraph(g.n, g.src, g.dst, g.cap, g.s, g.t, **opt) as G:
            assert np.array_equal(G.initial_labels()[0], h_want)
        with mf.MaxFlowGraph(g.n, g.src, g.dst, g.cap, g.s, g.t, **opt) as G:
            assert G.maxflow() == want
            side, cut = G.min_cut()
            assert cut == want and side[g.s] == 1 and side[g.t] == 0
            assert oracle.cert_check(g.n, g.src, g.dst, g.cap, g.s, g.t, None, side, want)[0] == 0
            assert G.apply_batch(*batch) == after
            assert G.min_cut()[1] == after


def funnel(width, layers, wide, seed):
    """s -> layers of `width` vertices, one to one -> `wide` vertices -> t: a
    BFS from t meets the wide layer first and the thin ones behind it."""
    rng = gen.rng_for(seed)
    a = np.arange(width)
    last = 1 + (layers - 1) * width
    first_wide = 1 + layers * width
    n = first_wide + wide + 1
    w = first_wide + np.arange(wide)
    u = [np.zeros(width, np.int64)] + [1 + i * width + a for i in range(layers - 1)] + [last + np.arange(wide) % width, w]
    v = [1 + a] + [1 + (i + 1) * width + a for i in range(layers - 1)] + [w, np.full(wide, n - 1)]
    u, v = np.concatenate(u), np.concatenate(v)
    c = rng.integers(1, 30, u.size)
    return gen.Graph(f"funnel_{width}_{wide}", n, u.astype(np.int32), v.astype(np.int32), c.astype(np.int32), 0, n - 1)


# Levels of 3600 rows of two slots come back from the multi-block levels: up to
# 8192 slots, but more pieces than one workgroup may have to hold (4096).  And
# levels of 20,000 slots, between what one workgroup holds and the limits asked
# for.  Both are the mid-size levels' (bfs_alpha: no bottom-up level takes them).
@pytest.mark.gpu
@pytest.mark.parametrize("make_graph,narrow,launches", [
    (lambda: funnel(3600, 40, 40_000, 63200), 8192, 7), (lambda: ring_layers(5000, 2, 12, 63300), 65536, 0)])
def test_levels_one_workgroup_refuses_run_mid_size(device, make_graph, narrow, launches):
    g = make_graph()
    h_want, _ = oracle.DynOracle(g.n, g.src, g.dst, g.cap, g.s, g.t).initial_labels()
    print(f"[test] refused levels {g.name} n={g.n}", flush=True)
    with mf.MaxFlowGraph(g.n, g.src, g.dst, g.cap, g.s, g.t, bfs_narrow_slots=narrow, bfs_alpha=-1) as G:
        for _ in range(2):                       # the second starts from what the first left
            G.profile(0xFF)                      # (counts afresh)
            assert np.array_equal(G.initial_labels()[0], h_want)
            assert G.stats()["kernel_launches"]["global_relabel"] <= launches
        assert G.maxflow() == oracle.DynOracle(g.n, g.src, g.dst, g.cap, g.s, g.t).static()


@pytest.mark.gpu
def test_bitmap_that_does_not_fit_in_lds_is_left_out(device):
    """bfs_lds_bitmap at a size where the device refuses that much LDS beside
    the level kernel's own: the graph loads, without the copy."""
    n, m = 1_160_000, 6000
    rng = gen.rng_for(63400)
    u = rng.integers(0, n, m)
    v = (u + 1 + rng.integers(0, n - 1, m)) % n
    u[:2], v[:2] = (0, 7), (7, n - 1)
    c = rng.integers(1, 50, m)
    e = [x.astype(np.int32) for x in (u, v, c)]
    want = oracle.DynOracle(n, *e, 0, n - 1).static()
    with mf.MaxFlowGraph(n, *e, 0, n - 1, bfs_lds_bitmap=1) as G:
        assert want > 0 and G.maxflow() == want


@pytest.mark.gpu
def test_cut_of_rows_that_grow_past_the_long_limit(device):
    """Rows of 256 slots at the load and at the first cut, of more after a
    batch of inserts, and after a batch that only changes capacities."""
    width = 256
    g = ring_layers(width, 1, 3, 63500)          # s: one slot per vertex of the first layer
    u = np.zeros(9, np.int32)
    v = (1 + width + np.arange(9)).astype(np.int32)
    c = np.full(9, 25, np.int32)
    o = oracle.DynOracle(g.n, g.src, g.dst, g.cap, g.s, g.t)
    with mf.MaxFlowGraph(g.n, g.src, g.dst, g.cap, g.s, g.t) as G:
        want = o.static()
        assert G.maxflow() == want and G.min_cut()[1] == want
        for batch in ((u, v, c), (u, v, c - 20), (u[:0], v[:0], c[:0])):
            want = o.apply(*batch)
            assert G.apply_batch(*batch) == want
            side, cut = G.min_cut()
            assert cut == want and side[g.s] == 1 and side[g.t] == 0
