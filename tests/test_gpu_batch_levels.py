"""Batched solve, bottom-up levels whose rows find their parent past the slots
a single thread checks: such rows go through the workgroup's list of deferred
rows, which every wave has to see whole."""
import numpy as np
import pytest

import oracle
import paper_2511_01235_amd as mf
from paper_2511_01235_amd import gen


def deferred_rows_graph(rows, seed):
    """s -> B -> A -> t with `rows` vertices B.  A row of B starts with 33 to
    70 slots to other vertices of B and ends with 12 to A (the higher ids), so
    the level that labels B from A looks through more than 32 slots first."""
    rng = gen.rng_for(seed)
    na = max(rows // 3, 16)
    n = 2 + rows + na
    e = []
    for b in range(1, rows + 1):
        e += [(0, b, int(rng.integers(1, 20)))]
        others = rng.choice(rows, min(rows - 1, int(rng.integers(33, 71))), replace=False) + 1
        e += [(b, int(x), int(rng.integers(1, 5))) for x in others if x != b]
        e += [(b, rows + 1 + int(x), int(rng.integers(0, 4))) for x in rng.choice(na, 12, replace=False)]
    e += [(rows + 1 + a, n - 1, int(rng.integers(1, 60))) for a in range(na)]
    u, v, c = np.array(e, np.int64).T
    return gen.Graph(f"deferred_{rows}", n, u.astype(np.int32), v.astype(np.int32), c.astype(np.int32), 0, n - 1)


@pytest.fixture(scope="module")
def device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"


@pytest.mark.gpu
@pytest.mark.parametrize("block", [256, 512, 1024])
def test_batched_bottom_up_deferred_rows(device, block):
    # rows below, at and above a workgroup's threads and a wave's lanes
    graphs = [deferred_rows_graph(r, 61000 + r) for r in (63, 255, 257, 700, 1024, 1025, 2100)]
    oracles = [oracle.DynOracle(g.n, g.src, g.dst, g.cap, g.s, g.t) for g in graphs]
    want = [o.static() for o in oracles]
    streams = [gen.BatchStream(g, 61100 + g.n, inc_max=10, new_cap_max=20) for g in graphs]
    print(f"[test] batched deferred rows, {block} threads", flush=True)
    with mf.MaxFlowBatch(graphs, batch_block=block) as B:
        assert B.maxflow().tolist() == want
        batches = [st.next_batch(max(1, g.m // 50)) for g, st in zip(graphs, streams)]
        assert B.apply(batches).tolist() == [o.apply(*b) for o, b in zip(oracles, batches)]


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [257, 700, 1500])
def test_rows_pushed_to_while_they_push(device, rows):
    """B's vertices push to one another as well as to A: what the lanes of a
    row push together is what leaves its vertex, whatever arrives meanwhile."""
    g = deferred_rows_graph(rows, 61000 + rows)
    o = oracle.DynOracle(g.n, g.src, g.dst, g.cap, g.s, g.t)
    st = gen.BatchStream(g, 61200 + rows, inc_max=10, new_cap_max=20)
    print(f"[test] rows pushed to meanwhile, {rows} rows", flush=True)
    with mf.MaxFlowGraph(g.n, g.src, g.dst, g.cap, g.s, g.t) as G:
        assert G.maxflow() == o.static()
        for _ in range(3):
            batch = st.next_batch(max(1, g.m // 20))
            assert G.apply_batch(*batch) == o.apply(*batch)
        inv = G.invariants()
        assert not any(inv[k] for k in ("negative_residuals", "pair_sums", "pair_links", "excess_mismatches"))
