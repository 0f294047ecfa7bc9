"""Re-planning a live graph with every device allocation failing in turn: the
call returns TP_ERR_OOM, the graph keeps its plan and its statistics, the
library holds what it held before, and the graph surveys as before.  The same
for the tuner, participation and the exact counting set."""
import math

import numpy as np
import pytest

import synth
from paper_2107_12330_amd import tripoll as tp
from tests.test_gpu_faults import fail_each_allocation

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    yield torch
    tp.tripoll_fail_alloc_after(0)


def complete(T, n):
    iu = np.triu_indices(n, 1)
    src, dst = (T.from_numpy(x.astype(np.uint32)).cuda() for x in iu)
    lab = T.from_numpy((np.arange(n) % 3).astype(np.uint8)).cuda()
    ts = T.from_numpy((np.arange(len(iu[0])) % 1000).astype(np.uint32)).cuda()
    return n, src, dst, ts, lab


# K_60: tiny and small targets; K_3400: every class, the huge one in pieces
@pytest.mark.parametrize("n", [60, 3400])
@pytest.mark.parametrize("caps", [(16,) * 4, (65536,) * 4])
def test_failed_set_plan_keeps_the_plan(T, n, caps):
    print("K_%d" % n, caps, flush=True)
    s = T.cuda.current_stream().cuda_stream
    with tp.build_graph(*complete(T, n), stream=s) as G:
        plan, st = tp.plan_dict(tp.tripoll_get_plan(G.handle)), G.stats()
        first = tp.survey(G, stream=s, outputs=("count", "close_hist"))
        assert first["triangles"] == math.comb(n, 3)
        seen = []

        def replan():
            # from the host, before anything is launched on the graph
            assert tp.plan_dict(tp.tripoll_get_plan(G.handle)) == plan
            assert G.stats() == st
            seen.append(1)
            tp.tripoll_set_plan(G.handle, tp.make_plan((0,) * 4, caps), s)

        calls, _ = fail_each_allocation(replan)
        assert calls == len(seen) - 1 >= 5
        assert tp.plan_dict(tp.tripoll_get_plan(G.handle))["tile_records"] == list(caps)
        got = tp.survey(G, stream=s, outputs=("count", "close_hist"))
        assert got["triangles"] == math.comb(n, 3) and np.array_equal(got["close_hist"], first["close_hist"])
        # and a survey right after a failure at each of the last allocations
        # (the lists of tiles)
        tp.tripoll_set_plan(G.handle, tp.make_plan((0,) * 4, (1024,) * 4), s)
        for k in range(max(1, calls - 8), calls + 1):
            tp.tripoll_fail_alloc_after(k)
            with pytest.raises(tp.TripollError) as e:
                tp.tripoll_set_plan(G.handle, tp.make_plan((0,) * 4, caps), s)
            assert e.value.status == tp.TP_ERR_OOM
            assert tp.plan_dict(tp.tripoll_get_plan(G.handle))["tile_records"] == [1024] * 4
            got = tp.survey(G, stream=s, outputs=("count", "close_hist"))
            assert got["triangles"] == math.comb(n, 3) and np.array_equal(got["close_hist"], first["close_hist"])


def test_failed_tune_participation_and_counting_set(T):
    s = T.cuda.current_stream().cuda_stream
    g = synth.generate(synth.GraphSpec("rmat", 10, 8, synth.MASTER_SEED + 811, ("uniform", 20), ("uniform", 4)))
    dev = [T.from_numpy(g[k]).cuda() for k in ("src", "dst", "ts", "vlab")]
    with tp.build_graph(g["n"], *dev, stream=s) as G:
        st, plan = G.stats(), tp.plan_dict(tp.tripoll_get_plan(G.handle))
        spec = tp.make_spec(outputs=("count", "close_hist"))
        first = tp.survey(G, stream=s, outputs=("count", "close_hist"))

        # (the blocks that hold the tiles may be other ones after a re-plan: the
        # bytes held are not compared here)
        sizes = {k: v for k, v in st.items() if k != "device_bytes"}
        for n in range(1, 400):
            tp.tripoll_fail_alloc_after(n)
            try:
                r = tp.tripoll_tune(G.handle, spec, s)
            except tp.TripollError as e:
                assert e.status == tp.TP_ERR_OOM and "injected" in str(e), n
                # a tuning run that failed on the way has put the plan back
                assert tp.plan_dict(tp.tripoll_get_plan(G.handle)) == plan, n
                assert {k: v for k, v in G.stats().items() if k != "device_bytes"} == sizes, n
                continue
            break
        tp.tripoll_fail_alloc_after(0)
        assert n > 20
        assert tp.plan_dict(tp.tripoll_get_plan(G.handle)) == tp.tune_dict(r)["chosen"]
        got = tp.survey(G, stream=s, outputs=("count", "close_hist"))
        assert got["triangles"] == first["triangles"] and np.array_equal(got["close_hist"], first["close_hist"])
        m = st["n_edges"]
        v = T.zeros(g["n"], dtype=T.int64, device="cuda")
        e = T.zeros(m, dtype=T.int64, device="cuda")
        for edges in (e.data_ptr(), 0):
            calls, t = fail_each_allocation(
                lambda: tp.tripoll_participation(G.handle, tp.make_spec(), v.data_ptr(), edges, s))
            assert calls >= 2 and t == first["triangles"]
            assert int(v.sum()) == 3 * first["triangles"]
        assert int(e.sum()) == 3 * first["triangles"]
        values = T.zeros(m, dtype=T.int32, device="cuda")
        counts = T.zeros(m, dtype=T.int64, device="cuda")
        calls, k = fail_each_allocation(
            lambda: tp.tripoll_max_edge_counts(G.handle, tp.make_spec(), values.data_ptr(), counts.data_ptr(), m, s))
        assert calls >= 6 and k > 0
        full = tp.max_edge_counts(G, T, stream=s)
        assert np.array_equal(values[:k].cpu().numpy().view(np.uint32), full[0])
        assert np.array_equal(counts[:k].cpu().numpy().view(np.uint64), full[1])
