"""Triangles counted per edge in 32 bits, widened in place to the caller's
64-bit words, and the edges' counts summed by time: sizes at the edges of the
widening steps (2048 counts in the last one, halves before it) and of the
packing tiles (4096 elements, 64 per round).  All values are integers: the
comparison is exact, with closed forms on a K_4 core joined to R vertices."""
import numpy as np
import pytest

import oracle
from paper_2107_12330_amd import tripoll as tp
from tests.test_gpu_work_tiles import CORE, dev, fan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    return torch


# m = 4 R + 6 edges; R = 0: the core alone
@pytest.mark.parametrize("R", [0, 1, 509, 510, 511, 512, 1021, 1022, 1023, 2049, 16383, 16385])
def test_edge_counts_widened_in_place(T, R):
    print("fan", R, flush=True)
    g = fan(R)
    s = T.cuda.current_stream().cuda_stream
    with tp.build_graph(*dev(T, g), stream=s) as G:
        m = G.stats()["n_edges"]
        assert m == 4 * R + 6
        guard = 64
        v = T.full((g[0] + guard,), -7, dtype=T.int64, device="cuda")
        e = T.full((m + guard,), -7, dtype=T.int64, device="cuda")
        assert tp.tripoll_participation(G.handle, tp.make_spec(), v.data_ptr(), e.data_ptr(), s) == 6 * R + 4
        T.cuda.synchronize()
        ev, vv = e.cpu().numpy(), v.cpu().numpy()
        assert (ev[m:] == -7).all() and (vv[g[0]:] == -7).all()
        x = tp.export(G)
        rows = np.repeat(np.arange(g[0]), np.diff(x["rowptr"].astype(np.int64)))
        core = (x["rank_to_id"][rows] < CORE) & (x["rank_to_id"][x["col"]] < CORE)
        assert np.array_equal(ev[:m], np.where(core, R + 2, 3))
        v2 = T.zeros(g[0], dtype=T.int64, device="cuda")
        tp.tripoll_participation(G.handle, tp.make_spec(), v2.data_ptr(), 0, s)  # counters of the call's own
        T.cuda.synchronize()
        assert np.array_equal(v2.cpu().numpy(), vv[:g[0]])


@pytest.mark.parametrize("R", [0, 1, 15, 16, 1022, 1023, 5000])
@pytest.mark.parametrize("times", ["equal", "index", "pairs"])
def test_max_edge_runs(T, R, times):
    """Runs of equal times within a round of 64, across rounds, waves and tiles."""
    print("fan", R, times, flush=True)
    n, src, dst, _, _ = fan(R)
    k = np.arange(len(src), dtype=np.uint32)
    ts = {"equal": np.full(len(src), 0xffffffff, np.uint32), "index": k, "pairs": k // 37}[times]
    vlab = np.concatenate([np.arange(CORE), np.full(R, CORE)]).astype(np.uint8)
    ref = oracle.max_edge_counts(n, src, dst, ts, vlab, n_labels=5)
    assert int(ref[1].sum()) == 6 * R + 4
    s = T.cuda.current_stream().cuda_stream
    d = dev(T, (n, src, dst, ts, vlab))
    with tp.build_graph(*d, stream=s) as G:
        got = tp.max_edge_counts(G, T, stream=s, n_labels=5)
        assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])
        # too small a capacity: the number needed, and the buffers as they were
        need = len(ref[0])
        a = T.full((max(need - 1, 1),), 7, dtype=T.int32, device="cuda")
        b = T.full((max(need - 1, 1),), 7, dtype=T.int64, device="cuda")
        with pytest.raises(tp.TripollError) as err:
            tp.tripoll_max_edge_counts(G.handle, tp.make_spec(n_labels=5), a.data_ptr(), b.data_ptr(), need - 1, s)
        assert err.value.status == tp.TP_ERR_INVALID and err.value.n_values == need
        T.cuda.synchronize()
        assert (a == 7).all().item() and (b == 7).all().item()
