"""The exact counting set of Algorithm 3 on huge targets, whose tiles hold a
piece of Adj+(q) and records cut to it: against the oracle value by value,
filtered and not, by tables and by search, and a complete graph's closed form."""
from math import comb

import numpy as np
import pytest

import oracle
from paper_2107_12330_amd import tripoll as tp
from tests import graphs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    return torch


def test_random_dense_pieces(T):
    n, src, dst, ts, vlab = graphs.huge_targets(929)
    s = T.cuda.current_stream().cuda_stream
    dev = [T.from_numpy(x).cuda() for x in (src, dst, ts, vlab)]
    with tp.build_graph(n, *dev, stream=s) as G:
        assert G.stats()["dplus_max"] > 3276 and G.stats()["class_tiles"][3] > 0
        for kw in (dict(), dict(window=(1 << 18, 3 << 20)), dict(label_mask={7, 11, 13, 16, 22, 25, 31})):
            print(kw, flush=True)
            ref = oracle.max_edge_counts(n, src, dst, ts, vlab, n_labels=5, **kw)
            assert len(ref[0])
            for strategy in (tp.TP_STRAT_AUTO, tp.TP_STRAT_GLOBAL_SEARCH, tp.TP_STRAT_TABLE_STRESS):
                got = tp.max_edge_counts(G, T, stream=s, n_labels=5, strategy=strategy, **kw)
                assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])


@pytest.mark.parametrize("cap", [16, 16384])
def test_complete_graph_pieces(T, cap):
    """K_3400, time(u, v) = max(u, v), labels by id modulo 3: c is the largest
    time of the pairs a < b < c with three distinct labels."""
    n = 3400
    iu = np.triu_indices(n, 1)
    src, dst = (x.astype(np.uint32) for x in iu)
    lab = (np.arange(n) % 3).astype(np.uint8)
    s = T.cuda.current_stream().cuda_stream
    with tp.build_graph(n, *(T.from_numpy(x).cuda() for x in (src, dst, dst.copy(), lab)), stream=s) as G:
        assert G.stats()["class_tiles"][3] > 0
        tp.tripoll_set_plan(G.handle, tp.make_plan((0,) * 4, (1024, 1024, 16384, cap)), s)
        values, counts = tp.max_edge_counts(G, T, stream=s, n_labels=3)
    below = np.array([[np.count_nonzero(lab[:c] == k) for k in range(3)] for c in range(n)], np.int64)
    want = np.array([below[c][(lab[c] + 1) % 3] * below[c][(lab[c] + 2) % 3] for c in range(n)], np.int64)
    assert want.sum() < comb(n, 3)
    assert np.array_equal(values, np.nonzero(want)[0].astype(np.uint32))
    assert np.array_equal(counts.astype(np.int64), want[want > 0])
