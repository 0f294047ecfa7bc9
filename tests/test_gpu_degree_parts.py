"""Degrees counted by parts of 25- and 26-bit ids (partitions of 10 bits, parts
of one and two ranges of counters), and from sorted ends beyond: every vertex
in the degree order, against the degrees of a ring with a few stars."""
import numpy as np
import pytest

from paper_2107_12330_amd import tripoll as tp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(1 << 24) + 3, (1 << 25) - 1, (1 << 25) + 5, (1 << 26) - 7, (1 << 26) + 9])
def test_degree_order_of_a_ring_with_stars(n):
    import torch as T
    T.cuda.set_device(0)
    print(n, flush=True)
    i = T.arange(n, device="cuda", dtype=T.int64)
    hubs = [0, n // 2 + 1, n - 1]
    src, dst = [i], [(i + 1) % n]
    want = T.full((n,), 2, dtype=T.int64, device="cuda")
    for k, h in enumerate(hubs):
        # vertices between the neighbours of all hubs, another residue for each
        x = T.arange(10 + k, n - 10, 1009, device="cuda", dtype=T.int64)
        x = x[(x - n // 2 - 1).abs() > 10]
        src.append(T.full_like(x, h))
        dst.append(x)
        want[x] += 1
        want[h] += x.numel()
    src, dst = T.cat(src).int(), T.cat(dst).int()
    s = T.cuda.current_stream().cuda_stream
    with tp.build_graph(n, src, dst, stream=s) as G:
        st = G.stats()
        assert st["n_edges"] == src.numel() >= n and st["d_max"] == int(want.max())
        order = np.zeros(n, np.uint32)
        tp.tripoll_graph_export(G.handle, rank_to_id=order)
    ids = T.from_numpy(order.view(np.int32)).cuda().long()
    assert (T.bincount(ids, minlength=n) == 1).all().item()
    d = want[ids]
    assert (d[1:] >= d[:-1]).all().item()
