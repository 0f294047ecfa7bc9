"""Runs of copies of one pair in the sorted raw edges, around the sizes where
the dedup changes hands: a round of 64, a wave's 1024, a tile's 4096, and runs
that start inside one and end in another; and sorts around the sizes where
their shape changes (one workgroup up to 8192 64-bit keys, 1024-key tiles up
to 65,536 keys, 4096-key ones, 8192-key ones from 2^22 keys).  Exact: integers
against numpy and the oracle."""
import numpy as np
import pytest

import oracle
from paper_2107_12330_amd import tripoll as tp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    return torch


def build(T, n, src, dst, ts, directed=False):
    d = [T.from_numpy(np.ascontiguousarray(x)).cuda() for x in (src, dst, ts, np.zeros(n, np.uint8))]
    return tp.build_graph(n, *d, stream=T.cuda.current_stream().cuda_stream, tie=tp.TP_TIE_ID, directed=directed), d


@pytest.mark.parametrize("run", [1, 2, 63, 64, 65, 1000, 1023, 1024, 1025, 4095, 4096, 4097, 20000])
@pytest.mark.parametrize("before", [0, 1, 62, 1023])
def test_run_of_copies(T, run, before):
    """`before` single pairs, then `run` copies of one pair whose smallest time
    is its last, middle or first copy, then single pairs; some self-loops."""
    print("run", run, "after", before, flush=True)
    rng = np.random.default_rng(run * 7 + before)
    n = 3000
    # sorted by pair: (0, 1 .. before), the run (1, 2), then (5, 6 ..)
    lo = np.concatenate([np.zeros(before), np.full(run, 1), np.full(70, 5)]).astype(np.uint32)
    hi = np.concatenate([1 + np.arange(before), np.full(run, 2), 6 + np.arange(70)]).astype(np.uint32)
    flip = rng.random(len(lo)) < 0.5
    src, dst = np.where(flip, hi, lo), np.where(flip, lo, hi)
    for place in {0, run // 2, run - 1}:
        ts = rng.integers(1000, 1 << 32, len(lo), dtype=np.uint64).astype(np.uint32)
        ts[before + place] = 7
        order = rng.permutation(len(lo))
        loops = rng.integers(0, n, 5).astype(np.uint32)
        s = np.concatenate([src[order], loops])
        d = np.concatenate([dst[order], loops])
        t = np.concatenate([ts[order], np.zeros(5, np.uint32)])
        G, keep = build(T, n, s, d, t)
        with G:
            st = G.stats()
            assert st["n_edges"] == before + 1 + 70 and st["n_self_loops"] == 5
            x = tp.export(G)
            rows = np.repeat(np.arange(n), np.diff(x["rowptr"].astype(np.int64)))
            a, b = x["rank_to_id"][rows], x["rank_to_id"][x["col"]]
            got = {(int(min(u, v)), int(max(u, v))): int(w) for u, v, w in zip(a, b, x["etime"])}
        want = {(0, 1 + i): int(ts[i]) for i in range(before)}
        want[(1, 2)] = 7
        want.update({(5, 6 + i): int(ts[before + run + i]) for i in range(70)})
        assert got == want


@pytest.mark.parametrize("run", [2, 64, 1024, 5000])
def test_directions_of_a_run(T, run):
    """One copy of the run goes the other way: the pair is mutual."""
    for place in (0, run // 2, run - 1):
        src = np.concatenate([np.full(run, 0), [1, 2]]).astype(np.uint32)
        dst = np.concatenate([np.full(run, 1), [2, 0]]).astype(np.uint32)
        src[place], dst[place] = 1, 0
        G, keep = build(T, 3, src, dst, np.arange(len(src), dtype=np.uint32), directed=True)
        with G:
            got = tp.survey(G, outputs=("count", "directed"))
            assert got["triangles"] == 1 and got["directed"][4] == 1  # 120C
    src, dst = np.full(run + 2, 0, np.uint32), np.full(run + 2, 1, np.uint32)
    src[-2:], dst[-2:] = (1, 2), (2, 0)
    G, keep = build(T, 3, src, dst, np.arange(len(src), dtype=np.uint32), directed=True)
    with G:
        assert tp.survey(G, outputs=("count", "directed"))["directed"][1] == 1  # 030C


@pytest.mark.parametrize("m", [1, 1023, 1024, 1025, 8192, 8193, 65535, 65536, 65537, 262144, 262145, (1 << 22) - 1, 1 << 22, (1 << 22) + 8191])
@pytest.mark.parametrize("n", [300, 1025, 8192, 8193, 70001])
def test_sort_shapes(T, m, n):
    """The CSR of random edges (sorts of about m keys), against numpy."""
    print("edges", m, "vertices", n, flush=True)
    rng = np.random.default_rng(m + n)
    src, dst = (rng.integers(0, n, m).astype(np.uint32) for _ in range(2))
    ts = rng.integers(0, 1 << 32, m, dtype=np.uint64).astype(np.uint32)
    G, keep = build(T, n, src, dst, ts)
    with G:
        x = tp.export(G)
    lo, hi = np.minimum(src, dst).astype(np.int64), np.maximum(src, dst).astype(np.int64)
    key = (lo * n + hi)[lo != hi]
    t = ts[lo != hi]
    order = np.lexsort((t, key))
    uk, first = np.unique(key[order], return_index=True)
    ut = t[order][first]
    deg = np.bincount(uk // n, minlength=n) + np.bincount(uk % n, minlength=n)
    perm = np.lexsort((np.arange(n), deg))
    rank = np.empty(n, np.int64)
    rank[perm] = np.arange(n)
    a, b = rank[uk // n], rank[uk % n]
    s, d = np.minimum(a, b), np.maximum(a, b)
    o = np.lexsort((d, s))
    assert np.array_equal(x["rank_to_id"], perm)
    assert np.array_equal(x["col"], d[o]) and np.array_equal(x["etime"], ut[o])
    assert np.array_equal(np.diff(x["rowptr"].astype(np.int64)), np.bincount(s, minlength=n))


def test_survey_after_many_builds(T):
    """Builds of different sizes in turn reuse each other's buffers."""
    rng = np.random.default_rng(5)
    graphs = []
    for n in (50, 3000, 400, 20000, 7):
        m = n * 9
        g = [rng.integers(0, n, m).astype(np.uint32), rng.integers(0, n, m).astype(np.uint32),
             rng.integers(0, 1 << 20, m).astype(np.uint32)]
        ref = oracle.survey(n, *g, np.zeros(n, np.uint8), outputs=("count", "close_hist"), n_labels=1)
        graphs.append((n, g, ref))
    held = []
    for i in range(15):
        n, g, ref = graphs[i % 5]
        G, keep = build(T, n, *g)
        held.append((G, ref))
        if i % 4 == 3:
            held.pop(0)[0].close()
        for H, r in held:
            got = tp.survey(H, outputs=("count", "close_hist"))
            assert got["triangles"] == r["triangles"] and np.array_equal(got["close_hist"], r["close_hist"])
    for H, _ in held:
        H.close()


@pytest.mark.parametrize("n", [4097, 8191, 8192, 8193, 1 << 17, (1 << 19) + 3])
@pytest.mark.parametrize("hub", [False, True])
def test_degrees_counted_by_parts(T, n, hub):
    """Degrees counted from a partition of the higher ends (from 2^20 edges of
    at least 13-bit ids on): every degree, through the order it gives, with
    the ends spread evenly or mostly at one vertex's part."""
    print("vertices", n, "hub", hub, flush=True)
    rng = np.random.default_rng(n)
    m = 2400000
    src, dst = (rng.integers(0, n, m).astype(np.uint32) for _ in range(2))
    if hub:
        dst[: m // 2] = n - 1 - rng.integers(0, min(n, 700), m // 2).astype(np.uint32)
    G, keep = build(T, n, src, dst, np.zeros(m, np.uint32))
    with G:
        st, x = G.stats(), tp.export(G)
    lo, hi = np.minimum(src, dst).astype(np.int64), np.maximum(src, dst).astype(np.int64)
    uk = np.unique((lo * n + hi)[lo != hi])
    assert len(uk) >= 1 << 20 and st["n_edges"] == len(uk)
    deg = np.bincount(uk // n, minlength=n) + np.bincount(uk % n, minlength=n)
    assert st["d_max"] == deg.max()
    assert np.array_equal(x["rank_to_id"], np.lexsort((np.arange(n), deg)))
