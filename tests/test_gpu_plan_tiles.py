"""The tiles that a survey walks under a plan: a cap that a caller chose is
walked as it is, the default cap is cut finer on small graphs (but not into
many times as many tiles), and the statistics report the walked tiles.  Targets of the tiny, small and large class
with record counts at the edges of a wave (64), of its blocks of records (128,
192) and of the caps, through every kernel form, against closed forms.  All
values are integers: the comparison is exact."""
from math import comb

import numpy as np
import pytest

from paper_2107_12330_amd import tripoll as tp

pytestmark = pytest.mark.gpu

TIME = 12345
DEFAULT = (1024, 1024, 16384, 16384)
BOUNDS = (51, 819, 3276)  # largest d+ of the tiny, small and large class
LEAST = (16, 32, 512, 512)  # fewest records of the finer cut's cap
CLAIMERS = (256 * 32, 256 * 5, 256, 256)
SHARE = (8, 8, 4, 4)  # tiles for each of them


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    return torch


def crown(T, c, R):
    """A clique of c vertices (labels 0 and 1 in turn) and R vertices (label 2)
    joined to all of it.  Every time is TIME.  The clique's vertex of rank i has
    d+ = c - 1 - i and R + i records."""
    iu = np.triu_indices(c, 1)
    src = np.concatenate([iu[0], np.tile(np.arange(c), R)]).astype(np.uint32)
    dst = np.concatenate([iu[1], np.repeat(c + np.arange(R), c)]).astype(np.uint32)
    lab = np.concatenate([np.arange(c) % 2, np.full(R, 2)]).astype(np.uint8)
    return (c + R,) + tuple(T.from_numpy(x).cuda() for x in (src, dst, np.full(len(src), TIME, np.uint32), lab))


def expected_tiles(G, caps):
    """Tiles and staged out-list entries of each class (no huge targets), cut
    with `caps`, from the exported rows."""
    x = tp.export(G)
    rp = x["rowptr"].astype(np.int64)
    d = np.diff(rp)
    src = np.repeat(np.arange(len(d)), d)
    rest = rp[src + 1] - 1 - np.arange(len(src))
    col = x["col"].astype(np.int64)
    keep = (rest > 0) & (d[col] > 0)
    cnt = np.bincount(col[keep], minlength=len(d))
    work = np.bincount(col[keep], weights=rest[keep].astype(float), minlength=len(d)).astype(np.int64)
    cls = np.searchsorted(BOUNDS, d, side="left")
    tiles, staged = [], []
    for k in range(4):
        on = (cls == k) & (cnt > 0)

        def cut(cap):
            return np.minimum(cnt[on], np.maximum(-(-cnt[on] // cap), -(-work[on] // (256 * cap))))

        n = cut(caps[k])
        if caps[k] == DEFAULT[k]:
            records = int(cnt[on].sum())
            finest = min(caps[k], max(LEAST[k], records // (SHARE[k] * CLAIMERS[k])))
            finer = cut(finest)
            if not (finer.sum() <= 4 * n.sum() or 8 * n.sum() < CLAIMERS[k] or work[on].sum() >= int(n.sum()) << 16
                    or (k == 0 and records < 1 << 20)):
                finer = cut(max(finest, records // max(2 * int(n.sum()), 2 * CLAIMERS[k] if k == 0 else 0)))
            n = finer
        tiles.append(int(n.sum()))
        staged.append(int((n * d[on]).sum()))
    return tiles, staged


def check_forms(T, G, c, R, s):
    n, m = c + R, comb(c, 2) + c * R
    core, rim = comb(c, 3), R * comb(c, 2)
    assert tp.survey(G, stream=s)["triangles"] == core + rim
    got = tp.survey(G, stream=s, outputs=("count", "close_hist", "label_table"), n_labels=3)
    assert got["triangles"] == core + rim and int(got["close_hist"][0]) == core + rim
    n0, n1 = (c + 1) // 2, c // 2
    table = {(2, 1, 0): R * n0 * n1, (2, 0, 0): R * comb(n0, 2), (2, 1, 1): R * comb(n1, 2)}
    for key, v in table.items():
        assert int(got["label_table"][tp.tripoll_msidx(*key)]) == v, key
    ext = tp.survey(G, stream=s, outputs=("count", "max_edge", "degree_table", "open_close"), n_labels=3,
                    max_edge_shift=5)
    assert int(ext["max_edge"][TIME >> 5]) == R * n0 * n1 and int(ext["degree_table"].sum()) == core + rim
    assert int(ext["open_close"][0][0]) == core + rim
    v = T.zeros(n, dtype=T.int64, device="cuda")
    e = T.zeros(m, dtype=T.int64, device="cuda")
    assert tp.tripoll_participation(G.handle, tp.make_spec(), v.data_ptr(), e.data_ptr(), s) == core + rim
    T.cuda.synchronize()
    assert (v[c:] == comb(c, 2)).all().item() and (v[:c] == comb(c - 1, 2) + R * (c - 1)).all().item()
    assert int((e == c - 1).sum()) == c * R and int((e == c - 2 + R).sum()) == comb(c, 2)
    values, counts = tp.max_edge_counts(G, T, stream=s, n_labels=3)
    assert values.tolist() == [TIME] and counts.tolist() == [R * n0 * n1]


SHAPES = [(20, R) for R in (15, 16, 17, 63, 64, 65, 127, 128, 129, 193, 1023, 1024, 1025)] + \
         [(60, R) for R in (31, 32, 33, 64, 129)] + [(830, R) for R in (511, 512, 513)]


@pytest.mark.parametrize("c,R", SHAPES)
def test_plan_is_walked(T, c, R):
    s = T.cuda.current_stream().cuda_stream
    assert not (R == c - 2 or R == 1)  # the two kinds of edges are told apart by their counts
    with tp.build_graph(*crown(T, c, R), stream=s) as G:
        assert tp.plan_dict(tp.tripoll_get_plan(G.handle))["tile_records"] == list(DEFAULT)
        for caps in (DEFAULT, (16,) * 4, (64, 32, 512, 16), (2048, 512, 8192, 16), (65536,) * 4, DEFAULT):
            print("K_%d + %d" % (c, R), caps, flush=True)
            tp.tripoll_set_plan(G.handle, tp.make_plan((0,) * 4, caps), s)
            st = G.stats()
            tiles, staged = expected_tiles(G, caps)
            assert st["class_tiles"] == tiles and st["class_staged"] == staged and st["n_tiles"] == sum(tiles)
            check_forms(T, G, c, R, s)


@pytest.mark.parametrize("c,R", [(20, 64), (20, 193), (60, 33), (830, 512)])
def test_plan_is_walked_by_served_requests(T, c, R):
    s = T.cuda.current_stream().cuda_stream
    total = comb(c, 3) + R * comb(c, 2)
    with tp.Server(max_slots=4, n_labels=3) as srv:
        gid = srv.add_graph(*crown(T, c, R))
        for caps in (DEFAULT, (16,) * 4, (65536,) * 4):
            tp.tripoll_set_plan(srv.graph(gid), tp.make_plan((0,) * 4, caps), s)
            tickets = [srv.submit(gid, outputs=("count", "close_hist", "label_table")) for _ in range(5)]
            for t in tickets:
                d = srv.wait(t)[0]
                assert d["triangles"] == total and int(d["close_hist"][0]) == total


def test_tuner_times_each_cap(T):
    """The four caps of the tuner are four cuts of a small graph (with the
    finer cut under every cap they were one)."""
    s = T.cuda.current_stream().cuda_stream
    with tp.build_graph(*crown(T, 20, 30000), stream=s) as G:
        seen = set()
        for cap in (256, 1024, 4096, 16384):
            tp.tripoll_set_plan(G.handle, tp.make_plan((0,) * 4, (cap,) * 4), s)
            seen.add(tuple(G.stats()["class_tiles"]))
        assert len(seen) == 4
        r = tp.tune_dict(tp.tripoll_tune(G.handle, tp.make_spec(), s))
        assert tp.plan_dict(tp.tripoll_get_plan(G.handle)) == r["chosen"]
        assert tp.survey(G, stream=s)["triangles"] == comb(20, 3) + 30000 * comb(20, 2)


@pytest.mark.parametrize("hubs,leaves,each", [(1500, 700_000, 4), (1500, 150_000, 4), (400, 60_000, 10)])
def test_hubs_of_leaves_are_cut_boundedly(T, hubs, leaves, each):
    """Few targets with most of the records: the finer cut is bounded from 2^20
    records of the tiny class on, and in the small class."""
    gen = T.Generator(device="cuda")
    gen.manual_seed(hubs + leaves)
    s = T.cuda.current_stream().cuda_stream
    a = T.randint(0, hubs, (hubs * each,), generator=gen, device="cuda")
    src = T.cat([a, T.arange(hubs, hubs + leaves, device="cuda").repeat_interleave(each)]).int()
    dst = T.randint(0, hubs, (src.numel(),), generator=gen, device="cuda").int()
    if each == 10:  # hubs joined to most others: small targets
        iu = np.triu_indices(hubs, 1)
        src = T.cat([src, T.from_numpy(iu[0].astype(np.int32)).cuda()])
        dst = T.cat([dst, T.from_numpy(iu[1].astype(np.int32)).cuda()])
    with tp.build_graph(hubs + leaves, src, dst, stream=s) as G:
        st = G.stats()
        print(st["class_records"], st["class_tiles"], flush=True)
        tiles, staged = expected_tiles(G, DEFAULT)
        assert st["class_tiles"] == tiles and st["class_staged"] == staged
        ref = tp.survey(G, stream=s, outputs=("count", "close_hist"), strategy=tp.TP_STRAT_GLOBAL_SEARCH)
        got = tp.survey(G, stream=s, outputs=("count", "close_hist"))
        assert got["triangles"] == ref["triangles"] and np.array_equal(got["close_hist"], ref["close_hist"])
        for caps in ((64,) * 4, (65536,) * 4):
            tp.tripoll_set_plan(G.handle, tp.make_plan((0,) * 4, caps), s)
            assert expected_tiles(G, caps) == (G.stats()["class_tiles"], G.stats()["class_staged"])
            again = tp.survey(G, stream=s, outputs=("count", "close_hist"))
            assert again["triangles"] == ref["triangles"] and np.array_equal(again["close_hist"], ref["close_hist"])
