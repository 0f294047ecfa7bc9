"""The cut of a small graph's records into work tiles, and the merge of the
workgroups' counters: one target with R in-edges, R around the smallest cap of
a work tile (32 records), the default cap (1024) and the wave (64), surveyed by
every kernel form, alone, in a batch and served, against closed forms and the
oracle.  All values are integers: the comparison is exact."""
import numpy as np
import pytest

import oracle
from paper_2107_12330_amd import tripoll as tp

pytestmark = pytest.mark.gpu

OUT = ("count", "close_hist", "label_table", "spread_count", "open_close")
CORE = 4


def fan(R):
    """A K_4 core (vertices 0..3) and R vertices joined to all of it: 6 R + 4
    triangles, and (up to ties) every fan vertex is a pivot of each core edge."""
    core = [(a, b) for a in range(CORE) for b in range(a + 1, CORE)]
    rim = [(a, CORE + i) for i in range(R) for a in range(CORE)]
    src, dst = (np.array(x, np.uint32) for x in zip(*(core + rim)))
    rng = np.random.default_rng(R)
    n = CORE + R
    return n, src, dst, rng.integers(0, 1 << 20, len(src)).astype(np.uint32), rng.integers(0, 5, n).astype(np.uint8)


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    return torch


def dev(T, g):
    return (g[0],) + tuple(T.from_numpy(x).cuda() for x in g[1:])


SIZES = [1, 31, 32, 33, 63, 64, 65, 127, 1023, 1024, 1025, 5000]


@pytest.mark.parametrize("R", SIZES)
def test_fan_every_form(T, R):
    print("fan", R, flush=True)
    g = fan(R)
    n, src, dst, ts, vlab = g
    ref = oracle.survey(n, src, dst, ts, vlab, outputs=OUT, n_labels=5, spread_lt=1 << 14)
    assert ref["triangles"] == 6 * R + 4
    s = T.cuda.current_stream().cuda_stream
    with tp.build_graph(*dev(T, g), stream=s) as G:
        st = G.stats()
        got = tp.survey(G, stream=s, outputs=OUT, n_labels=5, spread_lt=1 << 14)
        for k in ("triangles", "spread_count", "close_hist", "label_table", "open_close"):
            assert np.array_equal(np.asarray(got[k]), np.asarray(ref[k])), k
        assert sum(got["class_triangles"]) == 6 * R + 4 and got["probes"] == st["probes"]
        assert tp.survey(G, stream=s)["triangles"] == 6 * R + 4  # no metadata
        ext = tp.survey(G, stream=s, outputs=("count", "max_edge", "degree_table"), n_labels=5, max_edge_shift=10)
        assert int(ext["degree_table"].sum()) == 6 * R + 4
        v = T.zeros(n, dtype=T.int64, device="cuda")
        e = T.zeros(st["n_edges"], dtype=T.int64, device="cuda")
        assert tp.tripoll_participation(G.handle, tp.make_spec(), v.data_ptr(), e.data_ptr(), s) == 6 * R + 4
        T.cuda.synchronize()
        want = np.full(n, 6, np.int64)
        want[:CORE] = 3 * R + 3
        assert np.array_equal(v.cpu().numpy(), want)
        rec = T.zeros((6 * R + 4) * 9, dtype=T.int32, device="cuda")
        assert tp.tripoll_enumerate(G.handle, rec.data_ptr(), 6 * R + 4, s) == 6 * R + 4
        T.cuda.synchronize()
        assert len(np.unique(np.sort(rec.cpu().numpy().reshape(-1, 9)[:, :3], axis=1), axis=0)) == 6 * R + 4


def test_fans_in_a_batch_and_served(T):
    graphs = [fan(R) for R in SIZES] * 3
    eoff = np.concatenate([[0], np.cumsum([len(g[1]) for g in graphs])]).astype(np.uint64)
    vcnt = np.array([g[0] for g in graphs], np.uint32)
    cat = [T.from_numpy(np.concatenate([g[i] for g in graphs])).cuda() for i in (1, 2, 3, 4)]
    s = T.cuda.current_stream().cuda_stream
    refs = [oracle.survey(*g, outputs=("count", "close_hist", "label_table"), n_labels=5) for g in graphs[:len(SIZES)]]
    with tp.build_batch(eoff, vcnt, *cat, stream=s) as B:
        spec = tp.make_spec(outputs=("count", "close_hist", "label_table"), n_labels=5)
        out = T.zeros(len(graphs) * tp.tripoll_batch_words(spec) + tp.TP_BATCH_SCRATCH_WORDS, dtype=T.int64, device="cuda")
        for _ in range(3):  # the same buffer: its claim counters are cleared by the survey
            tp.tripoll_survey_batch(B.handle, spec, out.data_ptr(), s)
            T.cuda.synchronize()
            got = tp.batch_dicts(out.cpu().numpy(), len(graphs), spec, 5)
            for i, d in enumerate(got):
                ref = refs[i % len(SIZES)]
                assert d["triangles"] == ref["triangles"], i
                assert np.array_equal(d["close_hist"], ref["close_hist"]), i
                assert np.array_equal(d["label_table"], ref["label_table"]), i
    with tp.Server(max_slots=8, n_labels=5) as srv:
        ids = [srv.add_graph(*dev(T, g)) for g in graphs[:len(SIZES)]]
        tickets = [(i, srv.submit(gid, outputs=("count", "close_hist", "label_table"))) for _ in range(3)
                   for i, gid in enumerate(ids)]
        for i, t in tickets:
            d = srv.wait(t)[0]
            assert d["triangles"] == refs[i]["triangles"]
            assert np.array_equal(d["close_hist"], refs[i]["close_hist"])
            assert np.array_equal(d["label_table"], refs[i]["label_table"])
