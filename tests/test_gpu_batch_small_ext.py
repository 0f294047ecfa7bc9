"""The extended outputs of a batch of very many small graphs, whose waves claim
more tiles at a time: every graph's block against the batch's own union, and
sampled graphs against their own surveys.  All values are integers: the
comparison is exact."""
import numpy as np
import pytest

import oracle
from paper_2107_12330_amd import tripoll as tp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graphs,n,m", [(20000, 40, 120), (3000, 250, 2500), (40, 3000, 40000)])
def test_many_small_graphs(graphs, n, m):
    import torch as T
    T.cuda.set_device(0)
    print(graphs, n, m, flush=True)
    rng = np.random.default_rng(graphs)
    src = (rng.random((graphs, m)) ** 2 * n).astype(np.uint32)
    dst = (rng.random((graphs, m)) ** 2 * n).astype(np.uint32)
    ts = rng.integers(0, 1 << 20, (graphs, m)).astype(np.uint32)
    lab = rng.integers(0, 4, (graphs, n)).astype(np.uint8)
    s = T.cuda.current_stream().cuda_stream
    outputs = ("count", "close_hist", "open_close", "max_edge", "degree_table")
    kw = dict(outputs=outputs, n_labels=4, max_edge_shift=10)
    spec = tp.make_spec(**kw)
    words = tp.tripoll_batch_words(spec)
    dev = [T.from_numpy(x.reshape(-1)).cuda() for x in (src, dst, ts, lab)]
    with tp.build_batch(np.arange(graphs + 1, dtype=np.uint64) * m, np.full(graphs, n, np.uint32), *dev, stream=s) as B:
        out = T.zeros(graphs * words + tp.TP_BATCH_SCRATCH_WORDS, dtype=T.int64, device="cuda")
        for _ in range(2):
            tp.tripoll_survey_batch(B.handle, spec, out.data_ptr(), s)
        T.cuda.synchronize()
        total = out[:graphs * words].view(graphs, words).sum(0).cpu().numpy()
        union = tp.survey(B, stream=s, outputs=("count", "close_hist", "open_close", "max_edge"), n_labels=4,
                          max_edge_shift=10)
        both = tp.batch_dicts(total.view(np.uint64), 1, spec, 4)[0]
        assert both["triangles"] == union["triangles"] == int(both["degree_table"].sum()) > 0
        for k in ("close_hist", "open_close", "max_edge"):
            assert np.array_equal(np.asarray(both[k]), np.asarray(union[k])), k
        for i in rng.choice(graphs, 12, replace=False):
            i = int(i)
            got = tp.batch_dicts(out[i * words:(i + 1) * words].cpu().numpy().view(np.uint64), 1, spec, 4)[0]
            ref = oracle.survey(n, src[i], dst[i], ts[i], lab[i], outputs=outputs, n_labels=4, max_edge_shift=10)
            for k in ("triangles", "close_hist", "open_close", "max_edge", "degree_table"):
                assert np.array_equal(np.asarray(got[k]), np.asarray(ref[k])), (i, k)
