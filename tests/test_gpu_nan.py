"""A NaN among the features reaches the rows that depend on it and no other: what shares a tile, a wave or a zero weight with
it keeps its bits."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2603_21090_amd import synth
from tests.helpers import rings_matrix, rows_close, tiny_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    from paper_2603_21090_amd import binding as b
    return b


def _quiet_node(w, st):
    """A node of one or two edges whose place in a tile of sixteen is not the first."""
    deg = np.bincount(np.concatenate([st.src, st.dst]), minlength=w.num_nodes)
    at = np.nonzero((deg >= 1) & (deg <= 2) & (np.arange(w.num_nodes) % 16 > 3))[0]
    return int(at[at.size // 2])


def _check(binding, w, node=None, edge=None):
    """Poisons one column of a node's or an edge's features; the oracle says which rows that reaches."""
    W, nf, st = synth.make_weights(w), synth.node_features(w), synth.EdgeStream(w)
    bad_nf = None if nf is None else nf.copy()
    if node is not None:
        bad_nf[{"quiet": _quiet_node, "early": _early_nodes}.get(node, lambda *_: node)(w, st), 0] = np.nan
    o = orc.Oracle.from_workload(w, W, bad_nf)
    a, b = binding.StreamTGN.from_workload(w, W, nf), binding.StreamTGN.from_workload(w, W, bad_nf)
    for i in range(w.num_batches):
        s, d, t, ef = st.batch(i)
        bad_ef = ef.copy()
        if edge is not None and i == w.num_batches - edge:
            bad_ef[0 if i == 0 else len(s) // 2, 0] = np.nan
        a.ingest_batch(s, d, t, ef), b.ingest_batch(s, d, t, bad_ef)
        assert o.ingest(s, d, t, bad_ef)[0] == 0
    ref, every = o.embed_all(), np.arange(w.num_nodes, dtype=np.uint32)
    for what in ("streamed", "rebuilt"):
        for l in range(1, w.layers + 1):
            reached = np.isnan(ref[l - 1]).any(axis=1)
            assert 0 < reached.sum() < w.num_nodes // 2
            x, y = a.get_embeddings(every, layer=l), b.get_embeddings(every, layer=l)
            assert not np.isnan(x).any() and np.isnan(y[reached]).any(axis=1).all()
            off = np.nonzero((x != y).any(axis=1) & ~reached)[0]
            assert off.size == 0, f"{what}, layer {l}: rows {off[:8]} ({off.size} in all) beside the {reached.sum()} reached"
        a.full_rebuild(), b.full_rebuild()
    a.close(), b.close()


@pytest.mark.parametrize("d_node, heads", [(150, 1), (70, 1), (200, 2)])
def test_rows_of_a_tile(binding, d_node, heads):
    """Input rows longer than the head slots and of no whole 64 columns."""
    _check(binding, tiny_workload(num_nodes=400, num_edges=700, batch=100, zipf_s=0.6, d_mem=0, d_node=d_node, d_edge=0,
                                  d_emb=40 * heads, heads=heads, d_time=20, k=3), node="quiet")


@pytest.mark.parametrize("kw", [dict(d_mem=100, d_msg=100, d_edge=20), dict(d_mem=100, d_msg=100, d_edge=20, aggregator=1),
                                dict(d_mem=140, d_msg=150, d_edge=20)])
def test_endpoints_of_a_tile(binding, kw):
    """Message and memory rows of no whole 64 columns."""
    _check(binding, tiny_workload(**{**dict(num_nodes=3000, num_edges=1400, batch=200, zipf_s=0.6, d_emb=40, heads=1, d_time=20, k=3),
                                     **kw}), edge=2)


@pytest.mark.parametrize("kw", [dict(d_edge=9, heads=1, d_emb=40), dict(d_edge=9, heads=2, d_emb=100),
                                dict(d_edge=35, heads=1, d_emb=100), dict(d_edge=20, heads=4, d_emb=60)])
def test_tiles_of_a_workgroup(binding, kw):
    """Raw edge rows: columns of the padded slot that no tile of products writes, over several tiles per workgroup.  (The
    poisoned rows come early in the lists, so that tiles follow in their place.)"""
    _check(binding, tiny_workload(**{**dict(num_nodes=40_000, num_edges=60_000, batch=4_000, zipf_s=1.05, d_mem=0, d_node=20,
                                            d_time=70, k=3), **kw}), edge=1)


def _early_nodes(w, st):
    """Nodes without an edge in the later three quarters of the stream."""
    late = np.zeros(w.num_nodes, dtype=bool)
    late[st.src[w.num_edges // 4:]] = late[st.dst[w.num_edges // 4:]] = True
    return np.nonzero(~late)[0]


SHAPES = [dict(d_edge=0, heads=1, d_emb=40), dict(d_edge=9, heads=2, d_emb=100), dict(d_edge=70, heads=2, d_emb=100),
          dict(d_edge=5, heads=4, d_emb=60), dict(d_edge=0, heads=1, d_emb=200)]


@pytest.mark.parametrize("kw, poison", [(kw, p) for kw in SHAPES for p in ("node 0", "edge 0", "outside the window")
                                        if p != "edge 0" or kw["d_edge"]])
def test_entries_without_weight(binding, kw, poison):
    """Places past a row's entries name node 0 and edge 0, and entries outside the temporal window are gathered like the others:
    neither counts."""
    w = tiny_workload(**{**dict(num_nodes=900, num_edges=1500, batch=100, zipf_s=0.6, d_mem=0, d_node=20, d_time=20, k=9,
                                window=40.0 if poison == "outside the window" else 0.0), **kw})
    _check(binding, w, **{"node 0": dict(node=0), "edge 0": dict(edge=w.num_batches), "outside the window": dict(node="early")}[poison])


@pytest.mark.parametrize("kw", [dict(heads=1, d_emb=40), dict(heads=1, d_emb=40, d_edge=70), dict(heads=2, d_emb=100), dict(heads=2, d_emb=100, d_edge=70),
                                dict(heads=1, d_emb=100), dict(heads=1, d_emb=129, d_edge=70), dict(heads=2, d_emb=190), dict(heads=4, d_emb=128),
                                dict(heads=4, d_emb=60, d_edge=70), dict(heads=2, d_emb=100, d_edge=70, delta_mode=1),
                                dict(heads=1, d_emb=100, delta_mode=1), dict(heads=2, d_emb=128)])
@pytest.mark.parametrize("num_nodes", [900, 40_000])          # (rebuilds of 40,000 rows run tiles of 32)
def test_an_overflowed_key_takes_no_weight(binding, num_nodes, kw):
    """The last key column of every head overflows for one node in sixteen, against a query that makes the score minus infinity:
    such a neighbour has no weight, also where lanes past a head's floats meet its last key again."""
    delta = kw.get("delta_mode", 0)
    w = tiny_workload(**{**dict(num_nodes=num_nodes, num_edges=3 * num_nodes, batch=num_nodes // 5, zipf_s=0.3, layers=1, d_mem=0, d_node=20,
                                d_edge=9, d_time=20, k=5), **{x: v for x, v in kw.items() if x != "delta_mode"}})
    W, nf, st = synth.make_weights(w), synth.node_features(w), synth.EdgeStream(w)
    over = np.arange(num_nodes) % 16 == 5
    nf[:, 0] = np.where(over, 1e4, 0.0)
    wq, wk, wv = W["W_Q"][0], W["W_K"][0], W["W_V"][0]
    last = np.arange(1, w.heads + 1) * (w.d_emb // w.heads) - 1
    wq[0] = wk[0] = wv[0] = 0.0
    wq[:, last] = wk[:, last] = 0.0
    wq[w.d_node, last] = -1.0                                 # (the first time column is 1 at a distance of zero)
    wk[0, last] = 3e38
    o, g = orc.Oracle.from_workload(w, W, nf), binding.StreamTGN.from_workload(w, W, nf, delta_mode=delta, drift_gamma=0.9 if delta else 0.0)
    for i in range(w.num_batches):
        assert o.ingest(*st.batch(i))[0] == 0
        g.ingest_batch(*st.batch(i))
    nbr = rings_matrix(st.src, st.dst, w.num_edges, num_nodes, w.k)[0]
    hit = (nbr >= 0) & over[nbr]
    some = np.nonzero(~hit[:, :2].any(axis=1))[0]             # (a row's first chunk of entries gives the scores' reference: finite)
    assert hit[some].any(axis=1).sum() > num_nodes // 20
    ref = o.embed_all()[0][some]
    for what in ("streamed", "rebuilt"):
        close = rows_close(g.get_embeddings(some.astype(np.uint32), layer=1), ref)
        assert close.all(), f"{what}: {(~close).sum()} of {some.size} rows, {hit[some][~close].any(axis=1).sum()} of them with such a neighbour"
        g.full_rebuild()
    g.close()
