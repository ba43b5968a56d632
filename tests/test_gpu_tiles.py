"""Layer launches over lists of every length around what a workgroup's tiles and the tile counter make of them: a
row that a launch leaves out, or works on from another row's tile, differs from the rebuilt one."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2603_21090_amd import synth
from tests.helpers import rows_close, tiny_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [dict(d_mem=12, d_edge=70, heads=2, d_emb=100, d_time=100, k=5),     # two key slots
                                dict(d_mem=0, d_node=20, d_edge=9, heads=2, d_emb=20, d_time=30, k=20),    # raw edge rows, query cache at every layer
                                dict(d_mem=16, d_edge=0, heads=1, d_emb=66, d_time=70, k=10),              # one head of two slots
                                dict(d_mem=10, d_edge=66, heads=4, d_emb=32, d_time=20, k=3)])             # four
def test_streamed_rows_equal_a_rebuild_at_every_list_length(kw):
    """Endpoints drawn evenly over 70,001 nodes: batches of 8 to 8,000 edges list 16 to 70,001 rows per layer, on both sides of
    one, two and four tiles of 16 or 32 rows for each workgroup, and the rebuild lists them all."""
    import torch
    from paper_2603_21090_amd import binding
    w = tiny_workload(**{**dict(num_nodes=70_001, num_edges=120_000, batch=8_000, layers=2), **kw})
    W = synth.make_weights(w)
    nf = synth.node_features(w)
    g = binding.StreamTGN.from_workload(w, W, nf, max_batch=8_000)
    o = orc.Oracle.from_workload(w, W, nf)
    gen = np.random.default_rng(7)
    every = torch.arange(w.num_nodes, dtype=torch.int32, device="cuda")
    at, seen = 0.0, set()
    for b in (8_000, 1_500, 8, 4_000, 300, 8_000, 8_000, 8_000, 700, 8_000, 2_500, 40, 8_000, 8_000, 5_000):
        src = gen.integers(0, w.num_nodes, b).astype(np.uint32)
        dst = ((src + gen.integers(1, w.num_nodes, b)) % w.num_nodes).astype(np.uint32)
        ts = at + np.cumsum(gen.exponential(1.0, b))
        at = ts[-1]
        ef = gen.standard_normal((b, w.d_edge), dtype=np.float32)
        assert o.ingest(src, dst, ts, ef)[0] == 0
        seen.add(g.ingest_batch(src, dst, ts, ef, stats=True)["n_affected"])
        rows = [g.get_embeddings(every, layer=l) for l in (1, 2)]
        g.full_rebuild()
        for l, x in enumerate(rows, 1):
            y = g.get_embeddings(every, layer=l)
            assert torch.equal(x, y), (b, l, int((x != y).any(1).sum()))
    assert min(seen) < 8_192 and max(seen) > 32_768, sorted(seen)
    some = np.concatenate([gen.integers(0, w.num_nodes, 200), [0, 1, 65_535, 65_536, w.num_nodes - 1]]).astype(np.uint32)
    for l in (1, 2):
        assert rows_close(g.get_embeddings(some, layer=l), o.embed_nodes(some, layer=l)).all()
    g.close()


@pytest.mark.parametrize("kw", [dict(d_edge=70, heads=2, d_emb=100), dict(d_edge=0, heads=1, d_emb=100), dict(d_edge=0, heads=4, d_emb=60),
                                dict(d_edge=66, heads=2, d_emb=140, d_time=20)])
def test_a_nan_stays_in_the_rows_of_its_tile(kw):
    """Tiles of 32 rows share storage between their phases: one edge with a NaN among its features (no edge features: among a
    node's) in a late batch, over several tiles per workgroup, reaches the rows that the oracle says it reaches."""
    from paper_2603_21090_amd import binding
    from tests.test_gpu_nan import _check
    w = tiny_workload(**{**dict(num_nodes=40_000, num_edges=60_000, batch=4_000, zipf_s=1.05, d_mem=0, d_node=20, d_time=70, k=3), **kw})
    _check(binding, w, **(dict(edge=1) if w.d_edge else dict(node="quiet")))


@pytest.mark.parametrize("kw", [dict(d_edge=70, heads=2, d_emb=100, d_time=70), dict(d_edge=9, heads=2, d_emb=100, d_time=70), dict(d_edge=66, heads=2, d_emb=140, d_time=20),
                                dict(d_edge=66, heads=2, d_emb=140, d_time=70), dict(d_edge=0, heads=1, d_emb=100, d_time=20), dict(d_edge=9, heads=1, d_emb=100, d_time=70),
                                dict(d_edge=9, heads=1, d_emb=200, d_time=20), dict(d_edge=0, heads=1, d_emb=200, d_time=40), dict(d_edge=0, heads=4, d_emb=60, d_time=20),
                                dict(d_edge=70, heads=2, d_emb=100, d_mem=12, d_node=0, d_time=20)])
def test_nans_stay_in_their_rows_through_the_tiles_of_a_workgroup(kw):
    """A NaN in one node of sixty (models with a memory: one edge in a hundred of the last two batches) reaches rows of most tiles, so that
    tiles follow others that held one in the same place of the LDS.  Lists are long enough for tiles of 32 rows, and batches read the
    queries of some tiles back and project others; the rows that the oracle says are not reached keep their bits."""
    import torch
    from paper_2603_21090_amd import binding
    w = tiny_workload(**{**dict(num_nodes=42_001, num_edges=64_000, batch=8_000, zipf_s=0.2, layers=2, d_mem=0, d_node=20, k=4), **kw})
    W, nf, st = synth.make_weights(w), synth.node_features(w), synth.EdgeStream(w)
    bad_nf = None if nf is None else nf.copy()
    if nf is not None:
        bad_nf[7::60, 0] = np.nan
    o = orc.Oracle.from_workload(w, W, bad_nf)
    a, b = binding.StreamTGN.from_workload(w, W, nf), binding.StreamTGN.from_workload(w, W, bad_nf)
    every, long_lists = np.arange(w.num_nodes, dtype=np.uint32), 4 * 16 * 2 * torch.cuda.get_device_properties(0).multi_processor_count
    for i in range(w.num_batches):
        s, d, t, ef = st.batch(i)
        bad_ef = ef.copy()
        if nf is None and i >= 6:
            bad_ef[::100, 0] = np.nan
        listed = a.ingest_batch(s, d, t, ef, stats=True)["n_affected"]
        b.ingest_batch(s, d, t, bad_ef)
        assert o.ingest(s, d, t, bad_ef)[0] == 0
    assert listed > long_lists, listed
    ref = o.embed_all()
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


@pytest.mark.parametrize("heads, dk", [(1, 1), (1, 4), (1, 63), (1, 64), (1, 65), (1, 129), (1, 200), (2, 3), (2, 5), (2, 16), (2, 50), (2, 64),
                                       (2, 66), (2, 127), (4, 1), (4, 7), (4, 25), (4, 33), (4, 61)])
@pytest.mark.parametrize("kw", [dict(d_edge=9), dict(d_edge=70), dict(d_edge=0), dict(d_edge=9, delta_mode=1)])
def test_cached_rows_of_every_head_width(heads, dk, kw):
    """A cached row holds its heads' floats one behind the other, each rounded up to four and the row to sixteen: widths around
    four, a column tile and a slot, against the oracle (the embedding bar of 1e-4 per row)."""
    from paper_2603_21090_amd import binding
    delta = kw.get("delta_mode", 0)
    w = tiny_workload(num_nodes=120, num_edges=900, batch=90, d_emb=heads * dk, heads=heads, d_time=20, d_mem=12, d_edge=kw["d_edge"], k=4)
    W = synth.make_weights(w)
    o, g = orc.Oracle.from_workload(w, W), binding.StreamTGN.from_workload(w, W, delta_mode=delta, drift_gamma=0.9 if delta else 0.0)
    st = synth.EdgeStream(w)
    for b in range(w.num_batches):
        assert o.ingest(*st.batch(b))[0] == 0
        g.ingest_batch(*st.batch(b))
    if delta:
        g.full_rebuild()
    for l, ref in enumerate(o.embed_all(), 1):
        assert rows_close(g.get_embeddings(np.arange(w.num_nodes, dtype=np.uint32), layer=l), ref).all(), l
    g.close()


@pytest.mark.parametrize("k", [1, 2, 7, 31, 33, 64, 100])
def test_rings_of_every_length_wrap(k):
    """Rows whose degrees run from nothing to many times k: a ring's newest slot is the degree's remainder."""
    from paper_2603_21090_amd import binding
    w = tiny_workload(num_nodes=90, num_edges=120 * max(k, 10), batch=60 * max(k, 10), zipf_s=1.2, d_edge=9, d_time=20, d_emb=20, k=k)
    W, st = synth.make_weights(w), synth.EdgeStream(w)
    o, g = orc.Oracle.from_workload(w, W, None), binding.StreamTGN.from_workload(w, W, None)
    degree = np.bincount(np.concatenate([st.src[:w.num_edges], st.dst[:w.num_edges]]), minlength=w.num_nodes)
    assert (degree > 7 * k).any() and (degree % k != 0).any() or k == 1
    for i in range(w.num_batches):
        assert o.ingest(*st.batch(i))[0] == 0
        g.ingest_batch(*st.batch(i))
    ref = o.embed_all()
    for l in range(1, w.layers + 1):
        close = rows_close(g.get_embeddings(np.arange(w.num_nodes, dtype=np.uint32), layer=l), ref[l - 1])
        assert close.all(), f"layer {l}: rows {np.nonzero(~close)[0][:8]}"
    g.close()
