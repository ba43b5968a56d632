"""The layer kernel's operands at any common scale, workgroups that walk several tiles, and projected rows at the edges of
their staging."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2603_21090_amd import synth
from tests.helpers import rows_close, tiny_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    from paper_2603_21090_amd import binding as b
    return b


def _rescaled(w, W, s):
    """The same model in units of 1 / s of its embeddings: node features, caches and outputs come out s times as large,
    queries 1 / s times, scores and attention weights as they were."""
    V = dict(W)
    d_in = lambda l: (w.d_mem + w.d_node) if l == 0 else w.d_emb
    for name in ("W_Q", "W_K", "W_V"):
        V[name] = [m.copy() for m in W[name]]
    for l in range(w.layers):
        V["W_Q"][l][:d_in(l)] *= s ** -2
        V["W_Q"][l][d_in(l):] *= 1 / s
        V["W_K"][l][d_in(l):] *= s
        V["W_V"][l][d_in(l):] *= s
    V["b_O"] = [(b * s).astype(np.float32) for b in W["b_O"]]
    return V


@pytest.mark.parametrize("e", [-40, -11, 13, 40])
@pytest.mark.parametrize("kw", [dict(d_edge=6, heads=2, d_emb=100, d_time=100), dict(d_edge=70, heads=4, d_emb=64, d_time=30),
                                dict(d_edge=0, heads=1, d_emb=130, d_time=70)])
def test_powers_of_two_change_nothing(binding, kw, e):
    """A model rescaled by a power of two gives the same bits, rescaled: exact, no tolerance."""
    w = tiny_workload(num_nodes=300, num_edges=2400, batch=200, layers=2, d_mem=0, d_node=20, k=5, **kw)
    W, nf, st, s = synth.make_weights(w), synth.node_features(w), synth.EdgeStream(w), 2.0 ** e
    a = binding.StreamTGN.from_workload(w, W, nf)
    b = binding.StreamTGN.from_workload(w, _rescaled(w, W, s), (nf * s).astype(np.float32))
    for i in range(w.num_batches):
        batch = st.batch(i)
        a.ingest_batch(*batch), b.ingest_batch(*batch)
    every = np.arange(w.num_nodes, dtype=np.uint32)
    for l in (1, 2):
        x, y = a.get_embeddings(every, layer=l), b.get_embeddings(every, layer=l)
        assert np.abs(x).max() > 1e-3 and np.array_equal(x * np.float32(s), y), f"layer {l}"
    a.close(), b.close()


@pytest.mark.parametrize("kw", [
    dict(d_mem=20, d_edge=7, d_time=70, d_emb=100, heads=2),             # raw edges; time columns that end inside a slot
    dict(d_mem=20, d_edge=70, d_time=70, d_emb=100, heads=2),            # projected edges
    dict(d_mem=20, d_edge=0, d_time=20, d_emb=100, heads=1),             # one wide head, one time slot: output rows take the input rows' place
    dict(d_mem=20, d_node=130, d_edge=3, d_time=20, d_emb=40, heads=1, k=40),   # rows and lists too long to be staged a tile ahead
    dict(d_mem=20, d_edge=5, d_time=30, d_emb=60, heads=4),              # four heads, two passes of a wave
])
def test_workgroups_of_several_tiles(binding, kw):
    """More rows than a launch has workgroups for (two tiles and more per workgroup): what a tile leaves in LDS must not
    reach the next one's rows."""
    w = tiny_workload(**{**dict(num_nodes=26_000, num_edges=40_000, batch=8_000, layers=2, k=4, zipf_s=1.05, d_msg=20), **kw})
    W, nf, st = synth.make_weights(w), synth.node_features(w), synth.EdgeStream(w)
    o, g = orc.Oracle.from_workload(w, W, nf), binding.StreamTGN.from_workload(w, W, nf)
    for i in range(w.num_batches):
        batch = st.batch(i)
        assert o.ingest(*batch)[0] == 0
        g.ingest_batch(*batch)
    every, ref = np.arange(w.num_nodes, dtype=np.uint32), o.embed_all()
    for what in ("streamed", "rebuilt"):
        for l in (1, 2):
            ok = rows_close(g.get_embeddings(every, layer=l), ref[l - 1], 1e-4)
            assert ok.all(), f"{what}, layer {l}: {np.count_nonzero(~ok)} rows out of tolerance, first {np.argmin(ok)}"
        g.full_rebuild()
    g.close()


@pytest.mark.parametrize("kw", [
    dict(d_mem=0, d_node=30, d_edge=9, d_time=100, d_emb=100, heads=2),      # raw edges, both layers with a query cache
    dict(d_mem=0, d_node=30, d_edge=80, d_time=50, d_emb=100, heads=2),      # projected edges
    dict(d_mem=30, d_edge=9, d_time=100, d_emb=100, heads=2),                # the first layer alone has one
    dict(d_mem=0, d_node=30, d_edge=0, d_time=20, d_emb=100, heads=1),       # one wide head
    dict(d_mem=0, d_node=30, d_edge=9, d_time=70, d_emb=60, heads=4),        # four heads
    dict(d_mem=30, d_edge=9, d_time=70, d_emb=40, heads=1),                  # rows of one slot
    dict(d_mem=0, d_node=30, d_edge=9, d_time=100, d_emb=128, heads=4, k=20),   # more than 64 KB of LDS, rebuilds included
])
def test_queries_read_back_over_several_tiles(binding, kw):
    """Streamed rows (queries read back from the cache where they did not change) have the bits of rebuilt rows (everything
    projected)."""
    w = tiny_workload(**{**dict(num_nodes=40_000, num_edges=64_000, batch=4_000, layers=2, k=6, zipf_s=1.05, d_msg=30), **kw})
    g, st = binding.StreamTGN.from_workload(w, synth.make_weights(w), synth.node_features(w)), synth.EdgeStream(w)
    for i in range(w.num_batches):
        g.ingest_batch(*st.batch(i))
    every = np.arange(w.num_nodes, dtype=np.uint32)
    streamed = [g.get_embeddings(every, layer=l) for l in (1, 2)]
    g.full_rebuild()
    for l in (1, 2):
        assert np.array_equal(streamed[l - 1], g.get_embeddings(every, layer=l)), f"layer {l}"
    g.close()


@pytest.mark.parametrize("kw", [
    dict(d_mem=30, d_node=7, d_edge=70),            # memory ends inside a 16-byte piece, rows of no whole pieces
    dict(d_mem=32, d_node=100, d_edge=300),         # five chunks: more than are requested together
    dict(d_mem=0, d_node=130, d_edge=257),          # node rows too long for four tiles an item
    dict(d_mem=64, d_node=0, d_edge=65),
])
@pytest.mark.parametrize("shift", [0, 1])
def test_projected_rows(binding, kw, shift):
    """Cached key|value rows of nodes and edges at the edges of their staging, with features that start on a 16-byte boundary
    and off it."""
    import torch
    w = tiny_workload(num_nodes=200, num_edges=900, batch=90, layers=2, k=5, d_time=20, d_emb=40, d_msg=20, **kw)
    W, nf, st = synth.make_weights(w), synth.node_features(w), synth.EdgeStream(w)
    o, g = orc.Oracle.from_workload(w, W, nf), binding.StreamTGN.from_workload(w, W, nf)
    for i in range(w.num_batches):
        s, d, t, ef = st.batch(i)
        assert o.ingest(s, d, t, ef)[0] == 0
        room = torch.zeros(ef.size + shift, device="cuda")
        room[shift:] = torch.from_numpy(ef.reshape(-1)).cuda()
        g.ingest_batch(torch.from_numpy(s.astype(np.int32)).cuda(), torch.from_numpy(d.astype(np.int32)).cuda(),
                       torch.from_numpy(t).cuda(), room[shift:].view(ef.shape))
    every, ref = np.arange(w.num_nodes, dtype=np.uint32), o.embed_all()
    streamed = [g.get_embeddings(every, layer=l) for l in (1, 2)]
    g.full_rebuild()
    for l in (1, 2):
        assert rows_close(streamed[l - 1], ref[l - 1], 1e-4).all() and np.array_equal(streamed[l - 1], g.get_embeddings(every, layer=l))
    g.close()
