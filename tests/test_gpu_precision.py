"""Embeddings are computed in 32 bits throughout: magnitudes that differ inside a row or a matrix cost nothing, and whole
tables lie as near to 64-bit results as sums of 32-bit products do."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2603_21090_amd import synth
from tests.helpers import tiny_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    from paper_2603_21090_amd import binding as b
    return b


def _mixed_units(w, W, seed):
    """The same model with every input column, query / key column, value column and hidden column in a unit of its own, a
    power of two: each matrix takes back in its rows what the columns in front of it were given.  Returns the weights, the
    factors of the node features, edge features and final columns."""
    rng = np.random.default_rng(seed)
    f = lambda n: np.exp2(rng.integers(-30, 31, n)).astype(np.float32)
    V = dict(W)
    unit_in, unit_e = f(w.d_mem + w.d_node), f(w.d_edge)
    node_units = unit_in
    for name in ("W_Q", "W_K", "W_V", "W_O", "b_O"):
        V[name] = [m.copy() for m in W[name]]
    for l in range(w.layers):
        d_in, qk, v, out = len(unit_in), f(w.d_emb), f(w.d_emb), f(w.d_emb)
        V["W_Q"][l] = W["W_Q"][l] * qk
        V["W_K"][l] = W["W_K"][l] / qk
        V["W_V"][l] = W["W_V"][l] * v
        for name in ("W_Q", "W_K", "W_V"):
            V[name][l][:d_in] /= unit_in[:, None]
        for name in ("W_K", "W_V"):
            V[name][l][d_in:d_in + w.d_edge] /= unit_e[:, None]
        V["W_O"][l] = W["W_O"][l] / v[:, None] * out
        V["b_O"][l] = W["b_O"][l] * out
        unit_in = out
    return V, node_units, unit_e, unit_in


@pytest.mark.parametrize("kw", [dict(d_edge=9, heads=2, d_emb=100, d_time=100),            # raw edge rows
                                dict(d_edge=70, heads=4, d_emb=64, d_time=30),             # projected
                                dict(d_edge=0, d_node=150, heads=1, d_emb=130, d_time=70)])
def test_units_of_columns_change_nothing(binding, kw):
    """Factors of two inside rows and matrices leave every product and every sum what it was: the same bits, in the
    columns' own units.  Exact, no tolerance."""
    w = tiny_workload(**{**dict(num_nodes=300, num_edges=2400, batch=200, layers=2, d_mem=0, d_node=20, k=5), **kw})
    W, nf, st = synth.make_weights(w), synth.node_features(w), synth.EdgeStream(w)
    V, node_units, edge_units, out_units = _mixed_units(w, W, 5)
    a = binding.StreamTGN.from_workload(w, W, nf)
    b = binding.StreamTGN.from_workload(w, V, nf * node_units)
    for i in range(w.num_batches):
        s, d, t, ef = st.batch(i)
        a.ingest_batch(s, d, t, ef), b.ingest_batch(s, d, t, ef * edge_units)
    every = np.arange(w.num_nodes, dtype=np.uint32)
    for what in ("streamed", "rebuilt"):
        x, y = a.get_embeddings(every), b.get_embeddings(every)
        assert np.abs(x).max() > 1e-3 and np.array_equal(x * out_units, y), what
        a.full_rebuild(), b.full_rebuild()
    a.close(), b.close()


@pytest.mark.parametrize("kw", [
    dict(d_mem=100, d_edge=172, d_time=100, d_emb=100, d_msg=100, heads=2, k=10),
    dict(d_mem=0, d_node=100, d_edge=64, d_time=100, d_emb=100, heads=2, k=20),
    dict(d_mem=128, d_edge=0, d_time=64, d_emb=128, d_msg=128, heads=4, k=10),
    dict(d_mem=64, d_edge=16, d_time=64, d_emb=64, d_msg=64, heads=1, k=10),
    dict(d_mem=100, d_edge=4, d_time=128, d_emb=100, d_msg=100, heads=1, k=5),
])
@pytest.mark.parametrize("delta", [0, 1])
def test_whole_tables_against_64_bits(binding, kw, delta):
    """Rebuilt tables.  A sum of n 32-bit products is off by about sqrt(n / 2) roundings of 2^-24 (n up to 172: 5.5e-7), and a
    row passes five such sums, whose errors the averages over neighbours and the attention weights' own sums
    damp: about 3e-7 (2-norm) and 3e-6 of the root mean square (largest) were measured.  Four times that is allowed;
    operands rounded to 18 bits (2^-20 of an operand each, root mean square) are past it."""
    w = tiny_workload(**{**dict(num_nodes=1500, num_edges=8000, batch=200, layers=2), **kw})
    W, nf, st = synth.make_weights(w), synth.node_features(w), synth.EdgeStream(w)
    o = orc.Oracle.from_workload(w, W, nf)
    g = binding.StreamTGN.from_workload(w, W, nf, delta_mode=delta, drift_gamma=0.9 if delta else 0.0)
    for i in range(w.num_batches):
        batch = st.batch(i)
        assert o.ingest(*batch)[0] == 0
        g.ingest_batch(*batch)
    g.full_rebuild()
    every = np.arange(w.num_nodes, dtype=np.uint32)
    for l, ref in enumerate(o.embed_all(), 1):
        ref = ref.astype(np.float64)
        e = g.get_embeddings(every, layer=l).astype(np.float64) - ref
        rel, worst = np.linalg.norm(e) / np.linalg.norm(ref), np.abs(e).max() / np.sqrt((ref * ref).mean())
        print(f"layer {l}: {rel:.2e} {worst:.2e}")
        assert rel < 1.2e-6 and worst < 1.2e-5, f"layer {l}: {rel:.2e}, largest {worst:.2e}"
    g.close()
