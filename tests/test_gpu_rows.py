"""The row gather behind stgn_get_embeddings: every piece width it chooses (16, 8 and 4 bytes, by row width and by the
caller's alignment), list lengths around its workgroup's share, repeated and unknown ids -- byte for byte."""
import ctypes as C

import numpy as np
import pytest

from paper_2603_21090_amd import synth
from tests.helpers import tiny_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_emb", [1, 7, 50, 62, 100, 252])
def test_rows_in_every_piece_width(d_emb):
    import torch
    from paper_2603_21090_amd import binding
    w = tiny_workload(d_emb=d_emb, heads=1, num_nodes=300, num_edges=900, batch=300)
    g = binding.StreamTGN.from_workload(w, synth.make_weights(w))
    st = synth.EdgeStream(w)
    for b in range(w.num_batches):
        g.ingest_batch(*st.batch(b))
    table = np.stack([g.get_embeddings(np.array([v], dtype=np.uint32))[0] for v in range(w.num_nodes)])
    gen = np.random.default_rng(d_emb)
    per = max(8, 8192 // d_emb)                                    # at least a workgroup's share of a long list
    for n in (1, 2, 7, 8, 9, 63, per - 1, per, per + 1, 20_011, 2048 * per + 5 if d_emb >= 100 else 40_000):
        ids = gen.integers(0, w.num_nodes, n).astype(np.int32)
        ids[n // 2] = -1                                           # past the node count: a row of NaN
        dev = torch.from_numpy(ids).cuda()
        want = torch.from_numpy(table).cuda()[dev.clamp(min=0).long()]
        want[n // 2] = float("nan")
        for shift in (0, 1, 2):                                    # 16-, 4- and 8-byte aligned results
            buf = torch.full((n * d_emb + 8,), 7.0, device="cuda")
            rc = g._L.stgn_get_embeddings(g._h, 0, n, C.c_void_p(dev.data_ptr()), C.c_void_p(buf.data_ptr() + 4 * shift), 1)
            assert rc == 0
            got = buf[shift:shift + n * d_emb].view(n, d_emb)
            assert torch.equal(got.nan_to_num(nan=-3.0), want.nan_to_num(nan=-3.0)), (n, shift)
            assert bool((buf[:shift] == 7.0).all()) and bool((buf[shift + n * d_emb:] == 7.0).all()), (n, shift)
    g.close()


@pytest.mark.parametrize("d_emb,n,shift", [(252, 8 * 65_536 + 3, 1), (252, 4 * 8 * 65_536, 1), (1, 2 ** 32 - 5, 0)])
def test_lists_longer_than_the_largest_grid(d_emb, n, shift):
    """Eight rows per workgroup and 65,536 workgroups, by three rows and several times over; and a list whose length and the
    rows of a workgroup do not add up in 32 bits (34 GB of ids and results)."""
    import torch
    from paper_2603_21090_amd import binding
    w = tiny_workload(d_emb=d_emb, heads=1, num_nodes=300, num_edges=900, batch=300)
    g = binding.StreamTGN.from_workload(w, synth.make_weights(w))
    st = synth.EdgeStream(w)
    for b in range(w.num_batches):
        g.ingest_batch(*st.batch(b))
    table = g.get_embeddings(torch.arange(w.num_nodes, dtype=torch.int32, device="cuda"))
    step = (1 << 26) // d_emb
    ids = torch.empty(n, dtype=torch.int32, device="cuda")
    for lo in range(0, n, step):
        ids[lo:lo + step].random_(0, w.num_nodes)
    buf = torch.full((n * d_emb + 2,), 7.0, device="cuda")
    rc = g._L.stgn_get_embeddings(g._h, 0, n, C.c_void_p(ids.data_ptr()), C.c_void_p(buf.data_ptr() + 4 * shift), 1)
    assert rc == 0 and g.sync() == 0
    got = buf[shift:shift + n * d_emb].view(n, d_emb)
    for lo in range(0, n, step):
        assert torch.equal(got[lo:lo + step], table[ids[lo:lo + step].long()]), lo
    assert bool((buf[:shift] == 7.0).all()) and bool((buf[shift + n * d_emb:] == 7.0).all())
    g.close()
    del ids, buf, got
    torch.cuda.empty_cache()


@pytest.mark.parametrize("k", [1, 10, 11, 12, 20, 21, 22, 23, 24, 32, 33, 43, 44, 64])
@pytest.mark.parametrize("d_mem", [0, 16])
def test_regrouped_rows_equal_a_rebuild(k, d_mem):
    """Row lists regrouped by entry count, at the list lengths on both sides of each variant of the regrouping kernel (11 | 12
    and 21 | 22 where the query cache doubles the bins, up to 32; 23 | 24 for a rebuild's list and 43 | 44 past the cache)
    and with a last window of a few rows: an incremental row is the row a rebuild computes, byte for byte, so a row
    dropped, doubled or marked as unchanged by mistake shows."""
    import torch
    from paper_2603_21090_amd import binding
    w = tiny_workload(num_nodes=36_869, num_edges=24_000, batch=2_000, k=k, d_mem=d_mem, d_node=0 if d_mem else 16, zipf_s=0.9)
    nf = None if d_mem else np.random.default_rng(k).standard_normal((w.num_nodes, 16), dtype=np.float32)
    g = binding.StreamTGN.from_workload(w, synth.make_weights(w), nf)
    st = synth.EdgeStream(w)
    ids = torch.arange(w.num_nodes, dtype=torch.int32, device="cuda")
    for b in range(w.num_batches):
        g.ingest_batch(*st.batch(b))
        if b % 4 == 3:
            rows = [g.get_embeddings(ids, layer=l) for l in range(1, w.layers + 1)]
            g.full_rebuild()
            for l, r in enumerate(rows):
                assert torch.equal(r, g.get_embeddings(ids, layer=l + 1)), (b, l + 1)
    g.close()


@pytest.mark.parametrize("n", [1, 7, 8, 9, 31, 32, 33, 41, 130])
@pytest.mark.parametrize("aggregator", [1, 2])
def test_aggregated_messages_of_a_hub(n, aggregator):
    """Mean and Sum over n slots of one node in one batch, around the slots looked up ahead (32) and requested together (8),
    against the oracle (the embedding bar of 1e-4 per row)."""
    from oracle import oracle as orc
    from paper_2603_21090_amd import binding
    w = tiny_workload(num_nodes=300, num_edges=600, batch=150, aggregator=aggregator)
    W = synth.make_weights(w)
    o, g = orc.Oracle.from_workload(w, W), binding.StreamTGN.from_workload(w, W)
    gen = np.random.default_rng(n)
    hub = 17
    for b in range(3):
        other = gen.permutation(np.delete(np.arange(w.num_nodes), hub))[:n].astype(np.uint32)
        side = gen.random(n) < 0.5
        src, dst = np.where(side, hub, other).astype(np.uint32), np.where(side, other, hub).astype(np.uint32)
        ts = 10.0 * b + np.sort(gen.random(n))
        ef = gen.standard_normal((n, w.d_edge), dtype=np.float32)
        assert o.ingest(src, dst, ts, ef)[0] == 0
        g.ingest_batch(src, dst, ts, ef)
        ref = o.embed_all()
        ids = np.arange(w.num_nodes, dtype=np.uint32)
        for l in range(w.layers):
            got = g.get_embeddings(ids, layer=l + 1)
            err = np.linalg.norm(got - ref[l], axis=1) / (np.linalg.norm(ref[l], axis=1) + 1e-30)
            assert err.max() <= 1e-4, (b, l, err.max())
    g.close()


def test_rows_of_one_slot_do_the_work_of_one():
    """Mean over 1,000 rows: with one slot a row takes one cosine and one load per column, with eight it takes eight.  The launches
    were 31 and 41 us; 38 and 40 when every row went through eight places, 35 and 97 one slot at a time."""
    import torch
    from paper_2603_21090_amd import binding
    rows, best = 1_000, {}
    for slots in (1, 8):
        n = rows * slots // 2
        w = tiny_workload(num_nodes=60_000, num_edges=200_000, batch=n, k=10, layers=1, d_mem=100, d_edge=172, d_time=100,
                          d_emb=100, d_msg=100, aggregator=1)
        g = binding.StreamTGN.from_workload(w, synth.make_weights(w), max_edges=24 * n)
        gen, us = np.random.default_rng(slots), []
        for b in range(24):
            ends = np.repeat(gen.permutation(w.num_nodes)[:rows].astype(np.int32), slots)
            batch = (ends[:n], ends[n:], b + np.sort(gen.random(n)), gen.standard_normal((n, w.d_edge), dtype=np.float32))
            batch = [torch.from_numpy(x.copy()).cuda() for x in batch]
            torch.cuda.synchronize()
            g.kernel_times(enable=True, reset=True)
            g.ingest_batch(*batch)
            g.sync()
            us.append(g.kernel_times(enable=False, reset=True)["memory_update"]["usec"])
        best[slots] = min(us)
        g.close()
    assert best[1] <= 0.87 * best[8], best


@pytest.mark.parametrize("d_emb", [1, 62, 100, 252])
def test_scores_at_edge_time_around_a_tile(d_emb):
    """A tile of the layer kernel holds eight edges: calls of other sizes give the same scores byte for byte, an id past the node
    count on either side scores NaN alone, and a score is the head applied to the two rows."""
    import torch
    from paper_2603_21090_amd import binding
    w = tiny_workload(d_emb=d_emb, heads=1, num_nodes=300, num_edges=900, batch=300)
    g = binding.StreamTGN.from_workload(w, synth.make_weights(w))
    st = synth.EdgeStream(w)
    for b in range(w.num_batches):
        g.ingest_batch(*st.batch(b))
    gen = np.random.default_rng(d_emb)
    head = gen.standard_normal(2 * d_emb, dtype=np.float32)
    g.set_predictor(head, 0.5)
    # both ends queried at their own last-interaction time: the cached rows are the answer
    _, last = g.get_memory(np.arange(w.num_nodes, dtype=np.uint32))
    s, d = st.src[-40:].astype(np.int64), st.dst[-40:].astype(np.int64)
    rows = g.get_embeddings(np.arange(w.num_nodes, dtype=np.uint32)).astype(np.float64)
    src, dst = (torch.from_numpy(x.astype(np.int32)).cuda() for x in (s, d))
    ts = torch.from_numpy(last[s]).cuda()
    all_ = g.predict_batch(src, dst, ts, at_edge_time=True)
    same = last[s] == last[d]
    want = rows[s] @ head[:d_emb].astype(np.float64) + rows[d] @ head[d_emb:].astype(np.float64) + 0.5
    scale = np.linalg.norm(rows[s], axis=1) * np.linalg.norm(head[:d_emb]) + np.linalg.norm(rows[d], axis=1) * np.linalg.norm(head[d_emb:])
    assert same.any()
    # fp32 sum of 2 d products: at most 2 d roundings of 2^-24 of their absolute sum, which the two norms bound
    assert (np.abs(all_.cpu().numpy() - want)[same] <= (2 * d_emb + 2) * 2.0 ** -24 * (scale[same] + 0.5)).all()
    for n in (1, 7, 8, 9, 15, 16, 17, 40):
        assert torch.equal(g.predict_batch(src[:n].clone(), dst[:n].clone(), ts[:n].clone(), at_edge_time=True), all_[:n]), n
    bad_s, bad_d = src.clone(), dst.clone()
    bad_s[7] = -1
    bad_d[8] = w.num_nodes
    got = g.predict_batch(bad_s, bad_d, ts, at_edge_time=True)
    assert torch.isnan(got[7:9]).all() and torch.equal(got[:7], all_[:7]) and torch.equal(got[9:], all_[9:])
    g.close()


@pytest.mark.parametrize("d_emb", [7, 100])
def test_rows_to_host_arrays(d_emb):
    """Host lists on both sides of the pinned block (1 MiB of ids and rows), against the device call."""
    import torch
    from paper_2603_21090_amd import binding
    w = tiny_workload(d_emb=d_emb, heads=1, num_nodes=300, num_edges=900, batch=300)
    g = binding.StreamTGN.from_workload(w, synth.make_weights(w))
    st = synth.EdgeStream(w)
    for b in range(w.num_batches):
        g.ingest_batch(*st.batch(b))
    gen = np.random.default_rng(d_emb)
    edge = ((1 << 20) - 16) // (4 + 4 * d_emb)
    for n in (1, 3, 333, edge - 1, edge, edge + 1, 2 * edge + 5):
        ids = gen.integers(0, w.num_nodes, n).astype(np.uint32)
        want = g.get_embeddings(torch.from_numpy(ids.astype(np.int32)).cuda()).cpu().numpy()
        assert np.array_equal(g.get_embeddings(ids), want), n
    g.close()


def test_rows_despite_an_error_left_behind():
    """An error that an earlier call of the program left with the runtime is not this call's: rows to a host array (short list and
    long) and to the device come as they do without it."""
    import torch
    from paper_2603_21090_amd import binding
    w = tiny_workload(num_nodes=300, num_edges=900, batch=300)
    g = binding.StreamTGN.from_workload(w, synth.make_weights(w))
    st = synth.EdgeStream(w)
    for b in range(w.num_batches):
        g.ingest_batch(*st.batch(b))
    long_ = (1 << 20) // (4 * w.d_emb) + 1
    for n in (5, long_):
        ids = np.arange(n, dtype=np.uint32) % w.num_nodes
        dev = torch.from_numpy(ids.astype(np.int32)).cuda()
        want = g.get_embeddings(dev).cpu().numpy()
        host, rows = np.empty((n, w.d_emb), dtype=np.float32), torch.empty((n, w.d_emb), device="cuda")
        for out, nodes, on_device in ((host.ctypes.data, ids.ctypes.data, 0), (rows.data_ptr(), dev.data_ptr(), 1)):
            assert g._L.hipSetDevice(4096) != 0 and g._L.hipPeekAtLastError() != 0
            rc = g._L.stgn_get_embeddings(g._h, 0, n, C.c_void_p(nodes), C.c_void_p(out), on_device)
            g._L.hipGetLastError()
            assert rc == 0, (n, on_device, g.last_error())
        assert np.array_equal(host, want) and np.array_equal(rows.cpu().numpy(), want)
    g.close()
