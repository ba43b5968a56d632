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
