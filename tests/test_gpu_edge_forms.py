"""The two forms of the edge selection (candidate keys formed by the selection
itself, or by a launch of their own) on either side of the line between them,
the CSR of many questions, and the pooling launch at the edges of its batches
of rows: graphs and kept sets exact against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle as orc

from test_gpu_parity import (B, check_attention, check_graph, f64,  # noqa: F401
                             queries_from_batch, say, small_batch)
from test_gpu_regions import kept_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("metric", ["cosine", "dot"])
@pytest.mark.parametrize("dtype,H,d_h,k,P,n_q", [
    ("bf16", 4, 64, (128,), 8, 2),       # 1024 candidates, one a thread
    ("bf16", 4, 64, (129,), 8, 2),       # 1032: the key launch
    ("f32", 32, 64, (40, 7), 5, 2),           # d = 2048, 8 slices
    ("f32", 33, 64, (40, 7), 5, 2),           # 9 slices: the key launch
    ("bf16", 2, 128, (3, 1, 0), 2, 70),       # CSR offsets of 70 questions
])
def test_edge_selection_forms(B, dtype, H, d_h, k, P, n_q, metric):  # noqa: F811
    batch = small_batch(dtype, 5, B=n_q, H=H, d_h=d_h, P=(P,), L_p=(1, 9), k=k)
    say(f"edge forms {dtype} d={H * d_h} k={k} P={P} {metric}")
    db = B.to_device(batch, avg_degree=1.5, edge_metric=metric)
    Qh = queries_from_batch(batch)
    O, L, rp, col = B.bipartite_xattn(db, Qh.cuda())
    torch.cuda.synchronize()
    _, adj, O_ref, L_ref = orc.bipartite_xattn(
        Qh, batch.kept_offsets, batch.Kh, batch.Vh, batch.passage_offsets,
        batch.query_passages, batch.wl.scale, 1.5, edge_metric=metric)
    check_graph(batch, rp, col, adj)
    check_attention(f64(O), f64(L), np.concatenate(O_ref), np.concatenate(L_ref), dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows", [(1, 4, 5), (28, 29, 31), (32, 33, 61)])
def test_pooling_batches_of_rows(B, dtype, rows):  # noqa: F811
    """Questions and passages of so many rows: four waves take them in rounds
    of eight rows each."""
    batch = small_batch(dtype, 8, B=6, T=rows, L_p=rows, P=(2, 3), k=(1, 17, 40))
    say(f"pooling {dtype} rows={rows}")
    db = B.to_device(batch, avg_degree=1.5)
    idx = B.prune_topk(db, want_scores=False, want_rows=False)[0].cpu().numpy()
    kept = kept_oracle(batch)
    for b in range(batch.B):
        k0, k1 = batch.kept_offsets[b], batch.kept_offsets[b + 1]
        assert idx[k0:k1].tolist() == list(kept[b]), f"q{b} kept set"
    Qh = queries_from_batch(batch)
    _, _, rp, col = B.bipartite_xattn(db, Qh.cuda())
    torch.cuda.synchronize()
    _, adj, _, _ = orc.bipartite_xattn(
        Qh, batch.kept_offsets, batch.Kh, batch.Vh, batch.passage_offsets,
        batch.query_passages, batch.wl.scale, 1.5)
    check_graph(batch, rp, col, adj)


@pytest.mark.parametrize("dtype,d", [("bf16", 8), ("bf16", 512), ("bf16", 520), ("bf16", 2568),
                                     ("f32", 8), ("f32", 256), ("f32", 264), ("f32", 1288)])
def test_gather_short_and_long_rows(B, dtype, d):  # noqa: F811
    """Four rows a wave (up to 64 chunks of 16 bytes a row) or one: rows of one
    chunk to one more than a whole batch, counts about the rows of a workgroup."""
    batch = small_batch(dtype, 6, B=6, N=64, H=d // 8, d_h=8, k=(1, 3, 4, 5, 16, 17), P=(1,),
                        L_p=(1,))
    say(f"gather {dtype} d={d} k={batch.k.tolist()}")
    db = B.to_device(batch)
    idx, _, rows = B.prune_topk(db, want_scores=False)
    idx, rows = idx.cpu().long(), rows.cpu()
    for b in range(batch.B):
        k0, k1 = int(batch.kept_offsets[b]), int(batch.kept_offsets[b + 1])
        assert torch.equal(rows[k0:k1], batch.V[b][idx[k0:k1]]), f"q{b}"
