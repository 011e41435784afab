"""GPU parity of the passage-major sparse attention (bf16 problems past the
row-tile rule): one to several chunks of 192 rows, one or two blocks of 16 rows a
wave, passages of less than a tile to several, one-tile passages in a row (rows
change waves from one passage's blocks to the next's), a negative scale, and the
fused route's rows read through the kept indices.  Bars as in the other bf16
cases: graphs exact, attention by check_attention."""
import ctypes
import math

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2607_25422_amd import workloads as wls

from test_gpu_parity import (B, check_attention, check_graph, f64,  # noqa: F401
                             queries_from_batch, say)

pytestmark = pytest.mark.gpu


def past_the_tiles(k, d_h):
    """(questions, heads) that put k rows a question past the row tiles."""
    need = 49152 // ((k + 15) // 16 * d_h) + 1
    H = min(-(-need // 3), 4096 // d_h)
    return -(-need // H), H


def by_tiles(B, p):  # noqa: F811
    f = B.LIB["_ZN4skip13attn_by_tilesERK12skip_problem"]
    f.restype = ctypes.c_bool
    return f(ctypes.byref(p))


def run(B, batch, scale, degree):  # noqa: F811
    Qh = queries_from_batch(batch)
    _, adj, O_ref, L_ref = orc.bipartite_xattn(
        Qh, batch.kept_offsets, batch.Kh, batch.Vh, batch.passage_offsets,
        batch.query_passages, scale, degree)
    O_ref, L_ref = np.concatenate(O_ref), np.concatenate(L_ref)
    for f32_out in (False, True):
        db = B.to_device(batch, sm_scale=scale, avg_degree=degree, o_f32=f32_out)
        assert not by_tiles(B, db.p)
        O, L, rp, col = B.bipartite_xattn(db, Qh.cuda())
        torch.cuda.synchronize()
        check_graph(batch, rp, col, adj)
        check_attention(f64(O), f64(L), O_ref, L_ref, "bf16", f"f32out={f32_out}",
                        stored_bf16=not f32_out)


@pytest.mark.parametrize("d_h", [64, 128])
@pytest.mark.parametrize("k", [1, 17, 96, 97, 129, 192, 193, 300, 385, 500])
def test_sparse_row_layouts(B, k, d_h):  # noqa: F811
    n_q, H = past_the_tiles(k, d_h)
    batch = wls.make_batch("llava_bf16", 7, B=n_q, N=520, H=H, d_h=d_h, T=4, k=(k,), P=(2, 4),
                           L_p=(31, 64, 100))
    say(f"sparse layouts k={k} d_h={d_h} B={n_q} H={H} P={batch.P.tolist()}")
    run(B, batch, batch.wl.scale, 2.0)


@pytest.mark.parametrize("d_h", [64, 128])
def test_sparse_negative_scale_and_one_tile_passages(B, d_h):  # noqa: F811
    n_q, H = past_the_tiles(193, d_h)
    batch = wls.make_batch("llava_bf16", 8, B=n_q, N=520, H=H, d_h=d_h, T=4, k=(193, 60),
                           P=(16,), L_p=(1, 7, 32))
    say(f"sparse one-tile passages d_h={d_h} k={batch.k.tolist()}")
    run(B, batch, -0.2, 5.0)


@pytest.mark.parametrize("d_h", [64, 128])
def test_sparse_fused_route_reads_kept_rows(B, d_h):  # noqa: F811
    """The fused route (rows of V through the kept indices) and the two stages
    on the gathered rows: the same bits."""
    n_q, H = past_the_tiles(193, d_h)
    batch = wls.make_batch("llava_bf16", 9, B=n_q, N=520, H=H, d_h=d_h, T=(3, 9),
                           k=(193, 97), P=(5, 8), L_p=(40, 64))
    say(f"sparse fused d_h={d_h} k={batch.k.tolist()}")
    db = B.to_device(batch, o_f32=True)
    assert not by_tiles(B, db.p)
    idx, O, L = B.route_fused(db)
    idx2, _, rows = B.prune_topk(db, want_scores=False)
    O2, L2, _, _ = B.bipartite_xattn(db, rows.view(-1, H, d_h))
    torch.cuda.synchronize()
    assert torch.equal(idx, idx2) and torch.equal(O, O2) and torch.equal(L, L2)
    assert math.isfinite(float(O.abs().sum()))
