"""GPU parity of the row-tile attention (float32, and small bf16 problems) at
the edges of its tiles: 16-row tiles (fewer rows than one, a whole one, one
row more), token blocks of 16 (float32) and 32 (bf16) tokens (passages of one
token to one more than a block), fewer blocks than waves, both widths of the
float32 workgroup, rows without neighbours and a negative scale; bf16 also on
both sides of the rule that chooses the kernel.

Bars: float32 1e-5 of max(|y|, RMS(y)), as for the other float32 cases.  bf16
with float32 output: products of bf16 values are exact, the weights enter as
bf16 pairs (2^-16 relative) and |v| < 5.5 here, so an output, a weighted mean
of values, is off by less than 2^-16 * 5.5 = 8.4e-5 plus float32 rounding:
1.2e-4 absolute."""
import math

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2607_25422_amd import workloads as wls

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d_h", [64, 128])
@pytest.mark.parametrize("B,H,k,P,L_p,scale", [
    (2, 2, (1, 15), (1, 2), (1, 15), 0.125),            # less than a tile, less than a block
    (3, 3, (16, 17), (3,), (16, 17, 32, 33), 0.125),    # a whole tile and one row more
    (1, 4, (33,), (20,), (5, 40), -0.2),                # few rows of many passages; negative scale
    (12, 16, (47, 64), (5,), (31, 64), 0.125),          # 768 workgroups: the bf16 rule's line
    (13, 16, (47, 64), (5,), (31, 64), 0.125),          # past it
    (40, 8, (47, 64), (4, 5), (1, 31, 48), 0.125),      # 1280 workgroups: four waves each (f32)
    (8, 16, (47, 64), (3,), (257, 31), 0.125),          # 512 workgroups: the rule's line past 256 tokens
    (9, 16, (47, 64), (3,), (257, 31), 0.125),          # past it
])
def test_attn_tile_edges(B, H, k, P, L_p, scale, d_h, dtype):
    from paper_2607_25422_amd import binding as bnd
    batch = wls.make_batch("tiny_fp32" if dtype == "f32" else "llava_bf16", 29, B=B, N=128, H=H,
                           d_h=d_h, T=(4,), k=k, P=P, L_p=L_p)
    rng = np.random.default_rng(3)
    adj = [rng.random((int(a), int(b))) < 0.3 for a, b in zip(batch.k, batch.P)]
    adj[0][0] = False                                   # a row without neighbours
    rp, col = [0], []
    for row in (r for a in adj for r in a):
        col.extend(np.nonzero(row)[0].tolist())
        rp.append(len(col))
    Qh = torch.cat([batch.V[b, :int(n)] for b, n in enumerate(batch.k)]).view(-1, H, d_h)
    if dtype == "bf16":                                 # N(0, 1/d) tokens to order one
        Qh = (Qh.float() * math.sqrt(H * d_h)).bfloat16()
    db = bnd.to_device(batch, sm_scale=scale, o_f32=True)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")  # noqa: E731
    O, L, _, _ = bnd.bipartite_xattn(db, Qh.contiguous().cuda(), edges=(i32(rp), i32(col)))
    _, _, O_ref, L_ref = orc.bipartite_xattn(
        Qh, batch.kept_offsets, batch.Kh, batch.Vh, batch.passage_offsets,
        batch.query_passages, scale, adjacency=adj)
    O, L = O.cpu().double().numpy(), L.cpu().double().numpy()
    O_ref, L_ref = np.concatenate(O_ref), np.concatenate(L_ref)
    live = np.isfinite(L_ref)
    assert np.array_equal(live, np.isfinite(L)) and not live[0].any()
    assert np.all(L[~live] == -math.inf) and np.all(O[~live] == 0)
    if dtype == "f32":
        rms = math.sqrt(np.mean(O_ref[live] ** 2))
        assert np.max(np.abs(O - O_ref) / np.maximum(np.abs(O_ref), rms)) <= 1e-5
    else:
        assert batch.Vh.abs().max() < 5.5
        assert np.max(np.abs(O - O_ref)) <= 1.2e-4
    assert np.max(np.abs(L[live] - L_ref[live]) / np.maximum(1.0, np.abs(L_ref[live]))) <= 1e-5


def run_given_graph(bnd, batch, Qh, adj, H, scale):
    rp, col = [0], []
    for row in (r for a in adj for r in a):
        col.extend(np.nonzero(row)[0].tolist())
        rp.append(len(col))
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")  # noqa: E731
    db = bnd.to_device(batch, sm_scale=scale, o_f32=True)
    O, L, _, _ = bnd.bipartite_xattn(db, Qh.contiguous().cuda(), edges=(i32(rp), i32(col)))
    return O.cpu().double().numpy(), L.cpu().double().numpy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d_h", [64, 128])
def test_attn_tile_values_reach_only_adjacent_rows(d_h, dtype):
    """An infinity and a NaN among the values of two passages: rows without an
    edge to them keep the result of finite values (the bars of the tile tests),
    rows with one get the infinity (in the last token, which pads its block) or
    the NaN, in that feature alone."""
    from paper_2607_25422_amd import binding as bnd
    H = 3
    batch = wls.make_batch("tiny_fp32" if dtype == "f32" else "llava_bf16", 31, B=2, N=128, H=H,
                           d_h=d_h, T=(4,), k=(33, 20), P=(5,), L_p=(5, 17, 300))
    rng = np.random.default_rng(4)
    adj = [rng.random((int(a), int(b))) < 0.4 for a, b in zip(batch.k, batch.P)]
    Qh = torch.cat([batch.V[b, :int(n)] for b, n in enumerate(batch.k)]).view(-1, H, d_h)
    if dtype == "bf16":
        Qh = (Qh.float() * math.sqrt(H * d_h)).bfloat16()
    _, _, O_ref, _ = orc.bipartite_xattn(
        Qh, batch.kept_offsets, batch.Kh, batch.Vh, batch.passage_offsets,
        batch.query_passages, 0.125, adjacency=adj)
    ref = np.concatenate(O_ref)
    at = batch.passage_offsets
    Vh = batch.Vh.clone()
    Vh[int(at[2]) - 1, 1, 3] = math.inf               # question 0, passage 1, its last token
    Vh[int(at[5 + 3]), 2, d_h - 1] = math.nan         # question 1, passage 3, its first
    batch.Vh = Vh
    O, L = run_given_graph(bnd, batch, Qh, adj, H, 0.125)
    k0 = int(batch.k[0])
    inf_rows, nan_rows = np.nonzero(adj[0][:, 1])[0], k0 + np.nonzero(adj[1][:, 3])[0]
    assert 0 < len(inf_rows) < k0 and 0 < len(nan_rows) < int(batch.k[1])
    got = O[inf_rows, 1, 3]                           # (bf16: an infinity times a low part of 0 is no number)
    assert np.all(got == math.inf) if dtype == "f32" else not np.isfinite(got).any()
    assert np.all(np.isnan(O[nan_rows, 2, d_h - 1]))
    O[inf_rows, 1, 3] = ref[inf_rows, 1, 3]
    O[nan_rows, 2, d_h - 1] = ref[nan_rows, 2, d_h - 1]
    if dtype == "f32":
        rms = math.sqrt(np.mean(ref ** 2))
        assert np.max(np.abs(O - ref) / np.maximum(np.abs(ref), rms)) <= 1e-5
    else:
        assert np.max(np.abs(O - ref)) <= 1.2e-4


def test_attn_tile_large_values_do_not_overflow():
    """A value of 3e37 under a weight that the softmax's reference maximum, as
    the wave first meets it, would make 55: the weighted mean, 8.3e36, is far
    inside the range."""
    from paper_2607_25422_amd import binding as bnd
    batch = wls.make_batch("tiny_fp32", 1, B=1, N=128, H=1, d_h=64, T=(4,), k=(17,), P=(1,),
                           L_p=(144,))
    Qh = torch.zeros(17, 1, 64)
    Qh[:, 0, 0] = 1.0
    batch.Kh = torch.zeros_like(batch.Kh)
    batch.Vh = torch.zeros_like(batch.Vh)
    batch.Kh[128, 0, 0] = 4.0                          # a later block of the first wave
    batch.Vh[128, 0, 5] = 3e37
    O, _ = run_given_graph(bnd, batch, Qh, [np.ones((17, 1), dtype=bool)], 1, 1.0)
    want = 3e37 * math.exp(4.0) / (143 + math.exp(4.0))
    assert np.all(np.abs(O[:, 0, 5] / want - 1) <= 1e-5)
    O[:, 0, 5] = 0
    assert np.all(O == 0)


def test_attn_tile_more_workgroups_than_a_row_of_the_grid():
    """33 000 questions of one row and 128 heads make 4.2 million workgroups,
    more than one dimension of a launch holds: the last question of the first
    row of the grid and the ones beside it, the first and the last have a
    passage of one token, whose value is their result; the others have none."""
    from paper_2607_25422_amd import binding as bnd
    B, H, d_h = 33000, 128, 64
    at = [0, 2 ** 15 - 1, 2 ** 15, B - 1]             # 2^22 workgroups a row: 2^15 questions
    P = np.zeros(B, dtype=np.int64)
    P[at] = 1
    offs = dict(q_offsets=np.arange(B + 1), kept_offsets=np.arange(B + 1),
                passage_offsets=np.arange(len(at) + 1),
                query_passages=np.concatenate([[0], np.cumsum(P)]))
    offs = {n: a.astype(np.int32) for n, a in offs.items()}
    p = bnd.make_problem("f32", B=B, N=1, d=H * d_h, H=H, d_h=d_h, avg_degree=1.0, sm_scale=0.125,
                         o_f32=True, edge_rule="question", edge_metric="cosine", **offs)
    dev = {n: torch.from_numpy(a).cuda() for n, a in offs.items()}
    g = torch.Generator(device="cuda").manual_seed(1)
    Kh, Vh = (torch.randn(len(at), H, d_h, generator=g, device="cuda") for _ in range(2))
    Qh = torch.ones(B, H, d_h, device="cuda")
    db = bnd.DeviceBatch(p=p, V=Qh.view(B, 1, -1), Qtok=Qh.view(B, -1), q_offsets=dev["q_offsets"],
                         kept_offsets=dev["kept_offsets"], Kh=Kh, Vh=Vh,
                         passage_offsets=dev["passage_offsets"],
                         query_passages=dev["query_passages"], w_bias=None,
                         workspace=bnd.new_workspace(p, "cuda"))
    edges = (dev["query_passages"], torch.zeros(len(at), dtype=torch.int32, device="cuda"))
    O, L, _, _ = bnd.bipartite_xattn(db, Qh, edges=edges)
    assert torch.equal(O[at], Vh)
    want = 0.125 * Kh.double().sum(2)
    assert float((L[at].double() - want).abs().max()) <= 1e-5 * (1 + float(want.abs().max()))
    O[at] = 0
    assert not bool(O.any()) and int(torch.isneginf(L).sum()) == (B - len(at)) * H
