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
