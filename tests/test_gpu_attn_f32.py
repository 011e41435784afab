"""GPU parity of the float32 attention at the edges of its tiles: 16-row
tiles (fewer rows than one, a whole one, one row more), 16-token blocks
(passages of one token to one more than a block), fewer blocks than waves,
both widths of workgroup, rows without neighbours and a negative scale.
Bars as for the other float32 cases: 1e-5 of max(|y|, RMS(y))."""
import math

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2607_25422_amd import workloads as wls

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_h", [64, 128])
@pytest.mark.parametrize("B,H,k,P,L_p,scale", [
    (2, 2, (1, 15), (1, 2), (1, 15), 0.125),            # less than a tile, less than a block
    (3, 3, (16, 17), (3,), (16, 17, 33), 0.125),        # a whole tile and one row more
    (1, 4, (33,), (20,), (5, 40), -0.2),                # few rows of many passages; negative scale
    (40, 8, (47, 64), (4, 5), (1, 31, 48), 0.125),      # 1280 workgroups: four waves each
])
def test_attn_f32_tile_edges(B, H, k, P, L_p, scale, d_h):
    from paper_2607_25422_amd import binding as bnd
    batch = wls.make_batch("tiny_fp32", 29, B=B, N=128, H=H, d_h=d_h, T=(4,), k=k, P=P, L_p=L_p)
    rng = np.random.default_rng(3)
    adj = [rng.random((int(a), int(b))) < 0.3 for a, b in zip(batch.k, batch.P)]
    adj[0][0] = False                                   # a row without neighbours
    rp, col = [0], []
    for row in (r for a in adj for r in a):
        col.extend(np.nonzero(row)[0].tolist())
        rp.append(len(col))
    Qh = torch.cat([batch.V[b, :int(n)] for b, n in enumerate(batch.k)]).view(-1, H, d_h)
    db = bnd.to_device(batch, sm_scale=scale)
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
    rms = math.sqrt(np.mean(O_ref[live] ** 2))
    assert np.max(np.abs(O - O_ref) / np.maximum(np.abs(O_ref), rms)) <= 1e-5
    assert np.max(np.abs(L[live] - L_ref[live]) / np.maximum(1.0, np.abs(L_ref[live]))) <= 1e-5
