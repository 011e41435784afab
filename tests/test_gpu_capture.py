"""Calls captured in a HIP graph, in every form that their rules choose between:
three replays, with eager calls on the same buffers and a synchronisation
between them, each bitwise equal to the eager result."""
import numpy as np
import pytest
import torch

from paper_2607_25422_amd import workloads as wls

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2607_25422_amd import binding
    return binding


def check_replays(call):
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        want = [t.clone() for t in call()]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        out = call()
    for r in range(3):
        for t in out:
            t.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for x, y in zip(out, want):
            assert torch.equal(x, y), f"replay {r}"
        with torch.cuda.stream(s):
            for x, y in zip(call(), want):             # eager work between replays
                assert torch.equal(x, y), f"eager call after replay {r}"
        torch.cuda.synchronize()


@pytest.mark.parametrize("name,n_q", [("tiny_fp32", 4), ("llava_bf16", 3), ("llava_bf16", 9)])
def test_capture_two_stages(B, name, n_q):
    """float32 and small bf16 by row tiles, 9 questions by the sparse kernel."""
    db = B.to_device(wls.make_batch(name, 3, B=n_q))

    def call():
        idx, scores, rows = B.prune_topk(db)
        O, L, rp, col = B.bipartite_xattn(db, rows.view(-1, db.p.H, db.p.d_h))
        return idx, scores, rows, O, L, rp, col[:4 * db.p.total_kept]
    check_replays(call)


@pytest.mark.parametrize("k,n_iter", [(96, 10), (96, 2)])
def test_capture_regions(B, k, n_iter):
    """Gram matrix; a launch per step."""
    batch = wls.make_batch("llava_bf16", 3, B=3, k=(k,))
    db = B.to_device(batch)
    rows = torch.cat([batch.V[b, :k] for b in range(batch.B)]).contiguous().cuda()
    ws = torch.empty(B.workspace_bytes_regions(db.p, 8), dtype=torch.uint8, device="cuda")
    check_replays(lambda: B.region_kmeans(db, rows, n_iter=n_iter, workspace=ws))


@pytest.mark.parametrize("M,d,d_out", [(97, 1024, 256), (97, 64, 256), (192, 2048, 65536)])
def test_capture_projection(B, M, d, d_out):
    """The split contraction, 96-row tiles after packing, 192-row tiles."""
    g = torch.Generator(device="cuda").manual_seed(2)
    V = torch.randn(1, M, d, generator=g, device="cuda").bfloat16()
    W = (torch.randn(d_out, d, generator=g, device="cuda") / d ** 0.5).bfloat16()
    ko = np.array([0, M], dtype=np.int32)
    p = B.make_problem("bf16", B=1, N=M, d=d, H=1, d_h=d, avg_degree=4.0, sm_scale=1.0,
                       kept_offsets=ko)
    kd = torch.from_numpy(ko).cuda()
    db = B.DeviceBatch(p=p, V=V, Qtok=V, q_offsets=kd, kept_offsets=kd, Kh=V, Vh=V,
                       passage_offsets=kd, query_passages=kd, w_bias=None, workspace=V)
    ws = torch.empty(B.workspace_bytes_project(p, d_out), dtype=torch.uint8, device="cuda")
    check_replays(lambda: (B.gather_project(db, V[0], W, workspace=ws),))
