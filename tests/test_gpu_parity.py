"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle
on the same seeded inputs.

Bars: kept-token sets and edge sets identical (selection is decided in
float64 on both sides); attention outputs within 1e-5 relative (fp32 mode,
max |y - y_ref| / max(|y_ref|, RMS(y_ref))) or 2e-2 of the output RMS (bf16
mode); rows without neighbours exactly zero with LSE = -inf.

bf16 mode is checked twice.  With float32 output (o_f32) the raw error must
be within 2e-2 x RMS.  With bf16 output the one rounding of each stored value
(at most 2^-8 of its magnitude) is allowed on top of that bar: a correctly
rounded bf16 value can already differ from the float64 result by more than
2e-2 x RMS when |O| exceeds a few times the RMS.
"""
import math
import sys

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2607_25422_amd import workloads as wls

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def B():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2607_25422_amd import binding
    return binding


# --------------------------------------------------------------------------- helpers

def f64(t):
    return t.detach().cpu().to(torch.float64).numpy()


def check_attention(O, L, O_ref, L_ref, dtype, tag="", stored_bf16=None):
    """O, O_ref: [n, H, d_h]; L, L_ref: [n, H] (float64 numpy).  In bf16
    mode ``stored_bf16`` says whether O was written as bf16 (default) or as
    float32."""
    if stored_bf16 is None:
        stored_bf16 = dtype != "f32"
    if O_ref.size == 0:
        return
    live = np.isfinite(L_ref).all(axis=1)
    dead = ~live
    assert np.all(O[dead] == 0), f"{tag}: rows without neighbours must be 0"
    assert np.all(np.isneginf(L[dead])), f"{tag}: rows without neighbours need LSE = -inf"
    if not live.any():
        return
    y, r = O[live], O_ref[live]
    rms = math.sqrt(float(np.mean(r * r)))
    if dtype == "f32":
        err = np.max(np.abs(y - r) / np.maximum(np.abs(r), rms))
        assert err <= 1e-5, f"{tag}: fp32 max relative error {err:.3e}"
        lerr = np.max(np.abs(L[live] - L_ref[live]) / np.maximum(1.0, np.abs(L_ref[live])))
        assert lerr <= 1e-5, f"{tag}: LSE error {lerr:.3e}"
    else:
        allow = (2.0 ** -8) * np.abs(r) if stored_bf16 else 0.0
        raw = np.max(np.abs(y - r)) / rms
        err = np.max(np.abs(y - r) - allow) / rms
        say(f"{tag}: bf16 max error {raw:.3e} x RMS raw, {err:.3e} beyond storage rounding")
        assert err <= 2e-2, f"{tag}: bf16 max error {err:.3e} x RMS"
        lerr = np.max(np.abs(L[live] - L_ref[live]) / np.maximum(1.0, np.abs(L_ref[live])))
        assert lerr <= 1e-3, f"{tag}: LSE error {lerr:.3e}"


def oracle_route(batch, **kw):
    return orc.route(batch.V, batch.Qtok, batch.q_offsets, batch.kept_offsets, batch.Kh,
                     batch.Vh, batch.passage_offsets, batch.query_passages, batch.wl.scale,
                     batch.wl.avg_degree, w_bias=batch.w_bias, **kw)


def sample_rows(batch, per_q, seed=0):
    rng = np.random.default_rng(seed)
    out = {}
    for b in range(batch.B):
        k = int(batch.k[b])
        out[b] = sorted(rng.choice(k, size=min(per_q, k), replace=False).tolist()) if k else []
    return out


def small_batch(dtype, seed, **kw):
    name = "tiny_fp32" if dtype == "f32" else "llava_bf16"
    base = dict(B=5, N=300, H=4, d_h=64, T=(1, 3, 8), k=(0, 7, 33, 64, 300),
                P=(0, 1, 3, 6), L_p=(1, 5, 64, 100))
    base.update(kw)
    return wls.make_batch(name, seed, **base)


def run_prune(B, batch):
    db = B.to_device(batch)
    idx, scores, rows = B.prune_topk(db)
    torch.cuda.synchronize()
    return db, idx.cpu().numpy(), scores.cpu().numpy(), rows.cpu()


# --------------------------------------------------------------------------- stage 1

@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("seed", wls.SEEDS)
def test_prune_small_ragged(B, dtype, seed):
    batch = small_batch(dtype, seed, with_bias=True)
    say(f"prune small {dtype} seed={seed} k={batch.k.tolist()}")
    db, idx, scores, rows = run_prune(B, batch)
    ref = oracle_route(batch, with_attention=False)
    for b in range(batch.B):
        k0, k1 = batch.kept_offsets[b], batch.kept_offsets[b + 1]
        assert idx[k0:k1].tolist() == ref.kept_idx[b].tolist(), f"question {b}"
        np.testing.assert_allclose(scores[b], ref.scores[b], rtol=1e-6, atol=1e-30)
        assert torch.equal(rows[k0:k1], batch.V[b][torch.from_numpy(ref.kept_idx[b])])


def test_prune_ties_lowest_index(B):
    # identical visual tokens score identically: the lowest indices must win
    batch = wls.make_batch("llava_bf16", 7, B=3, N=200, H=4, d_h=64, k=(5, 50, 199))
    V = batch.V.clone()
    V[:, 100:] = V[:, 0:100]          # every token duplicated 100 positions later
    V[1, :, :] = V[1, 0, :]           # question 1: all 200 tokens equal
    batch.V = V
    db, idx, _, _ = run_prune(B, batch)
    ref = oracle_route(batch, with_attention=False)
    for b in range(batch.B):
        k0, k1 = batch.kept_offsets[b], batch.kept_offsets[b + 1]
        assert idx[k0:k1].tolist() == ref.kept_idx[b].tolist()
    k0, k1 = batch.kept_offsets[1], batch.kept_offsets[2]
    assert idx[k0:k1].tolist() == list(range(k1 - k0))


@pytest.mark.parametrize("k", [100, 400])
@pytest.mark.parametrize("n_equal", [30, 200, 600])
def test_prune_tie_band_at_the_cut(B, n_equal, k):
    # n_equal tokens are made copies of the token ranked k - n_equal/2 (or of
    # the top token), so the k-th largest logit is shared by a band of equal
    # values on both sides of the cut, from a few to more than k of them: the
    # selection must take every logit above the band and the band's lowest
    # indices, as the oracle does.
    batch = wls.make_batch("llava_bf16", 11, B=3, N=1024, H=4, d_h=64, k=(k,))
    V = batch.V.clone()
    w = None if batch.w_bias is None else batch.w_bias.double().numpy()
    for b in range(batch.B):
        t0, t1 = int(batch.q_offsets[b]), int(batch.q_offsets[b + 1])
        q_bar = orc.mean_pool_question(batch.Qtok[t0:t1].double().numpy())
        z = orc.qvs_logits(V[b].double().numpy(), q_bar, w)
        order = np.argsort(-z, kind="stable")
        pivot = int(order[max(0, k - n_equal // 2)])
        V[b, torch.from_numpy(order[-n_equal:].copy())] = V[b, pivot].clone()   # lowest ranks become copies
    batch.V = V
    db, idx, _, _ = run_prune(B, batch)
    ref = oracle_route(batch, with_attention=False)
    for b in range(batch.B):
        k0, k1 = batch.kept_offsets[b], batch.kept_offsets[b + 1]
        assert idx[k0:k1].tolist() == ref.kept_idx[b].tolist(), f"question {b}"


@pytest.mark.parametrize("seed", wls.SEEDS)
@pytest.mark.parametrize("name", wls.ORDER)
def test_prune_named_full_size(B, name, seed):
    batch = wls.make_batch(name, seed, threads=16)
    say(f"prune {name} seed {seed} full size B={batch.B} N={batch.wl.N}")
    db, idx, scores, rows = run_prune(B, batch)
    ref = oracle_route(batch, with_attention=False)
    for b in range(batch.B):
        k0, k1 = batch.kept_offsets[b], batch.kept_offsets[b + 1]
        assert idx[k0:k1].tolist() == ref.kept_idx[b].tolist(), f"{name} question {b}"
        if batch.planted[b].size:
            kept = set(idx[k0:k1].tolist())
            pl = set(batch.planted[b].tolist())
            assert pl <= kept or kept <= pl, f"{name} q{b}: planted tokens lost"
    b = batch.B - 1
    np.testing.assert_allclose(scores[b], ref.scores[b], rtol=1e-6)


# --------------------------------------------------------------------------- stage 2

def queries_from_batch(batch):
    """Kept-row queries for the stand-alone graph + attention call: the first
    k_b visual tokens of each question viewed as [H, d_h]."""
    H, d_h = batch.Kh.shape[1], batch.Kh.shape[2]
    rows = [batch.V[b, :int(batch.k[b])] for b in range(batch.B)]
    return torch.cat(rows, 0).reshape(-1, H, d_h).contiguous()


def check_graph(batch, rp, col, adj_ref):
    rp = rp.cpu().numpy()
    col = col.cpu().numpy()
    for b in range(batch.B):
        k0 = int(batch.kept_offsets[b])
        want_rp, want_col = orc.adjacency_to_csr(adj_ref[b])
        got_rp = rp[k0:k0 + len(want_rp)] - rp[k0]
        assert got_rp.tolist() == want_rp.tolist(), f"question {b}: row pointers"
        got_col = col[rp[k0]:rp[k0] + len(want_col)]
        assert got_col.tolist() == want_col.tolist(), f"question {b}: columns"
    assert rp[-1] == sum(int(a.sum()) for a in adj_ref)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("seed", wls.SEEDS)
@pytest.mark.parametrize("deg", [4.0, 1.5])
def test_xattn_small_ragged(B, dtype, seed, deg):
    batch = small_batch(dtype, seed, H=2, d_h=128)
    say(f"xattn small {dtype} seed={seed} deg={deg} P={batch.P.tolist()}")
    db = B.to_device(batch, avg_degree=deg)
    Qh = queries_from_batch(batch)
    O, L, rp, col = B.bipartite_xattn(db, Qh.cuda())
    torch.cuda.synchronize()
    cos, adj, O_ref, L_ref = orc.bipartite_xattn(
        Qh, batch.kept_offsets, batch.Kh, batch.Vh, batch.passage_offsets,
        batch.query_passages, batch.wl.scale, deg)
    check_graph(batch, rp, col, adj)
    check_attention(f64(O), f64(L), np.concatenate(O_ref), np.concatenate(L_ref), dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_xattn_given_graph_and_keys(B, dtype):
    batch = small_batch(dtype, 11, B=4, k=(20, 64), P=(3, 7), L_p=(2, 70))
    H, d_h = batch.Kh.shape[1], batch.Kh.shape[2]
    db = B.to_device(batch)
    Qh = queries_from_batch(batch)
    rng = np.random.default_rng(5)
    adj = [rng.random((int(k), int(P))) < 0.4 for k, P in zip(batch.k, batch.P)]
    adj[0][0] = False                     # a row with no neighbour
    adj[1][1] = True                      # a row adjacent to every passage
    rp = [0]
    cols = []
    for a in adj:
        for row in a:
            cols.extend(np.nonzero(row)[0].tolist())
            rp.append(len(cols))
    edges = (torch.tensor(rp, dtype=torch.int32, device="cuda"),
             torch.tensor(cols, dtype=torch.int32, device="cuda"))
    O, L, _, _ = B.bipartite_xattn(db, Qh.cuda(), edges=edges)
    _, _, O_ref, L_ref = orc.bipartite_xattn(
        Qh, batch.kept_offsets, batch.Kh, batch.Vh, batch.passage_offsets,
        batch.query_passages, batch.wl.scale, adjacency=adj)
    check_attention(f64(O), f64(L), np.concatenate(O_ref), np.concatenate(L_ref), dtype, "csr")
    # caller-given passage keys replace the pooled keys
    keys = torch.randn(int(batch.query_passages[-1]), H * d_h, generator=torch.Generator().manual_seed(3))
    O2, L2, rp2, col2 = B.bipartite_xattn(db, Qh.cuda(), passage_keys=keys.cuda())
    _, adj2, O2_ref, L2_ref = orc.bipartite_xattn(
        Qh, batch.kept_offsets, batch.Kh, batch.Vh, batch.passage_offsets,
        batch.query_passages, batch.wl.scale, passage_key_table=keys.double())
    check_graph(batch, rp2, col2, adj2)
    check_attention(f64(O2), f64(L2), np.concatenate(O2_ref), np.concatenate(L2_ref), dtype, "keys")


# Kept-row counts about the edges of blocks of 16 and 32 rows and of chunks of
# rows.  (Two heads of three questions go by row tiles; the sparse kernel's
# layouts are in test_gpu_attn_sparse.py.)
ROW_COUNTS = (1, 31, 33, 64, 65, 129, 160, 161, 193, 224, 256, 300, 450, 512)


@pytest.mark.parametrize("d_h", [64, 128])
@pytest.mark.parametrize("k", ROW_COUNTS)
def test_xattn_row_block_layouts(B, k, d_h):
    batch = wls.make_batch("llava_bf16", 7, B=3, N=520, H=2, d_h=d_h, T=4, k=(k,),
                           P=(3, 5), L_p=(40, 64, 100))
    say(f"xattn layouts k={k} d_h={d_h} P={batch.P.tolist()}")
    Qh = queries_from_batch(batch)
    _, adj, O_ref, L_ref = orc.bipartite_xattn(
        Qh, batch.kept_offsets, batch.Kh, batch.Vh, batch.passage_offsets,
        batch.query_passages, batch.wl.scale, 2.0)
    O_ref, L_ref = np.concatenate(O_ref), np.concatenate(L_ref)
    for f32_out in (False, True):
        db = B.to_device(batch, avg_degree=2.0, o_f32=f32_out)
        O, L, rp, col = B.bipartite_xattn(db, Qh.cuda())
        torch.cuda.synchronize()
        check_graph(batch, rp, col, adj)
        check_attention(f64(O), f64(L), O_ref, L_ref, "bf16", f"k={k} f32out={f32_out}",
                        stored_bf16=not f32_out)


EDGE_VARIANTS = [("question", "dot", 0.1), ("row", "cosine", 0.1), ("row", "dot", 0.1),
                 ("fraction", "cosine", 0.1), ("fraction", "dot", 0.35)]


@pytest.mark.parametrize("rule,metric,beta", EDGE_VARIANTS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_xattn_edge_rules_and_metrics(B, rule, metric, beta, dtype):
    """The other edge cuts (per-row top, top fraction) and the scaled-dot
    compatibility: identical graphs, attention to the usual bar."""
    batch = small_batch(dtype, 42, H=2, d_h=128)
    say(f"xattn edges {rule}/{metric} beta={beta} {dtype} P={batch.P.tolist()} k={batch.k.tolist()}")
    db = B.to_device(batch, avg_degree=2.5, edge_rule=rule, edge_metric=metric, edge_beta=beta)
    Qh = queries_from_batch(batch)
    O, L, rp, col = B.bipartite_xattn(db, Qh.cuda())
    torch.cuda.synchronize()
    _, adj, O_ref, L_ref = orc.bipartite_xattn(
        Qh, batch.kept_offsets, batch.Kh, batch.Vh, batch.passage_offsets,
        batch.query_passages, batch.wl.scale, 2.5, edge_rule=rule, edge_metric=metric,
        edge_beta=beta)
    check_graph(batch, rp, col, adj)
    check_attention(f64(O), f64(L), np.concatenate(O_ref), np.concatenate(L_ref), dtype)


@pytest.mark.parametrize("rule,metric", [("question", "cosine"), ("fraction", "dot")])
def test_xattn_edge_tie_groups_at_the_cut(B, rule, metric):
    """All kept rows of a question but its last three are copies of its first
    row, so each passage's candidates form a group of equal compatibilities
    (bit-equal on both sides: equal rows take the same arithmetic) and the
    per-question cut falls inside one of them: the selection must take the
    group's lowest flat indices i * P + j, as the oracle does."""
    batch = small_batch("bf16", 7, H=2, d_h=128)
    Qh = queries_from_batch(batch).clone()
    for b in range(batch.B):
        k0, k1 = int(batch.kept_offsets[b]), int(batch.kept_offsets[b + 1])
        if k1 - k0 > 4:
            Qh[k0:k1 - 3] = Qh[k0].clone()
    say(f"xattn edge ties {rule}/{metric} P={batch.P.tolist()} k={batch.k.tolist()}")
    db = B.to_device(batch, avg_degree=2.5, edge_rule=rule, edge_metric=metric, edge_beta=0.3)
    O, L, rp, col = B.bipartite_xattn(db, Qh.cuda())
    torch.cuda.synchronize()
    _, adj, O_ref, L_ref = orc.bipartite_xattn(
        Qh, batch.kept_offsets, batch.Kh, batch.Vh, batch.passage_offsets,
        batch.query_passages, batch.wl.scale, 2.5, edge_rule=rule, edge_metric=metric,
        edge_beta=0.3)
    # the cut splits a tie group: some row of a group is kept and a later one
    # of the same group is not
    split = False
    for a in adj:
        if a.shape[0] > 4:
            for j in range(a.shape[1]):
                col_j = a[:-3, j]
                split |= bool(col_j.any() and not col_j.all())
    assert split, "no tie group straddles the cut; the test input needs changing"
    check_graph(batch, rp, col, adj)
    check_attention(f64(O), f64(L), np.concatenate(O_ref), np.concatenate(L_ref), "bf16")


@pytest.mark.parametrize("dtype,H,d_h,P", [("bf16", 5, 64, (2, 9)), ("f32", 3, 128, (4, 7)),
                                          ("bf16", 2, 128, (17, 20)), ("f32", 4, 64, (18,))])
def test_graph_ragged_slices_and_passage_groups(B, dtype, H, d_h, P):
    """The edge dot products work on column slices of 512 and on tiles of at
    most 16 passages: d = 320 and 384 leave a slice partly empty, 17-20
    passages take two passage tiles.  Graphs exact, attention to the usual
    bar."""
    batch = small_batch(dtype, 9, H=H, d_h=d_h, P=P, L_p=(3, 40), k=(1, 30, 200, 260))
    say(f"graph ragged {dtype} d={H * d_h} P={batch.P.tolist()} k={batch.k.tolist()}")
    db = B.to_device(batch, avg_degree=3.0)
    Qh = queries_from_batch(batch)
    O, L, rp, col = B.bipartite_xattn(db, Qh.cuda())
    torch.cuda.synchronize()
    _, adj, O_ref, L_ref = orc.bipartite_xattn(
        Qh, batch.kept_offsets, batch.Kh, batch.Vh, batch.passage_offsets,
        batch.query_passages, batch.wl.scale, 3.0)
    check_graph(batch, rp, col, adj)
    check_attention(f64(O), f64(L), np.concatenate(O_ref), np.concatenate(L_ref), dtype)


@pytest.mark.parametrize("rule,metric,beta", [("row", "cosine", 0.1), ("fraction", "dot", 0.1)])
def test_fused_edge_rules_full_size(B, rule, metric, beta):
    """highres_bf16 through the fused route under the other cuts: kept sets
    and graphs exact for every question, attention on sampled rows."""
    batch = wls.make_batch("highres_bf16", 2026, threads=16)
    say(f"fused highres {rule}/{metric} beta={beta}")
    db = B.to_device(batch, edge_rule=rule, edge_metric=metric, edge_beta=beta)
    idx, _, Vk = B.prune_topk(db, want_scores=False)
    Qh = Vk.view(-1, batch.Kh.shape[1], batch.Kh.shape[2])
    _, _, rp, col = B.bipartite_xattn(db, Qh)
    fidx, fO, fL = B.route_fused(db)
    torch.cuda.synchronize()
    rows = sample_rows(batch, 8)
    ref = oracle_route(batch, attn_rows=rows, edge_rule=rule, edge_metric=metric, edge_beta=beta)
    idx = fidx.cpu().numpy()
    for b in range(batch.B):
        k0, k1 = batch.kept_offsets[b], batch.kept_offsets[b + 1]
        assert idx[k0:k1].tolist() == ref.kept_idx[b].tolist(), f"q{b} kept set"
    check_graph(batch, rp, col, ref.adj)
    Of, Lf = f64(fO), f64(fL)
    got_O, got_L, want_O, want_L = [], [], [], []
    for b, rs in rows.items():
        k0 = int(batch.kept_offsets[b])
        for r in rs:
            got_O.append(Of[k0 + r]); got_L.append(Lf[k0 + r])
            want_O.append(ref.O[b][r]); want_L.append(ref.LSE[b][r])
    check_attention(np.stack(got_O), np.stack(got_L), np.stack(want_O), np.stack(want_L),
                    "bf16", f"highres {rule}/{metric}")


# --------------------------------------------------------------------------- main-text scorer

def mlp_device(B, w):
    return B.QvsMlp(w.W1.cuda(), w.b1.cuda(), w.w2.cuda(), w.b2)


def check_mlp_prune(batch, w, idx, scores, Vk, questions=None, tag=""):
    """Scores within a float32-accumulation bound of the float64 oracle; the
    kept set a valid top-k of the GPU's own scores; any difference from the
    oracle's kept set inside the tie band (reported, never silent); kept rows
    bitwise equal to V."""
    idx = idx.cpu().numpy()
    s_gpu = scores.cpu().double().numpy()
    Vk = Vk.cpu() if Vk is not None else None
    W1, b1, w2 = w.W1.double().numpy(), w.b1.double().numpy(), w.w2.double().numpy()
    events = 0
    for b in (range(batch.B) if questions is None else questions):
        Q = batch.Qtok[int(batch.q_offsets[b]):int(batch.q_offsets[b + 1])].double().numpy()
        s_ref = orc.qvs_mlp_scores(batch.V[b].double().numpy(), orc.mean_pool_question(Q),
                                   W1, b1, w2, w.b2)
        err = float(np.max(np.abs(s_gpu[b] - s_ref)))
        tol = 2e-5 * (1.0 + float(np.max(np.abs(s_ref))))
        assert err <= tol, f"{tag} q{b}: score error {err:.3e} > {tol:.3e}"
        k0, k1 = int(batch.kept_offsets[b]), int(batch.kept_offsets[b + 1])
        k = k1 - k0
        got = idx[k0:k1]
        assert got.tolist() == sorted(got.tolist()), f"{tag} q{b}: not ascending"
        if Vk is not None:
            assert torch.equal(Vk[k0:k1], batch.V[b][torch.from_numpy(got.astype(np.int64))])
        if k == 0 or k == batch.wl.N:
            assert got.tolist() == list(range(k))
            continue
        rest = np.setdiff1d(np.arange(batch.wl.N), got)
        assert s_gpu[b][got].min() >= s_gpu[b][rest].max(), f"{tag} q{b}: not a top-k of its scores"
        want = orc.qvs_topk(s_ref, k)
        if got.tolist() != want.tolist():
            srt = np.sort(s_ref)[::-1]
            cut = 0.5 * (srt[k - 1] + srt[k])
            diff = np.setxor1d(got, want)
            band = np.abs(s_ref[diff] - cut)
            say(f"{tag} q{b}: tie-band event, tokens {diff.tolist()} at {band.max():.2e} "
                f"from the cut (score error {err:.2e})")
            assert band.max() <= 2 * err, f"{tag} q{b}: kept set differs outside the tie band"
            events += 1
    return events


@pytest.mark.parametrize("hidden", [256, 512])
@pytest.mark.parametrize("seed", wls.SEEDS)
def test_prune_mlp_small_ragged(B, hidden, seed):
    batch = wls.make_batch("llava_bf16", seed, B=4, N=300, H=4, d_h=64, T=(1, 3, 8),
                           k=(0, 7, 33, 64, 300))
    w = wls.make_scorer_weights(batch.wl, hidden, seed)
    say(f"mlp scorer small h={hidden} seed={seed} k={batch.k.tolist()}")
    db = B.to_device(batch)
    idx, scores, Vk = B.prune_topk_mlp(db, mlp_device(B, w))
    torch.cuda.synchronize()
    check_mlp_prune(batch, w, idx, scores, Vk, tag=f"h{hidden}")


def test_prune_mlp_without_b1_and_repeatable(B):
    batch = wls.make_batch("llava_bf16", 11, B=3, N=260, H=2, d_h=128, T=(2, 5), k=(1, 50))
    w = wls.make_scorer_weights(batch.wl, 256, 11)
    w0 = wls.ScorerWeights(w.W1, torch.zeros_like(w.b1), w.w2, w.b2)
    db = B.to_device(batch)
    m = B.QvsMlp(w.W1.cuda(), None, w.w2.cuda(), w.b2)
    a = B.prune_topk_mlp(db, m)
    b = B.prune_topk_mlp(db, m)
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    check_mlp_prune(batch, w0, *a, tag="no b1")


def test_prune_mlp_full_size(B):
    """highres_bf16 (N = 2304, d = 4096) with a 512-unit scorer, in the launch
    configuration the benchmark times; the oracle checks three questions."""
    batch = wls.make_batch("highres_bf16", 2026, threads=16)
    w = wls.make_scorer_weights(batch.wl, 512, 2026)
    say("mlp scorer full size highres_bf16 h=512")
    db = B.to_device(batch)
    idx, scores, Vk = B.prune_topk_mlp(db, mlp_device(B, w))
    torch.cuda.synchronize()
    check_mlp_prune(batch, w, idx, scores, Vk, questions=[0, 7, 15], tag="highres")


# --------------------------------------------------------------------------- fused

@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("seed", wls.SEEDS)
def test_fused_small_ragged(B, dtype, seed):
    batch = small_batch(dtype, seed, H=4, d_h=64, with_bias=True)
    say(f"fused small {dtype} seed={seed}")
    db = B.to_device(batch)
    idx, O, L = B.route_fused(db)
    torch.cuda.synchronize()
    ref = oracle_route(batch)
    idx = idx.cpu().numpy()
    for b in range(batch.B):
        k0, k1 = batch.kept_offsets[b], batch.kept_offsets[b + 1]
        assert idx[k0:k1].tolist() == ref.kept_idx[b].tolist()
    check_attention(f64(O), f64(L), np.concatenate(ref.O), np.concatenate(ref.LSE), dtype)


@pytest.mark.parametrize("seed", wls.SEEDS)
@pytest.mark.parametrize("name", wls.ORDER)
def test_named_full_size_staged_and_fused(B, name, seed):
    """Full-size workloads in the launch configuration the benchmark times, at
    each of the three seeds: exact kept sets and edge sets for every question,
    attention on at least 16 sampled rows of every question, and the fused
    route bitwise equal to the staged calls."""
    batch = wls.make_batch(name, seed, threads=16)
    say(f"full {name} seed {seed}: B={batch.B} N={batch.wl.N} d={batch.wl.d}")
    db = B.to_device(batch)
    idx, _, Vk = B.prune_topk(db, want_scores=False)
    Qh = Vk.view(-1, batch.Kh.shape[1], batch.Kh.shape[2])
    O, L, rp, col = B.bipartite_xattn(db, Qh)
    fidx, fO, fL = B.route_fused(db)
    _, O32, _ = B.route_fused(B.with_f32_output(db))
    torch.cuda.synchronize()
    assert torch.equal(idx, fidx)
    assert torch.equal(O, fO) and torch.equal(L, fL), "fused != staged"
    per_q = 24 if batch.B <= 16 else 16
    rows = sample_rows(batch, per_q, seed=seed)
    ref = oracle_route(batch, attn_rows=rows)
    idx = idx.cpu().numpy()
    for b in range(batch.B):
        k0, k1 = batch.kept_offsets[b], batch.kept_offsets[b + 1]
        assert idx[k0:k1].tolist() == ref.kept_idx[b].tolist(), f"{name} q{b} kept set"
    check_graph(batch, rp, col, ref.adj)
    Of, Lf, O32f = f64(O), f64(L), f64(O32)
    got_O, got_O32, got_L, want_O, want_L = [], [], [], [], []
    for b, rs in rows.items():
        k0 = int(batch.kept_offsets[b])
        for r in rs:
            got_O.append(Of[k0 + r]); got_O32.append(O32f[k0 + r]); got_L.append(Lf[k0 + r])
            want_O.append(ref.O[b][r]); want_L.append(ref.LSE[b][r])
    want_O, want_L = np.stack(want_O), np.stack(want_L)
    tag = f"{name} seed {seed}"
    check_attention(np.stack(got_O), np.stack(got_L), want_O, want_L, batch.wl.dtype, tag)
    check_attention(np.stack(got_O32), np.stack(got_L), want_O, want_L, batch.wl.dtype,
                    tag + " f32-out", stored_bf16=False)


def test_fused_deterministic_and_stream(B):
    batch = wls.make_batch("llava_bf16", 42)
    db = B.to_device(batch)
    a = [t.clone() for t in B.route_fused(db)]
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        b = [t.clone() for t in B.route_fused(db)]
    s.synchronize()
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y)


def test_fused_concurrent_streams(B):
    """Fused routes in flight at once on two streams, each with its own
    workspace: C3 on one stream, C2 and a second C3 (same inputs as the first,
    another workspace) on the other.  Both streams are held by a spin kernel
    first, so the routes are queued together and run side by side.  Each
    result is bitwise equal to the same call made alone."""
    hi = B.to_device(wls.make_batch("highres_bf16", 42, threads=16))
    lo = B.to_device(wls.make_batch("llava_bf16", 42))

    def outs(db):
        p = db.p
        return (torch.empty(p.total_kept, dtype=torch.int32, device="cuda"),
                torch.empty((p.total_kept, p.H, p.d_h), dtype=torch.bfloat16, device="cuda"),
                torch.empty((p.total_kept, p.H), dtype=torch.float32, device="cuda"))

    def call(db, out, ws, stream=None):
        B.skip_route_fused(db.p, db.V, db.Qtok, db.q_offsets, db.w_bias, db.kept_offsets,
                           db.Kh, db.Vh, db.passage_offsets, db.query_passages, *out,
                           workspace=ws, stream=stream)

    ws = {n: B.new_workspace(db.p) for n, db in (("a", hi), ("b", lo), ("c", hi))}
    eager = {}
    for n, db in (("a", hi), ("b", lo), ("c", hi)):
        o = outs(db)
        call(db, o, ws[n])
        torch.cuda.synchronize()
        eager[n] = [t.clone() for t in o]
    got = {n: outs(db) for n, db in (("a", hi), ("b", lo), ("c", hi))}
    for o in got.values():
        for t in o:
            t.zero_()
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(s1):
        torch.cuda._sleep(1 << 21)
        call(hi, got["a"], ws["a"], s1)
    with torch.cuda.stream(s2):
        torch.cuda._sleep(1 << 21)
        call(lo, got["b"], ws["b"], s2)
        call(hi, got["c"], ws["c"], s2)
    torch.cuda.synchronize()
    for n in ("a", "b", "c"):
        for x, y in zip(got[n], eager[n]):
            assert torch.equal(x, y), f"route {n} differs from its eager result"


def test_fused_graph_replay(B):
    """The fused route allocates nothing and records no memory fills, so a
    caller can capture it in a HIP graph: four replays, each after eager
    calls on the same buffers and a synchronisation, each bitwise equal to
    the eager result."""
    batch = wls.make_batch("llava_bf16", 42)
    db = B.to_device(batch)
    p = db.p
    out = (torch.empty(p.total_kept, dtype=torch.int32, device="cuda"),
           torch.empty((p.total_kept, p.H, p.d_h), dtype=torch.bfloat16, device="cuda"),
           torch.empty((p.total_kept, p.H), dtype=torch.float32, device="cuda"))
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        B.route_fused(db, out=out)
    torch.cuda.synchronize()
    ref = [t.clone() for t in out]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        B.route_fused(db, out=out)
    torch.cuda.synchronize()
    for r in range(4):
        for t in out:
            t.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for x, y in zip(out, ref):
            assert torch.equal(x, y), f"replay {r}"
        with torch.cuda.stream(s):
            B.route_fused(db, out=out)          # eager work between replays
        torch.cuda.synchronize()


def test_degenerate_shapes(B):
    # every question: one question token; passages of one token; k = N; P = 0
    batch = wls.make_batch("llava_bf16", 137, B=4, N=64, H=4, d_h=64, T=1, k=(0, 64),
                           P=(0, 1, 2), L_p=1)
    say(f"degenerate k={batch.k.tolist()} P={batch.P.tolist()}")
    db = B.to_device(batch)
    idx, O, L = B.route_fused(db)
    torch.cuda.synchronize()
    ref = oracle_route(batch)
    idx = idx.cpu().numpy()
    for b in range(batch.B):
        k0, k1 = batch.kept_offsets[b], batch.kept_offsets[b + 1]
        assert idx[k0:k1].tolist() == ref.kept_idx[b].tolist()
    check_attention(f64(O), f64(L), np.concatenate(ref.O), np.concatenate(ref.LSE), "bf16")
