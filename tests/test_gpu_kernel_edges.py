"""Kernels at the edges of their tiles, chunks and dispatch rules, against the fp64 oracle."""
import numpy as np
import pytest

from ea_inputs import CONFIGS, make_layer, widen
from oracle import ea_extensions as X
from oracle import ea_oracle as O
from tests import parity as P
import paper_2510_00636_amd as ea

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 127, 129, 2047, 66000])
@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (256, "f32")])
def test_keydiff_chunk_edges(n, d, dtype):
    """One row, one row around a 128-row chunk, and heads long enough for several chunks of both
    passes.  Tolerance: fp32 sums of n unit vectors, n 2^-24 / sqrt(n) of the anchor's length, and a
    d-term fp32 dot product; below 2e-6 absolute (scores lie in [0, 2])."""
    import torch
    cfg = CONFIGS["c2"].with_(dtype=dtype, head_dim=d, n_q_heads=2, n_kv_heads=2)
    if n > 10000 and d == 256:
        cfg = cfg.with_(n_q_heads=1, n_kv_heads=1)
    lay = make_layer(cfg, n=n, window=min(n, 2))
    p = P.params_for(cfg)
    sc = torch.full((1, cfg.n_kv_heads, n), -1.0, device="cuda")
    ea.score_baseline(p, ea.SCORER_KEYDIFF, P.to_dev(lay["k"]), n, n, 0, sc, P.workspace(p, n, 1))
    torch.cuda.synchronize()
    assert np.abs(sc.cpu().numpy() - X.keydiff_scores(widen(lay["k"]))).max() <= 2e-6


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("hq,hkv,n", [(4, 2, 1), (4, 2, 63), (6, 2, 65), (4, 1, 1023), (8, 2, 8201)])
def test_fp32_scores_tile_edges(d, hq, hkv, n):
    """fp32 caches: heads shorter than a key tile, around 64 and 128 keys, spans of more than one
    tile and (8 heads x 8201 keys) the two-tile instances, with a Sigma that is not symmetric.  The
    logits are fp64 sums of the given fp32 numbers, so a score carries the rounding of ||v|| and its
    own to fp32: 2^-23, and the 2^-22 allowed here."""
    import torch
    rng = np.random.default_rng(7 * n + d)
    cfg = CONFIGS["c1"].with_(head_dim=d, n_q_heads=hq, n_kv_heads=hkv)
    lay = make_layer(cfg, n=n, window=min(n, 2))
    a = rng.standard_normal((1, hq, d, d)) / np.sqrt(d)
    sigma = (a @ a.transpose(0, 1, 3, 2) + 0.05 * rng.standard_normal((1, hq, d, d))).astype(np.float32)
    mu = rng.standard_normal((1, hq, d)).astype(np.float32)
    got = P.run_score(cfg, lay, mu, sigma, 0.02, n_cap=n + 3)
    ref = O.scores(widen(lay["k"]), widen(lay["v"]), mu.astype(np.float64), sigma.astype(np.float64), 0.02)
    P.check_scores(got, ref, 2.0 ** -22)


@pytest.mark.parametrize("d,hq,hkv,batch,n", [
    (128, 5, 1, 260, 1030),      # a second round of four units
    (128, 7, 1, 150, 1030),      # the same in two passes
    (64, 2, 1, 300, 1500),       # more units than CUs
    (256, 2, 1, 140, 1030),      # too short for what a spare workgroup loads at d = 256
    (256, 2, 1, 140, 1290),      # fewer jobs than CUs
    (256, 4, 1, 130, 1030),
    (128, 4, 1, 150, 1000),      # too short for spare workgroups
])
def test_scores_with_spare_workgroups(d, hq, hkv, batch, n):
    """Calls whose units do not fill the chip: workgroups dispatched late join heads in progress.
    Against the oracle at the bf16 tolerance of the score path."""
    cfg = CONFIGS["c2"].with_(head_dim=d, n_q_heads=hq, n_kv_heads=hkv, batch=batch)
    lay = make_layer(cfg, n=n, window=64)
    mu, sigma = O.query_stats(widen(lay["q_win"]), lay["q_pos0"], lay["inv_freq"], lay["t_next"], T=cfg.horizon_T)
    mu, sigma = mu.astype(np.float32), sigma.astype(np.float32)
    got = P.run_score(cfg, lay, mu, sigma, 0.02)
    P.check_scores(got, O.scores(widen(lay["k"]), widen(lay["v"]), mu, sigma, 0.02), 2e-3)


def _same_operands(d, heads, a, b):
    if d == 64 or heads >= 192:
        assert np.array_equal(a, b)
    else:
        np.testing.assert_allclose(a, b, rtol=1e-6, atol=0)


@pytest.mark.parametrize("d,hq,hkv,batch", [
    (64, 8, 1, 1), (64, 5, 1, 3),           # G = 5 in an eight-head instance: rows and fragments of no head
    (128, 4, 1, 47), (128, 4, 1, 48),       # 188 and 192 heads: either side of the rule
    (128, 7, 1, 40), (128, 5, 1, 77),       # two passes with room for an eighth head; 385 heads: the other order of sums
])
@pytest.mark.parametrize("w,layout", [(2, 0), (17, 1), (64, 0), (65, 1), (130, 0)])
def test_fused_statistics_give_the_same_operands(d, hq, hkv, batch, w, layout):
    """compress_layer's scores are those of query_stats followed by score, bit for bit (both calls go to the same score
    kernel at this length): the statistics
    kernel that writes the score kernel's operands itself makes the ones that the separate kernels
    make of mu and sigma.  (Those are compared with the oracle elsewhere.)  Where two workgroups share a head (d = 128, under
    192 heads) its power of two may differ, and with it the rounding of entries under 2^-26 of the largest: d^2 of them
    move a logit by less than d 2^-37 of the quadratic term, 1e-8 here, next to fp32 sums of 2^-24."""
    import torch
    n = 300
    cfg = CONFIGS["c2"].with_(head_dim=d, n_q_heads=hq, n_kv_heads=hkv, batch=batch)
    lay = make_layer(cfg, n=n, window=w, interleaved=bool(layout))
    p = P.params_for(cfg, rope_layout=layout)
    ws = P.workspace(p, n, w)
    q, k, v, inv = (P.to_dev(lay[x]) for x in ("q_win", "k", "v", "inv_freq"))
    mu = torch.empty(batch, hq, d, device="cuda")
    sigma = torch.empty(batch, hq, d, d, device="cuda")
    sc = [torch.empty(batch, hkv, n, device="cuda") for _ in range(2)]
    ea.query_stats(p, q, w, lay["q_pos0"], inv, lay["t_next"], mu, sigma, ws)
    ea.score(p, k, v, n, n, mu, sigma, sc[0], ws)
    ea.compress_layer(p, q, w, lay["q_pos0"], inv, lay["t_next"], k, v, n, n, n // 2, sc[1], None, ws)
    torch.cuda.synchronize()
    _same_operands(d, hq * batch, sc[0].cpu().numpy(), sc[1].cpu().numpy())


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1024, 1025, 4095, 4096, 4097, 8192, 8193, 9217, 16383, 16384, 16385])
@pytest.mark.parametrize("kind", ["spread", "ties", "equal"])
def test_select_row_edges(n, kind):
    """Heads around the row and register counts of the one-launch selection, few distinct values and one
    single value among the inputs: the kept positions are exactly the stable top-k's."""
    rng = np.random.default_rng(n)
    shape = (1, 3, n)
    sc = (np.exp(rng.standard_normal(shape)) if kind == "spread" else
          rng.integers(0, 5, shape).astype(np.float64) if kind == "ties" else np.ones(shape)).astype(np.float32)
    cfg = CONFIGS["c1"].with_(n_q_heads=3, n_kv_heads=3)
    for n_keep in {1, n, max(1, n // 2), max(1, n - 1), min(n, 65)}:
        idx = P.run_select(cfg, sc, n_keep)
        assert np.array_equal(idx.astype(np.int64), O.select(sc.astype(np.float64), n_keep)), n_keep


@pytest.mark.parametrize("n,n_keep,floor", [(4095, 2000, 1), (4096, 4000, 4000), (4097, 1500, 700), (5500, 5500, 17),
                                            (8193, 300, 300), (16385, 9000, 4097)])
def test_adaptive_selection_block_edges(n, n_keep, floor):
    """Budgets shared by three heads of one block of 4096 scores and of a few, where every head's own digits are found
    by its last block, with floors from one to all of the budget and scores of different scales: lists and lengths
    are exactly the oracle's.  The whole call is made twice on one workspace: nothing of the first may be left in it."""
    import torch
    cfg = CONFIGS["c2"].with_(batch=2, n_kv_heads=3, n_q_heads=3)
    p = P.params_for(cfg)
    rng = np.random.default_rng(n + floor)
    ws = P.workspace(p, n, 1)
    for rep in range(2):
        sc = np.exp(rng.standard_normal((2, 3, n))).astype(np.float32)
        sc[:, 1] *= 3.0
        sc[0, 0, ::3] = sc[0, 0, 0]
        idx = torch.full((2, 3, n), -7, dtype=torch.int32, device="cuda")
        lengths = torch.full((2, 3), -1, dtype=torch.int32, device="cuda")
        ea.select_adaptive(p, P.to_dev(sc), n, n_keep, floor, idx, lengths, ws)
        torch.cuda.synchronize()
        rl, rk = X.select_adaptive(sc.astype(np.float64), n_keep, floor)
        gl, gi = lengths.cpu().numpy(), idx.cpu().numpy()
        assert np.array_equal(gl, rl)
        assert all(np.array_equal(gi[b, h, :gl[b, h]], rk[b][h]) for b in range(2) for h in range(3))
    assert ea.debug_status(p, n, 1, ws) == 0


@pytest.mark.parametrize("n", [16385, 20480, 20481, 24577, 28672, 28673, 270000])
@pytest.mark.parametrize("kind", ["spread", "ties", "equal"])
def test_select_blocks(n, kind):
    """Selections of several launches (from 24577 scores on) and long ones of one: last blocks of one score and of 4096,
    more than 64 blocks, ties that run across blocks; several on one workspace, where a call must not see the counts of
    the one before."""
    import torch
    rng = np.random.default_rng(n)
    cfg = CONFIGS["c1"].with_(n_q_heads=3, n_kv_heads=3)
    p = P.params_for(cfg)
    ws = P.workspace(p, n, 1)
    for n_keep in (n // 2, n - 1, 1, 5000):
        shape = (1, 3, n)
        sc = (np.exp(rng.standard_normal(shape)) if kind == "spread" else
              rng.integers(0, 5, shape).astype(np.float64) if kind == "ties" else np.ones(shape)).astype(np.float32)
        idx = torch.full((1, 3, n_keep), -1, dtype=torch.int32, device="cuda")
        ea.select(p, P.to_dev(sc), n, n_keep, idx, ws)
        torch.cuda.synchronize()
        assert np.array_equal(idx.cpu().numpy().astype(np.int64), O.select(sc.astype(np.float64), n_keep)), n_keep
    assert ea.debug_status(p, n, 1, ws) == 0


@pytest.mark.parametrize("d,layout", [(64, 0), (128, 0), (128, 1), (256, 0)])
@pytest.mark.parametrize("w", [2, 15, 17, 32, 33, 64, 65, 127, 200])
def test_fp32_statistics_window_edges(d, layout, w):
    """fp32 windows around the eight-pair steps and 64-sample chunks of the covariance loop, against the
    oracle at the statistics tolerance."""
    cfg = CONFIGS["c1"].with_(head_dim=d, n_q_heads=3, n_kv_heads=1, n_outliers=2, outlier_offset=8.0)
    lay = make_layer(cfg, n=w + 7, window=w, interleaved=bool(layout), pos0=50000)
    mu, sg = P.run_query_stats(cfg, lay, rope_layout=layout)
    rmu, rsg = O.query_stats(widen(lay["q_win"]), lay["q_pos0"], lay["inv_freq"], lay["t_next"], T=cfg.horizon_T,
                             layout=layout)
    P.check_stats(mu, sg, rmu, rsg)


@pytest.mark.parametrize("hq,n", [(20, 2048), (24, 2048), (28, 4100), (32, 2100)])
def test_one_kv_head_with_many_query_heads_on_every_cache_layout(hq, n):
    """One KV head, five to eight passes at d = 128, on every cache layout in the one workspace that
    workspace_bytes gives.  Scores against the oracle at the bf16 tolerance, the paged ones against the
    contiguous call's to 2e-5 (the same fp16 products), and a NaN value row of the 8-bit cache
    shows in the status word."""
    import torch
    from ea_inputs import make_block_pools, quantize_fp8
    cfg = CONFIGS["c2"].with_(n_q_heads=hq, n_kv_heads=1)
    w = 64
    lay = make_layer(cfg, n=n, window=w)
    p = P.params_for(cfg, epsilon=0.02)
    mu, sigma = O.query_stats(widen(lay["q_win"]), lay["q_pos0"], lay["inv_freq"], lay["t_next"], T=cfg.horizon_T)
    mu, sigma = mu.astype(np.float32), sigma.astype(np.float32)
    contiguous = P.run_score(cfg, lay, mu, sigma, 0.02)
    P.check_scores(contiguous, O.scores(widen(lay["k"]), widen(lay["v"]), mu, sigma, 0.02), 2e-3)
    kp, vp, tab, nb = make_block_pools(lay["k"], lay["v"], 64, 5)
    tabd = torch.from_numpy(tab).cuda()
    sc = torch.empty(1, 1, n, device="cuda")
    ws = P.workspace(p, n, 1)
    ws.fill_(255)
    ea.score_paged(p, P.to_dev(kp), P.to_dev(vp), ea.make_paged(tabd, 64, nb), n, P.to_dev(mu), P.to_dev(sigma), sc, ws)
    torch.cuda.synchronize()
    np.testing.assert_allclose(sc.cpu().numpy(), contiguous, rtol=2e-5, atol=0)

    k8, ks = quantize_fp8(widen(lay["k"]))
    v8, vs = quantize_fp8(widen(lay["v"]))
    k8d, v8d, ksd, vsd = (torch.from_numpy(x).cuda() for x in (k8, v8, ks, vs))
    ws.fill_(255)
    ea.score_fp8(p, k8d, v8d, ksd, vsd, n, n, P.to_dev(mu), P.to_dev(sigma), sc, ws)
    torch.cuda.synchronize()
    real = [X.fp8_e4m3_decode(c) * s.astype(np.float64)[:, :, None, None] for c, s in ((k8, ks), (v8, vs))]
    P.check_scores(sc.cpu().numpy(), O.scores(real[0], real[1], mu.astype(np.float64), sigma.astype(np.float64), 0.02), 2e-3)

    ws = P.workspace(p, n, w)
    for bad in (False, True):
        if bad:
            v8d[0, 0, 5] = 0x7F
        ea.compress_layer_fp8(p, P.to_dev(lay["q_win"]), w, lay["q_pos0"], P.to_dev(lay["inv_freq"]), lay["t_next"],
                              k8d.clone(), v8d.clone(), ksd, vsd, n, n, n // 2, 0, None, None, None, ws)
        assert ea.debug_status(p, n, w, ws) == (ea.STATUS_BAD_SCORE if bad else 0)


@pytest.mark.parametrize("kind", ["spread", "ties"])
@pytest.mark.parametrize("blocks", [1024, 1025, 2049])
def test_select_more_blocks_than_one_sweep_of_the_counts(blocks, kind):
    """Heads of so many 4096-score blocks that a workgroup adds up the counts in front of it in more than one
    sweep (four words per thread), the last block a single score: exactly the stable top-k."""
    n = (blocks - 1) * 4096 + 1
    rng = np.random.default_rng(blocks)
    sc = (np.exp(rng.standard_normal((1, 1, n))) if kind == "spread" else
          rng.integers(0, 5, (1, 1, n)).astype(np.float64)).astype(np.float32)
    cfg = CONFIGS["c1"].with_(n_q_heads=1, n_kv_heads=1)
    for n_keep in (n // 3, n - 1):
        idx = P.run_select(cfg, sc, n_keep)
        assert np.array_equal(idx.astype(np.int64), O.select(sc.astype(np.float64), n_keep)), n_keep


@pytest.mark.parametrize("dtype,d,many", [("bf16", 64, 8), ("bf16", 128, 8), ("bf16", 128, 400), ("bf16", 256, 8),
                                          ("f32", 64, 8), ("f32", 128, 8), ("f32", 256, 8)])
def test_statistics_do_not_hang_on_layout_or_call_size(dtype, d, many):
    """A head's statistics have the same bits in a call of 8 heads (at d = 128 two workgroups a head) and of
    many (one), and its mean also when the channels come interleaved instead of half-split: one rounding
    rule for the rotation, and the same sums in the same order."""
    import torch
    rng = np.random.default_rng(d + many)
    w, few = 70, 8
    q = rng.standard_normal((1, many, w, d)) * 3.0 + rng.standard_normal((1, many, 1, d))
    q = torch.from_numpy(q.astype(np.float32)).cuda().to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    half_to_inter = np.arange(d).reshape(2, d // 2).T.reshape(-1)      # interleaved channel 2c + b = half-split b d/2 + c
    inv = P.to_dev(1e4 ** (-np.arange(0, d, 2, dtype=np.float64) / d))

    def stats(x, layout):
        heads = x.shape[1]
        cfg = CONFIGS["c2"].with_(dtype=dtype, head_dim=d, n_q_heads=heads, n_kv_heads=heads)
        p = P.params_for(cfg, rope_layout=layout)
        mu = torch.empty(1, heads, d, device="cuda")
        sigma = torch.empty(1, heads, d, d, device="cuda")
        ea.query_stats(p, x.contiguous(), w, 4000, inv, 4000 + w, mu, sigma, P.workspace(p, 1, w))
        torch.cuda.synchronize()
        return mu.cpu().numpy()[:, :few], sigma.cpu().numpy()[:, :few]
    plain, sigma = stats(q[:, :few], 0)
    mu_many, sigma_many = stats(q, 0)
    assert np.array_equal(mu_many, plain) and np.array_equal(sigma_many, sigma)
    assert np.array_equal(stats(q[..., half_to_inter], 1)[0], plain[..., half_to_inter])


@pytest.mark.parametrize("form", ["layer", "fp8"])
def test_compress_takes_the_other_score_kernel(form):
    """Five query heads per KV head, 16 x 4600 keys: the score call goes to the LDS-fragment kernel, the compress call,
    whose statistics make the other one's operands, to the register-fragment kernel.  The scores agree to 2e-5, the
    bound between kernels that add the same fp16 products in another order."""
    import torch
    from ea_inputs import quantize_fp8
    n, w = 4600, 64
    cfg = CONFIGS["c2"].with_(n_q_heads=10, n_kv_heads=2, batch=8)
    lay = make_layer(cfg, n=n, window=w)
    p = P.params_for(cfg)
    ws = P.workspace(p, n, w)
    win = (P.to_dev(lay["q_win"]), w, lay["q_pos0"], P.to_dev(lay["inv_freq"]), lay["t_next"])
    mu, sigma = torch.empty(8, 10, 128, device="cuda"), torch.empty(8, 10, 128, 128, device="cuda")
    want, got = (torch.empty(8, 2, n, device="cuda") for _ in range(2))
    ea.query_stats(p, *win, mu, sigma, ws)
    if form == "fp8":
        (k8, ks), (v8, vs) = quantize_fp8(widen(lay["k"])), quantize_fp8(widen(lay["v"]))
        k, v, ks, vs = (torch.from_numpy(x).cuda() for x in (k8, v8, ks, vs))
        ea.score_fp8(p, k, v, ks, vs, n, n, mu, sigma, want, ws)
        ea.compress_layer_fp8(p, *win, k, v, ks, vs, n, n, 2000, 0, got, None, None, ws)
    else:
        k, v = P.to_dev(lay["k"]), P.to_dev(lay["v"])
        ea.score(p, k, v, n, n, mu, sigma, want, ws)
        ea.compress_layer(p, *win, k, v, n, n, 2000, got, None, ws)
    torch.cuda.synchronize()
    np.testing.assert_allclose(got.cpu().numpy(), want.cpu().numpy(), rtol=2e-5, atol=0)


@pytest.mark.parametrize("form,d,hq,hkv,batch,w", [
    (form, *shape) for form in ("unordered", "paged", "fp8", "adaptive")
    for shape in ((64, 5, 1, 3, 17), (128, 4, 1, 47, 64), (128, 4, 1, 48, 65), (128, 5, 1, 77, 2))
    if not (form == "fp8" and shape[0] == 64)])                    # (8-bit rows have 128 channels or more)
def test_fused_statistics_behind_every_compress_call(form, d, hq, hkv, batch, w):
    """The other compress calls, on either side of the number of heads from which the statistics kernel writes
    the score kernel's operands: their scores are those of query_stats followed by the score call of the
    same cache layout, bit for bit, or to the bound given there."""
    import torch
    from ea_inputs import make_block_pools, quantize_fp8
    n, n_keep = 300, 120
    cfg = CONFIGS["c2"].with_(head_dim=d, n_q_heads=hq, n_kv_heads=hkv, batch=batch)
    lay = make_layer(cfg, n=n, window=w)
    p = P.params_for(cfg)
    ws = P.workspace(p, n, w)
    q, k, v, inv = (P.to_dev(lay[x]) for x in ("q_win", "k", "v", "inv_freq"))
    win = (q, w, lay["q_pos0"], inv, lay["t_next"])
    mu = torch.empty(batch, hq, d, device="cuda")
    sigma = torch.empty(batch, hq, d, d, device="cuda")
    want, got = (torch.empty(batch, hkv, n, device="cuda") for _ in range(2))
    idx = torch.empty(batch, hkv, n, dtype=torch.int32, device="cuda")
    lengths = torch.empty(batch, hkv, dtype=torch.int32, device="cuda")
    ea.query_stats(p, *win, mu, sigma, ws)
    if form == "paged":
        kp, vp, tab, nb = make_block_pools(lay["k"], lay["v"], 32, 3)
        k, v, tabd = P.to_dev(kp), P.to_dev(vp), torch.from_numpy(tab).cuda()
        pg = ea.make_paged(tabd, 32, nb)
        ea.score_paged(p, k, v, pg, n, mu, sigma, want, ws)
        ea.compress_layer_paged(p, *win, k, v, pg, n, n_keep, 0, got, None, None, ws)
    elif form == "fp8":
        k8, ks = quantize_fp8(widen(lay["k"]))
        v8, vs = quantize_fp8(widen(lay["v"]))
        k, v, ks, vs = (torch.from_numpy(x).cuda() for x in (k8, v8, ks, vs))
        ea.score_fp8(p, k, v, ks, vs, n, n, mu, sigma, want, ws)
        ea.compress_layer_fp8(p, *win, k, v, ks, vs, n, n, n_keep, 1, got, None, None, ws)
    else:
        ea.score(p, k, v, n, n, mu, sigma, want, ws)
        if form == "unordered":
            ea.compress_layer_unordered(p, *win, k, v, n, n, n_keep, got, None, None, ws)
        else:
            ea.compress_layer_adaptive(p, *win, k, v, n, n, n_keep, 30, got, idx, lengths, ws)
    torch.cuda.synchronize()
    _same_operands(d, hq * batch, got.cpu().numpy(), want.cpu().numpy())


@pytest.mark.parametrize("n,w,floor", [(16385, 64, 300), (20481, 2, 300), (20481, 64, 0), (16385, 3, 6000), (4096, 64, 0), (777, 20, 0)])
def test_adaptive_pass_over_long_heads(n, w, floor):
    """The whole adaptive call over heads of several blocks: their first digits counted on the way, everything cleared at
    the start of the call, also under windows of a few samples (one or two workgroups for the table); and over short
    layers without a floor, which one workgroup selects from.  Two passes over different caches on one
    workspace that starts with rubbish; lists, lengths and moved rows are exactly the oracle's for the
    call's own scores, and a NaN value row shows in the status word."""
    import torch
    cfg = CONFIGS["c2"].with_(batch=2, n_q_heads=4, n_kv_heads=2)
    n_keep = int(0.4 * n)
    p = P.params_for(cfg)
    ws = P.workspace(p, n, w)
    ws.fill_(255)
    for rep in range(2):
        lay = make_layer(cfg, layer=rep, n=n, window=w)
        k, v = P.to_dev(lay["k"]), P.to_dev(lay["v"])
        sc = torch.empty(2, 2, n, device="cuda")
        idx = torch.full((2, 2, n), -7, dtype=torch.int32, device="cuda")
        lengths = torch.full((2, 2), -1, dtype=torch.int32, device="cuda")
        ea.compress_layer_adaptive(p, P.to_dev(lay["q_win"]), w, lay["q_pos0"], P.to_dev(lay["inv_freq"]), lay["t_next"],
                                   k, v, n, n, n_keep, floor, sc, idx, lengths, ws)
        assert ea.debug_status(p, n, w, ws) == 0
        own = sc.cpu().numpy().astype(np.float64)
        rl, rk = X.select_adaptive(own, n_keep, floor)
        gl, gi, ko, vo = lengths.cpu().numpy(), idx.cpu().numpy(), P.to_host(k), P.to_host(v)
        moved = X.compact_ragged(lay["k"], lay["v"], rk)
        assert np.array_equal(gl, rl)
        for b in range(2):
            for h in range(2):
                m = gl[b, h]
                assert np.array_equal(gi[b, h, :m], rk[b][h])
                assert np.array_equal(ko[b, h, :m], moved[b][h][0]) and np.array_equal(vo[b, h, :m], moved[b][h][1])
                assert np.array_equal(ko[b, h, m:], lay["k"][b, h, m:])
    if w >= 16:                                            # (near-rank-one covariances: see the accuracy of ea_score)
        rmu, rsg = O.query_stats(widen(lay["q_win"]), lay["q_pos0"], lay["inv_freq"], lay["t_next"], T=cfg.horizon_T)
        P.check_scores(own, O.scores(widen(lay["k"]), widen(lay["v"]), rmu, rsg, cfg.epsilon), 2e-3)
    v = P.to_dev(lay["v"])
    v[1, 1, n // 2] = float("nan")
    ea.compress_layer_adaptive(p, P.to_dev(lay["q_win"]), w, lay["q_pos0"], P.to_dev(lay["inv_freq"]), lay["t_next"],
                               P.to_dev(lay["k"]), v, n, n, n_keep, floor, None, idx, lengths, ws)
    assert ea.debug_status(p, n, w, ws) & ea.STATUS_BAD_SCORE


@pytest.mark.parametrize("hq,hkv", [(1, 1), (6, 2), (4, 1), (5, 1), (6, 1), (14, 2), (9, 1)])
@pytest.mark.parametrize("n", [63, 64, 65, 128, 1000, 1040])
def test_register_fragment_scores_at_tile_edges(hq, hkv, n):
    """d = 128, passes of four query heads with one to four wavefronts at work, tiles of 64 keys: heads around one
    tile, the ragged last one inside a group of 16 keys and at its edge, on contiguous tensors (rows beyond n hold
    NaN), block pools and 8-bit caches, all in the workspace that workspace_bytes gives.  Against the oracle at the
    bf16 tolerance; the pools' scores against the contiguous ones to 2e-5 (the same fp16 products)."""
    import torch
    from ea_inputs import make_block_pools, quantize_fp8
    cfg = CONFIGS["c2"].with_(n_q_heads=hq, n_kv_heads=hkv)
    lay = make_layer(cfg, n=n, window=32)
    p = P.params_for(cfg, epsilon=0.02)
    mu, sigma = O.query_stats(widen(lay["q_win"]), lay["q_pos0"], lay["inv_freq"], lay["t_next"], T=cfg.horizon_T)
    mu, sigma = mu.astype(np.float32), sigma.astype(np.float32)
    contiguous = P.run_score(cfg, lay, mu, sigma, 0.02, n_cap=n + 5)
    P.check_scores(contiguous, O.scores(widen(lay["k"]), widen(lay["v"]), mu, sigma, 0.02), 2e-3)
    kp, vp, tab, nb = make_block_pools(lay["k"], lay["v"], 16, 3)
    tabd = torch.from_numpy(tab).cuda()
    sc = torch.empty(1, hkv, n, device="cuda")
    ws = P.workspace(p, n, 1)
    ea.score_paged(p, P.to_dev(kp), P.to_dev(vp), ea.make_paged(tabd, 16, nb), n, P.to_dev(mu), P.to_dev(sigma), sc, ws)
    torch.cuda.synchronize()
    np.testing.assert_allclose(sc.cpu().numpy(), contiguous, rtol=2e-5, atol=0)
    k8, ks = quantize_fp8(widen(lay["k"]))
    v8, vs = quantize_fp8(widen(lay["v"]))
    k8d, v8d, ksd, vsd = (torch.from_numpy(x).cuda() for x in (k8, v8, ks, vs))
    ea.score_fp8(p, k8d, v8d, ksd, vsd, n, n, P.to_dev(mu), P.to_dev(sigma), sc, ws)
    torch.cuda.synchronize()
    real = [X.fp8_e4m3_decode(c) * s.astype(np.float64)[:, :, None, None] for c, s in ((k8, ks), (v8, vs))]
    P.check_scores(sc.cpu().numpy(), O.scores(real[0], real[1], mu.astype(np.float64), sigma.astype(np.float64), 0.02), 2e-3)


@pytest.mark.parametrize("w,dm,hq", [(16, 64, 2), (17, 512, 2), (33, 520, 2), (65, 2056, 2), (100, 4104, 24),
                                     (100, 2040, 32), (50, 4104, 32)])     # 64 samples x four parts, 32 x eight
def test_projection_tile_edges(w, dm, hq):
    """bf16 projections around the edges of their tiles of 16, 32 and 64 samples, four and eight parts of the d_model
    axis, parts that are empty and parts that end inside a block of 64 entries.  Against Eq. 5 in fp64 at the tolerance
    of the statistics: products of bf16 numbers are exact, their fp32 sums carry about sqrt(d_model) 2^-24."""
    import torch
    from ea_inputs import bf16_bits_from_f64, inv_freq_table
    cfg = CONFIGS["c2"].with_(n_q_heads=hq, n_kv_heads=2)
    r = np.random.default_rng(w + dm)
    hb = bf16_bits_from_f64(r.standard_normal((1, w, dm)) * 1.5 + r.standard_normal(dm))
    wb = bf16_bits_from_f64(r.standard_normal((hq, 128, dm)) / np.sqrt(dm))
    inv = inv_freq_table(128, cfg.rope_base)
    p = P.params_for(cfg)
    mu, sg = torch.empty(1, hq, 128, device="cuda"), torch.empty(1, hq, 128, 128, device="cuda")
    ea.query_stats_hidden(p, P.to_dev(hb), P.to_dev(wb), dm, w, P.to_dev(inv), 70000, mu, sg, P.workspace(p, 8, w))
    torch.cuda.synchronize()
    rmu, rsg = X.query_stats_hidden(widen(hb), widen(wb), inv, 70000, T=cfg.horizon_T)
    P.check_stats(mu.cpu().numpy(), sg.cpu().numpy(), rmu, rsg)


@pytest.mark.parametrize("d,hq,hkv,n", [(64, 4, 2, 200), (64, 5, 1, 33), (128, 4, 2, 40), (128, 5, 1, 63), (128, 8, 2, 300),
                                        (256, 1, 1, 200), (256, 4, 2, 300)])
def test_bf16_scores_with_a_sigma_that_is_not_symmetric(d, hq, hkv, n):
    """k^T Sigma k takes both entries of every pair of channels, also inside the blocks on the diagonal, on every cache
    layout.  Sigma is a covariance of unit scale plus noise of 5 %, against the oracle at the bf16 tolerance of the
    score path; an entry of either side that is not a number has to show in the head's scores."""
    import torch
    from ea_inputs import make_block_pools, quantize_fp8
    rng = np.random.default_rng(11 * n + d)
    cfg = CONFIGS["c2"].with_(head_dim=d, n_q_heads=hq, n_kv_heads=hkv)
    lay = make_layer(cfg, n=n, window=2)
    p = P.params_for(cfg, epsilon=0.02)
    a = rng.standard_normal((1, hq, d, d)) / np.sqrt(d)
    sigma = (a @ a.transpose(0, 1, 3, 2) + 0.05 * rng.standard_normal((1, hq, d, d))).astype(np.float32)
    mu = rng.standard_normal((1, hq, d)).astype(np.float32)
    ref = O.scores(widen(lay["k"]), widen(lay["v"]), mu.astype(np.float64), sigma.astype(np.float64), 0.02)
    P.check_scores(P.run_score(cfg, lay, mu, sigma, 0.02), ref, 2e-3)
    kp, vp, tab, nb = make_block_pools(lay["k"], lay["v"], 16, 3)
    tabd = torch.from_numpy(tab).cuda()
    sc = torch.empty(1, hkv, n, device="cuda")
    ws = P.workspace(p, n, 1)
    ea.score_paged(p, P.to_dev(kp), P.to_dev(vp), ea.make_paged(tabd, 16, nb), n, P.to_dev(mu), P.to_dev(sigma), sc, ws)
    torch.cuda.synchronize()
    P.check_scores(sc.cpu().numpy(), ref, 2e-3)
    if d >= 128:
        (k8, ks), (v8, vs) = quantize_fp8(widen(lay["k"])), quantize_fp8(widen(lay["v"]))
        k8d, v8d, ksd, vsd = (torch.from_numpy(x).cuda() for x in (k8, v8, ks, vs))
        ea.score_fp8(p, k8d, v8d, ksd, vsd, n, n, P.to_dev(mu), P.to_dev(sigma), sc, ws)
        torch.cuda.synchronize()
        real = [X.fp8_e4m3_decode(c) * s.astype(np.float64)[:, :, None, None] for c, s in ((k8, ks), (v8, vs))]
        P.check_scores(sc.cpu().numpy(), O.scores(real[0], real[1], mu.astype(np.float64), sigma.astype(np.float64), 0.02), 2e-3)
    for i, j in ((3, 9), (9, 3), (0, d - 1), (d - 1, 0)):
        bad = sigma.copy()
        bad[0, 0, i, j] = np.nan
        got = torch.empty(1, hkv, n, device="cuda")
        ea.score(p, P.to_dev(lay["k"]), P.to_dev(lay["v"]), n, n, P.to_dev(mu), P.to_dev(bad), got, ws)
        torch.cuda.synchronize()
        assert torch.isnan(got[0, 0]).all() and torch.isfinite(got[0, 1:]).all(), (i, j)


@pytest.mark.parametrize("hq,batch", [(4, 300), (7, 150)])
def test_register_fragment_scores_with_spare_workgroups(hq, batch):
    """d = 128, more jobs than whole workgroups per job fill the chip with: all tiles are drawn, and workgroups come when
    their unit has none left.  On contiguous tensors, block pools and 8-bit caches, and in the two forms without a value
    side, with a ragged last tile.  Against the oracle at the bf16 tolerance; norms at half of it (a square root)."""
    import torch
    from ea_inputs import make_block_pools, quantize_fp8
    n, eps = 1030, 0.02
    cfg = CONFIGS["c2"].with_(n_q_heads=hq, n_kv_heads=1, batch=batch)
    lay = make_layer(cfg, n=n, window=32)
    p = P.params_for(cfg, epsilon=eps)
    mu, sigma = O.query_stats(widen(lay["q_win"]), lay["q_pos0"], lay["inv_freq"], lay["t_next"], T=cfg.horizon_T)
    mu, sigma = mu.astype(np.float32), sigma.astype(np.float32)
    mud, sgd, k, v = (P.to_dev(x) for x in (mu, sigma, lay["k"], lay["v"]))
    ws = P.workspace(p, n, 1)
    sc = torch.empty(batch, 1, n, device="cuda")
    ref = O.scores(widen(lay["k"]), widen(lay["v"]), mu, sigma, eps)
    ea.score(p, k, v, n, n, mud, sgd, sc, ws)
    torch.cuda.synchronize()
    contiguous = sc.cpu().numpy()
    P.check_scores(contiguous, ref, 2e-3)
    kp, vp, tab, nb = make_block_pools(lay["k"], lay["v"], 16, 3)
    tabd = torch.from_numpy(tab).cuda()
    ea.score_paged(p, P.to_dev(kp), P.to_dev(vp), ea.make_paged(tabd, 16, nb), n, mud, sgd, sc, ws)
    torch.cuda.synchronize()
    np.testing.assert_allclose(sc.cpu().numpy(), contiguous, rtol=2e-5, atol=0)
    (k8, ks), (v8, vs) = quantize_fp8(widen(lay["k"])), quantize_fp8(widen(lay["v"]))
    k8d, v8d, ksd, vsd = (torch.from_numpy(x).cuda() for x in (k8, v8, ks, vs))
    ea.score_fp8(p, k8d, v8d, ksd, vsd, n, n, mud, sgd, sc, ws)
    torch.cuda.synchronize()
    real = [X.fp8_e4m3_decode(c) * s.astype(np.float64)[:, :, None, None] for c, s in ((k8, ks), (v8, vs))]
    P.check_scores(sc.cpu().numpy(), O.scores(real[0], real[1], mu.astype(np.float64), sigma.astype(np.float64), eps), 2e-3)
    wo = np.random.default_rng(5).standard_normal((hq, 128, 128)) / 12
    gram = np.ascontiguousarray(np.swapaxes(wo, 1, 2) @ wo, np.float32)
    wn = torch.empty(batch, hq, n, device="cuda")
    ea.value_norms_wo(p, v, n, n, torch.from_numpy(gram).cuda(), wn, ws)
    torch.cuda.synchronize()
    vals = widen(lay["v"]).astype(np.float64)[:, 0]
    norms = np.stack([np.sqrt(np.maximum(((vals @ m.astype(np.float64)) * vals).sum(-1), 0)) for m in gram], 1)
    np.testing.assert_allclose(wn.cpu().numpy(), norms, rtol=1e-3)
    # the same attention, weighed by ones: (mean_g a + eps)
    ea.score_wo(p, k, v, n, n, mud, sgd, torch.ones(batch, hq, n, device="cuda"), sc, ws)
    torch.cuda.synchronize()
    P.check_scores(sc.cpu().numpy(), ref / np.linalg.norm(vals, axis=-1)[:, None], 2e-3)


@pytest.mark.parametrize("n", [20480, 24575, 24576, 24577, 28673])
@pytest.mark.parametrize("kind", ["spread", "ties", "special"])
def test_select_around_the_one_launch_limit(n, kind):
    """Heads on both sides of the longest that one workgroup selects, with last rows of one score, of 63 and of 64, ties that run
    across rows and wavefronts, and scores among zero, denormals, the largest number and infinity: exactly the stable top-k."""
    rng = np.random.default_rng(n)
    shape = (1, 3, n)
    sc = np.exp(rng.standard_normal(shape)).astype(np.float32)
    if kind == "ties":
        sc = rng.integers(0, 3, shape).astype(np.float32)
    elif kind == "special":
        sc = rng.choice(np.array([0.0, 1e-45, 1e-40, 1.0, 3.4028235e38, np.inf], dtype=np.float32), shape)
    cfg = CONFIGS["c1"].with_(n_q_heads=3, n_kv_heads=3)
    for n_keep in (1, 64, n // 2, n - 1, n):
        idx = P.run_select(cfg, sc, n_keep)
        assert np.array_equal(idx.astype(np.int64), O.select(sc.astype(np.float64), n_keep)), n_keep


@pytest.mark.parametrize("w,dm,hq,hkv", [(520, 200, 16, 2), (513, 72, 16, 2), (40, 136, 3, 1), (1, 8, 1, 1), (127, 1000, 5, 1)])
def test_projection_blocks_of_whole_lines(w, dm, hq, hkv):
    """bf16 projections with 64 samples per workgroup (enough of them for that), d_model of less than one block of 64 entries
    and ends inside a block (rows then start in the middle of a line of memory), and channel counts that the eight dies do not
    divide.  Against Eq. 5 in fp64 at the tolerance of the statistics, as in the test above of the same tiles."""
    import torch
    from ea_inputs import bf16_bits_from_f64, inv_freq_table
    cfg = CONFIGS["c2"].with_(n_q_heads=hq, n_kv_heads=hkv)
    r = np.random.default_rng(w + dm)
    hb = bf16_bits_from_f64(r.standard_normal((1, w, dm)) * 1.5 + r.standard_normal(dm))
    wb = bf16_bits_from_f64(r.standard_normal((hq, 128, dm)) / np.sqrt(dm))
    inv = inv_freq_table(128, cfg.rope_base)
    p = P.params_for(cfg)
    mu, sg = torch.empty(1, hq, 128, device="cuda"), torch.empty(1, hq, 128, 128, device="cuda")
    ea.query_stats_hidden(p, P.to_dev(hb), P.to_dev(wb), dm, w, P.to_dev(inv), 70000, mu, sg, P.workspace(p, 8, w))
    torch.cuda.synchronize()
    rmu, rsg = X.query_stats_hidden(widen(hb), widen(wb), inv, 70000, T=cfg.horizon_T)
    P.check_stats(mu.cpu().numpy(), sg.cpu().numpy(), rmu, rsg)


@pytest.mark.parametrize("hkv,n", [(3, 4096), (5, 4097), (16, 300), (17, 300), (40, 5000), (2, 25000), (130, 300), (70, 9000),
                                   (1, 3), (1, 64), (2, 4096), (3, 2731), (2047, 4), (2048, 4)])
@pytest.mark.parametrize("kind", ["spread", "ties", "equal", "special", "shared"])
def test_adaptive_selection_shares_out_ties(hkv, n, kind):
    """Budgets shared by a layer's heads where the floor's threshold of a head lies above the pool's, at it and below it: few
    distinct values and a single one (all that decides is the order of heads and positions), zero, denormals and infinity,
    and heads whose first digits agree and whose later ones do not; heads of one block and of several, more heads than a
    wavefront has lanes, and layers on both sides of the limits (scores and heads) up to which one workgroup takes them; floors of none, one, some and all of the budget.  Exactly the oracle's lists."""
    import torch
    cfg = CONFIGS["c2"].with_(batch=2, n_kv_heads=hkv, n_q_heads=hkv)
    p = P.params_for(cfg)
    rng = np.random.default_rng(n + hkv)
    shape = (2, hkv, n)
    sc = np.exp(rng.standard_normal(shape)).astype(np.float32)
    if kind == "ties":
        sc = rng.integers(0, 4, shape).astype(np.float32)
    elif kind == "equal":
        sc = np.ones(shape, dtype=np.float32)
    elif kind == "special":
        sc = rng.choice(np.array([0.0, 1e-45, 1e-40, 1.0, 3.4028235e38, np.inf], dtype=np.float32), shape)
    elif kind == "shared":
        sc = (1.0 + rng.integers(0, 3000, shape) * 2.0 ** -23).astype(np.float32)
        sc[:, 0] = (1.0 + rng.integers(0, 3, (2, n)) * 2.0 ** -13).astype(np.float32)
    ws = P.workspace(p, n, 1)
    for n_keep, floor in ((n // 2, 0), (n // 2, n // 8), (n // 2, n // 2), (n // 3, n // 3 - 1), (n, 1), (n, n), (1, 1), (1, 0), (0, 0)):
        idx = torch.full(shape, -7, dtype=torch.int32, device="cuda")
        lengths = torch.full((2, hkv), -1, dtype=torch.int32, device="cuda")
        ea.select_adaptive(p, P.to_dev(sc), n, n_keep, floor, idx, lengths, ws)
        torch.cuda.synchronize()
        rl, rk = X.select_adaptive(sc.astype(np.float64), n_keep, floor)
        gl, gi = lengths.cpu().numpy(), idx.cpu().numpy()
        assert np.array_equal(gl, rl), (n_keep, floor)
        for b in range(2):
            for h in range(hkv):
                assert np.array_equal(gi[b, h, :gl[b, h]], rk[b][h]), (n_keep, floor, b, h)
                assert np.all(gi[b, h, gl[b, h]:] == -7)
        assert ea.debug_status(p, n, 1, ws) == 0


@pytest.mark.parametrize("hq,batch,n", [(5, 36, 4100), (5, 36, 4097), (5, 300, 1030), (5, 40, 64 * 65), (9, 9, 16449), (10, 64, 2049),
                                        (10, 9, 16449), (10, 100, 1030), (13, 200, 64), (15, 150, 1030)])
def test_five_heads_per_pass_in_registers(hq, batch, n):
    """d = 128, passes of five query heads of which the wavefronts share the last: heads whose last tile of 64 keys holds 1, 4,
    6 or all of them, spare workgroups, a second pass of four heads and of five, three passes, both with spare workgroups (the
    row of 64 sequences takes four heads per pass: the rule's other side), on contiguous tensors, 8-bit caches and the
    forms without a value side, and behind the statistics that make the operands tile by tile.  Against the oracle at the bf16
    tolerance (norms at half of it, a square root); twice with the same bits; a head's NaN stays its own."""
    import torch
    from ea_inputs import quantize_fp8
    eps, w = 0.02, 32
    cfg = CONFIGS["c2"].with_(n_q_heads=hq, n_kv_heads=1, batch=batch)
    lay = make_layer(cfg, n=n, window=w)
    p = P.params_for(cfg, epsilon=eps)
    mu, sigma = O.query_stats(widen(lay["q_win"]), lay["q_pos0"], lay["inv_freq"], lay["t_next"], T=cfg.horizon_T)
    mu, sigma = mu.astype(np.float32), sigma.astype(np.float32)
    mud, sgd, k, v = (P.to_dev(x) for x in (mu, sigma, lay["k"], lay["v"]))
    ws = P.workspace(p, n, w)
    ref = O.scores(widen(lay["k"]), widen(lay["v"]), mu, sigma, eps)
    sc, again, fused = (torch.empty(batch, 1, n, device="cuda") for _ in range(3))
    ea.score(p, k, v, n, n, mud, sgd, sc, ws)
    ea.score(p, k, v, n, n, mud, sgd, again, ws)
    torch.cuda.synchronize()
    P.check_scores(sc.cpu().numpy(), ref, 2e-3)
    assert torch.equal(sc, again)
    ea.compress_layer(p, P.to_dev(lay["q_win"]), w, lay["q_pos0"], P.to_dev(lay["inv_freq"]), lay["t_next"], k.clone(), v.clone(),
                      n, n, n // 2, fused, None, ws)
    torch.cuda.synchronize()
    P.check_scores(fused.cpu().numpy(), ref, 2e-3)
    gram = np.stack([np.eye(128) * (1 + g) for g in range(hq)]).astype(np.float32)
    wn = torch.empty(batch, hq, n, device="cuda")
    ea.value_norms_wo(p, v, n, n, P.to_dev(gram), wn, ws)
    torch.cuda.synchronize()
    norms = np.linalg.norm(widen(lay["v"]), axis=-1)
    P.check_scores(wn.cpu().numpy(), norms * np.sqrt(1.0 + np.arange(hq))[None, :, None], 1e-3)
    ones = torch.ones(batch, hq, n, device="cuda")
    ea.score_wo(p, k, v, n, n, mud, sgd, ones, again, ws)
    torch.cuda.synchronize()
    P.check_scores(again.cpu().numpy(), ref / norms, 2e-3)
    if batch * n <= 150000:
        (k8, ks), (v8, vs) = quantize_fp8(widen(lay["k"])), quantize_fp8(widen(lay["v"]))
        k8d, v8d, ksd, vsd = (torch.from_numpy(x).cuda() for x in (k8, v8, ks, vs))
        ea.score_fp8(p, k8d, v8d, ksd, vsd, n, n, mud, sgd, again, ws)
        torch.cuda.synchronize()
        real = [X.fp8_e4m3_decode(c) * s.astype(np.float64)[:, :, None, None] for c, s in ((k8, ks), (v8, vs))]
        P.check_scores(again.cpu().numpy(), O.scores(real[0], real[1], mu.astype(np.float64), sigma.astype(np.float64), eps), 2e-3)
    for g in (0, 4, hq - 1):                               # of the first sequence: all its scores, and no other sequence's
        bad = mu.copy()
        bad[0, g, 5] = np.nan
        ea.score(p, k, v, n, n, P.to_dev(bad), sgd, again, ws)
        torch.cuda.synchronize()
        assert torch.isnan(again[0]).all() and torch.equal(again[1:], sc[1:]), g


@pytest.mark.parametrize("dtype,n,heads", [(t, n, (5, 9)) for t in ("bf16", "f32") for n in (1, 63, 64, 1023, 1024, 1025, 2048, 2049, 3073, 4095, 4096, 4097)] +
                         [("bf16", 5120, (5, 9)), ("bf16", 5121, (5, 9))] +
                         [("bf16", 640, (17, 63, 64)), ("bf16", 641, (64,)), ("bf16", 2400, (16, 17)), ("f32", 336, (17, 64)), ("f32", 337, (64,)),
                          ("f32", 1075, (20,))])
def test_finalize_and_selection_in_one_launch(dtype, n, heads):
    """Compress calls around the rows per thread of the launch that finishes the scores of a head and selects from them, and on
    both sides of its limits, with five and nine query heads per KV head (four are added up at a time) and with more of them
    than its wavefronts, which then take several log-sum-exps each.  The scores are the
    score call's bit for bit where the operands are (fp32), the positions the stable top-k of the call's own scores, the
    rows moved accordingly, and a NaN value row shows in the status word."""
    import torch
    for hq in heads:
        cfg = CONFIGS["c2" if dtype == "bf16" else "c1"].with_(n_q_heads=hq, n_kv_heads=1, batch=2)
        w = min(n, 20)
        lay = make_layer(cfg, n=n, window=w)
        p = P.params_for(cfg, epsilon=0.02)
        ws = P.workspace(p, n, w)
        win = (P.to_dev(lay["q_win"]), w, lay["q_pos0"], P.to_dev(lay["inv_freq"]), lay["t_next"])
        d = cfg.head_dim
        mu, sigma = torch.empty(2, hq, d, device="cuda"), torch.empty(2, hq, d, d, device="cuda")
        want, got = torch.empty(2, 1, n, device="cuda"), torch.empty(2, 1, n, device="cuda")
        k, v = P.to_dev(lay["k"]), P.to_dev(lay["v"])
        ea.query_stats(p, *win, mu, sigma, ws)
        ea.score(p, k, v, n, n, mu, sigma, want, ws)
        for n_keep in {1, (n + 1) // 2, n}:
            k, v = P.to_dev(lay["k"]), P.to_dev(lay["v"])
            idx = torch.full((2, 1, n_keep), -1, dtype=torch.int32, device="cuda")
            ea.compress_layer(p, *win, k, v, n, n, n_keep, got, idx, ws)
            torch.cuda.synchronize()
            if dtype == "f32":
                assert torch.equal(got, want)
            else:                                          # other operands by at most 2^-26 of the largest, other kernels' sums
                np.testing.assert_allclose(got.cpu().numpy(), want.cpu().numpy(), rtol=2e-5, atol=0)
            own = O.select(got.cpu().numpy().astype(np.float64), n_keep)
            assert np.array_equal(idx.cpu().numpy(), own)
            rk, rv = O.compact(lay["k"], lay["v"], own)
            assert np.array_equal(P.to_host(k)[:, :, :n_keep], rk) and np.array_equal(P.to_host(v)[:, :, :n_keep], rv)
            assert ea.debug_status(p, n, w, ws) == 0
        v = P.to_dev(lay["v"])
        v[1, 0, n // 2] = float("nan")
        ea.compress_layer(p, *win, P.to_dev(lay["k"]), v, n, n, n, got, None, ws)
        assert ea.debug_status(p, n, w, ws) & ea.STATUS_BAD_SCORE


@pytest.mark.parametrize("d,hq,hkv,n", [(128, 40, 8, 20011), (128, 180, 36, 4100), (128, 81, 9, 16449), (128, 90, 9, 16420), (128, 1000, 100, 1030),
                                        (128, 2250, 150, 1030), (128, 5, 1, 2049), (128, 4, 1, 1001), (128, 14, 2, 777), (128, 2, 2, 64),
                                        (128, 3, 1, 63), (64, 8, 2, 1037), (256, 6, 2, 1037)])
def test_scores_do_not_hang_on_the_cache_layout(d, hq, hkv, n):
    """The same logical rows in one tensor and in block pools of the smallest and of larger blocks: the same scores bit for bit,
    by the score call and by the compress call, and the same kept set.  Passes of five and of four query heads in
    registers, several of them and spare workgroups, and passes with fragments in LDS; heads whose last tile is short (it ends
    at the head's last row in one tensor and starts at a multiple of the tile in pools)."""
    import torch
    from ea_inputs import make_block_pools
    cfg = CONFIGS["c2"].with_(n_q_heads=hq, n_kv_heads=hkv, head_dim=d)
    w = min(n, 40)
    lay = make_layer(cfg, n=n, window=w)
    p = P.params_for(cfg, epsilon=0.02)
    ws = P.workspace(p, n, w)
    win = (P.to_dev(lay["q_win"]), w, lay["q_pos0"], P.to_dev(lay["inv_freq"]), lay["t_next"])
    mu, sigma = torch.empty(1, hq, d, device="cuda"), torch.empty(1, hq, d, d, device="cuda")
    ea.query_stats(p, *win, mu, sigma, ws)
    want, fused, got = (torch.empty(1, hkv, n, device="cuda") for _ in range(3))
    n_keep = (n + 1) // 2
    kept, other = (torch.empty(1, hkv, n_keep, dtype=torch.int32, device="cuda") for _ in range(2))
    ea.score(p, P.to_dev(lay["k"]), P.to_dev(lay["v"]), n, n, mu, sigma, want, ws)
    ea.compress_layer(p, *win, P.to_dev(lay["k"]), P.to_dev(lay["v"]), n, n, n_keep, fused, kept, ws)
    for bs in (16, 64):
        kp, vp, tab, nb = make_block_pools(lay["k"], lay["v"], bs, n + bs)
        table = torch.from_numpy(tab).cuda()
        pools = (P.to_dev(kp), P.to_dev(vp), ea.make_paged(table, bs, nb))
        ea.score_paged(p, *pools, n, mu, sigma, got, ws)
        torch.cuda.synchronize()
        assert torch.equal(got, want), bs
        ea.compress_layer_paged(p, *win, *pools, n, n_keep, 0, got, other, None, ws)
        torch.cuda.synchronize()
        assert torch.equal(got, fused) and torch.equal(other, kept), bs


def test_adaptive_selection_does_not_search_every_head_in_every_block():
    """Floors close to the budget put most heads' thresholds into the bin of the pool's: the selection then takes about what it
    takes with floors of a quarter, where few heads share it (137 and 156 us; 154 and 928 when every block of scores
    searched through all of the heads that do).  Three times as long is the limit: far from either."""
    import torch
    cfg = CONFIGS["c2"].with_(n_q_heads=512, n_kv_heads=512)
    p, n = P.params_for(cfg), 9000
    torch.manual_seed(3)
    sc = (torch.exp(2 * torch.randn(1, 512, n, device="cuda")) / n + 0.02) * torch.exp(0.5 * torch.randn(1, 512, n, device="cuda"))
    ws = P.workspace(p, n, 1)
    idx, lengths = torch.empty(1, 512, n, dtype=torch.int32, device="cuda"), torch.empty(1, 512, dtype=torch.int32, device="cuda")

    def fastest(floor):
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                ea.select_adaptive(p, sc, n, n // 2, floor, idx, lengths, ws)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    assert fastest(n // 2 * 9 // 10) < 3 * fastest(n // 8)
