"""Parity of the speculation-phase and verification-rule entry points (affinity table, nearest
draft expert, draft routing, sampling-based acceptance, greedy head, active-expert volume)
against the CPU oracle.  Needs an MI355X:  python -m pytest tests -m gpu"""
import numpy as np
import pytest
import torch

import paper_2604_10152_amd as sm
from oracle import moe_verify_oracle as orc
from workloads import synth
from _util import TOL, LazyF64, dev, f64, row_rel_err

pytestmark = pytest.mark.gpu
I32 = torch.int32
AFFINITY_RTOL = 1e-6     # fp64 sums on both sides, one rounding of the distance to fp32;
                         # the kernel squares 4 or 8 differences in fp32 before widening


def _say(msg):
    print(f"[case] {msg}", flush=True)


def _weights(E, d, f, dtype, seed, planted=True):
    g = torch.Generator(device="cpu").manual_seed(seed)
    mk = lambda *shape: (torch.randn(*shape, generator=g) * 0.02).to(dtype)
    wg, wu, wd = mk(E, f, d), mk(E, f, d), mk(E, d, f)
    if planted and E >= 4:
        # expert 3 is a copy of expert 1; expert 2 is expert 0 plus a small perturbation
        for w in (wg, wu, wd):
            w[3] = w[1]
            w[2] = (w[0].float() + 0.002 * torch.randn(w[0].shape, generator=g)).to(dtype)
    return wg, wu, wd


def _gpu_affinity(wg, wu, wd):
    E = wg.shape[0]
    table = torch.full((E, E), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty((sm.moe_affinity_table_workspace_bytes(E),), dtype=torch.uint8, device="cuda")
    sm.moe_affinity_table(dev(wg), dev(wu), dev(wd), table, ws)
    torch.cuda.synchronize()
    return table.cpu().numpy()


# ------------------------------------------------------------------ n2 affinity table
@pytest.mark.parametrize("E,d,f,dtype", [(8, 256, 512, torch.float32), (12, 128, 192, torch.bfloat16),
                                         (5, 64, 64, torch.bfloat16), (64, 128, 64, torch.bfloat16),
                                         (17, 20, 12, torch.float32)])
def test_affinity_table_matches_oracle(E, d, f, dtype):
    _say(f"affinity table E={E} d={d} f={f} {dtype}")
    wg, wu, wd = _weights(E, d, f, dtype, seed=100 + E)
    got = _gpu_affinity(wg, wu, wd)
    want = orc.affinity_table(f64(wg), f64(wu), f64(wd))
    assert np.all(np.diag(got) == 0) and np.array_equal(got, got.T)
    np.testing.assert_allclose(got, want, rtol=AFFINITY_RTOL, atol=0)
    if E >= 4:
        assert got[1, 3] == 0


def test_affinity_table_cfg3_shape_sampled_pairs():
    """Full fine-grained shape (64 experts x 3 x 2048 x 1408, bf16): the oracle evaluates a seeded
    sample of pairs; symmetry and the zero diagonal are checked on the whole table."""
    cfg = synth.CONFIGS[3]
    _say("affinity table cfg3 full shape")
    L = synth.make_layer(cfg, "cuda", seed=3)
    got = _gpu_affinity(L["w_gate"], L["w_up"], L["w_down"])
    assert np.all(np.diag(got) == 0) and np.array_equal(got, got.T) and np.all(np.isfinite(got))
    rng = np.random.default_rng(5)
    for _ in range(6):
        i, j = rng.choice(cfg.E, size=2, replace=False)
        sq = 0.0
        for W in (L["w_gate"], L["w_up"], L["w_down"]):
            sub = orc.affinity_table([f64(W[i]), f64(W[j])], [np.zeros(1)] * 2, [np.zeros(1)] * 2)
            sq += sub[0, 1] ** 2
        assert got[i, j] == pytest.approx(np.sqrt(sq), rel=AFFINITY_RTOL)
    # i.i.d. N(0, 0.02^2) weights: every distance is close to 0.02 * sqrt(2 * 3*d*f)
    off = got[~np.eye(cfg.E, dtype=bool)]
    assert np.allclose(off, 0.02 * np.sqrt(6.0 * cfg.d_model * cfg.d_ff), rtol=5e-3)


# ------------------------------------------------------------------ n2 nearest draft expert
def _gpu_remap(table, draft_ids):
    E = table.shape[0]
    remap = torch.full((E,), -9, dtype=I32, device="cuda")
    sm.moe_nearest_draft_expert(torch.from_numpy(table.astype(np.float32)).cuda(),
                                torch.tensor(draft_ids, dtype=I32, device="cuda"), remap)
    torch.cuda.synchronize()
    return remap.cpu().numpy()


def test_nearest_draft_expert_matches_oracle():
    _say("nearest draft expert")
    rng = np.random.default_rng(11)
    for E in (4, 8, 64, 130, 1024):
        A = rng.integers(1, 6, size=(E, E)).astype(np.float32)      # few values -> many exact ties
        A = np.triu(A, 1) + np.triu(A, 1).T
        for N in sorted({1, 2, max(1, E // 4), E}):
            draft = rng.permutation(E)[:N].tolist()                  # unsorted
            got = _gpu_remap(A, draft)
            want = orc.nearest_draft_expert(A.astype(np.float64), draft)
            assert np.array_equal(got, want), (E, N)
    # ids outside [0, E) are ignored
    A = np.array([[0, 2, 1], [2, 0, 3], [1, 3, 0]], dtype=np.float32)
    assert _gpu_remap(A, [7, 2, -1]).tolist() == [2, 2, 2]


@pytest.mark.parametrize("N", [1, 2, 3, 16, 17, 64, 65, 130])
def test_nearest_draft_expert_in_steps(N):
    """Ids are taken 64 and distances 2 or 16 at a time: whole and partial steps, with invalid
    ids and repeats among them."""
    _say(f"nearest draft expert, {N} ids")
    rng = np.random.default_rng(N)
    E = 140
    A = rng.integers(1, 4, size=(E, E)).astype(np.float32)
    A = np.triu(A, 1) + np.triu(A, 1).T
    for _ in range(4):
        draft = rng.integers(-3, E + 3, size=N).tolist()
        draft[-1] = int(rng.integers(0, E))
        valid = [q for q in draft if 0 <= q < E]
        assert np.array_equal(_gpu_remap(A, draft), orc.nearest_draft_expert(A.astype(np.float64), valid))
    assert _gpu_remap(A, [-1] * (N - 1) + [E]).tolist() == list(range(E))       # none valid: identity


# ------------------------------------------------------------------ n2 draft routing and layer
def _draft_setup(cfg, seed, n_draft):
    """Verification pass -> hot experts -> remap, all on the GPU; returns the pieces."""
    L = synth.make_layer(cfg, "cuda", seed=seed)
    layer = sm.MoEVerifyLayer(cfg.T, cfg.d_model, cfg.d_ff, cfg.E, cfg.k, cfg.torch_dtype,
                              renorm=cfg.renorm)
    layer.forward(L["x"], L["w_router"], L["w_gate"], L["w_up"], L["w_down"], L["bias"])
    hot = torch.empty((n_draft,), dtype=I32, device="cuda")
    sm.moe_hot_experts(layer.expert_offsets, hot)
    table = torch.empty((cfg.E, cfg.E), dtype=torch.float32, device="cuda")
    ws = torch.empty((sm.moe_affinity_table_workspace_bytes(cfg.E),), dtype=torch.uint8, device="cuda")
    sm.moe_affinity_table(L["w_gate"], L["w_up"], L["w_down"], table, ws)
    remap = torch.empty((cfg.E,), dtype=I32, device="cuda")
    sm.moe_nearest_draft_expert(table, hot, remap)
    torch.cuda.synchronize()
    return L, layer, hot, table, remap


@pytest.mark.parametrize("cfg_id,n_draft", [(1, 3), (3, 16), (3, 6), (2, 2)])
def test_draft_routing_matches_oracle(cfg_id, n_draft):
    """The real chain: counts of a verification pass choose the draft experts (HotTemporal), the
    table maps every other expert to one of them, the draft router uses the map.  The oracle
    gets the GPU's fp32 table (the table itself is checked above), so ids must match exactly."""
    cfg = synth.CONFIGS[cfg_id]
    _say(f"draft routing cfg{cfg_id} N={n_draft}")
    L, layer, hot, table, remap = _draft_setup(cfg, seed=cfg_id, n_draft=n_draft)
    counts = np.diff(layer.expert_offsets.cpu().numpy())
    hot_want = orc.hot_experts(counts, n_draft)
    assert np.array_equal(hot.cpu().numpy(), hot_want)
    tab64 = table.cpu().numpy().astype(np.float64)
    assert np.array_equal(remap.cpu().numpy(), orc.nearest_draft_expert(tab64, hot_want))
    idx = torch.full((cfg.T, cfg.k), -1, dtype=I32, device="cuda")
    w = torch.full((cfg.T, cfg.k), -1.0, dtype=torch.float32, device="cuda")
    sm.moe_route_topk_draft(L["x"], L["w_router"], L["bias"], cfg.k, cfg.renorm, remap, idx, w)
    torch.cuda.synchronize()
    bias = None if L["bias"] is None else f64(L["bias"])
    idx_want, w_want = orc.route_topk_draft(f64(L["x"]), f64(L["w_router"]), cfg.k, hot_want,
                                            tab64, bias, cfg.renorm)
    assert np.array_equal(idx.cpu().numpy(), idx_want)
    np.testing.assert_allclose(w.cpu().numpy(), w_want, rtol=2e-6, atol=0)
    assert set(np.unique(idx_want)) <= set(hot_want.tolist())


@pytest.mark.parametrize("cfg_id,n_draft,n_tok", [(1, 3, 16), (3, 16, 24)])
def test_draft_layer_matches_oracle(cfg_id, n_draft, n_tok):
    """Whole MoE block in draft mode (only the N resident experts compute) against the oracle on
    the first n_tok tokens (tokens are independent)."""
    cfg = synth.CONFIGS[cfg_id]
    _say(f"draft layer cfg{cfg_id} N={n_draft}")
    L, layer, hot, table, remap = _draft_setup(cfg, seed=cfg_id, n_draft=n_draft)
    out = layer.forward(L["x"], L["w_router"], L["w_gate"], L["w_up"], L["w_down"], L["bias"],
                        draft_remap=remap)
    torch.cuda.synchronize()
    counts = np.diff(layer.expert_offsets.cpu().numpy())
    assert set(np.nonzero(counts)[0].tolist()) <= set(hot.cpu().numpy().tolist())
    bias = None if L["bias"] is None else f64(L["bias"])
    want, idx_want, _ = orc.moe_layer_draft(
        f64(L["x"][:n_tok]), f64(L["w_router"]), LazyF64(L["w_gate"]), LazyF64(L["w_up"]),
        LazyF64(L["w_down"]), cfg.k, hot.cpu().numpy(), table.cpu().numpy().astype(np.float64),
        bias, cfg.renorm)
    assert np.array_equal(layer.topk_idx[:n_tok].cpu().numpy(), idx_want)
    err = row_rel_err(out[:n_tok].float().cpu().numpy(), want)
    print(f"   draft layer row error {err:.3e}")
    assert err <= TOL[cfg.torch_dtype]


# ------------------------------------------------------------------ n3 sampling-based acceptance
def _gpu_accept_sample(draft, pd, pt, ua, us):
    B, gp1, V = pt.shape
    alen = torch.full((B,), -7, dtype=I32, device="cuda")
    out = torch.full((B, gp1), -7, dtype=I32, device="cuda")
    sm.spec_accept_sample(dev(draft), dev(pd), dev(pt), dev(ua), dev(us), alen, out)
    torch.cuda.synchronize()
    return alen.cpu().numpy(), out.cpu().numpy()


def _draw_is_valid(weights, u, tok):
    """tok is a correct inverse-CDF draw up to the rounding of the running sums."""
    c = np.cumsum(np.asarray(weights, dtype=np.float64))
    thr = np.float64(u) * c[-1]
    below = c[tok - 1] if tok > 0 else 0.0
    return weights[tok] > 0 and below <= thr * (1 + 1e-12) and c[tok] >= thr * (1 - 1e-12)


def _sample_case(B, gamma, V, seed, sharp=1.0, agree=0.6):
    g = torch.Generator(device="cpu").manual_seed(seed)
    pt = torch.softmax(torch.randn(B, gamma + 1, V, generator=g) * sharp, dim=-1)
    pd = torch.softmax(torch.log(pt[:, :gamma]) + 0.7 * torch.randn(B, gamma, V, generator=g), dim=-1)
    draft = torch.multinomial(pd.reshape(-1, V), 1, generator=g).reshape(B, gamma).to(I32) \
        if gamma > 0 else torch.zeros((B, 0), dtype=I32)
    ua = torch.rand(B, gamma, generator=g)
    us = torch.rand(B, generator=g)
    return draft, pd.contiguous(), pt.contiguous(), ua, us


@pytest.mark.parametrize("B,gamma,V,sharp", [(64, 5, 1000, 2.0), (8, 7, 32000, 3.0), (33, 1, 17, 1.0),
                                              (16, 0, 50, 1.0), (4, 64, 300, 2.0), (256, 7, 4096, 4.0)])
def test_accept_sample_matches_oracle(B, gamma, V, sharp):
    _say(f"spec_accept_sample B={B} gamma={gamma} V={V}")
    draft, pd, pt, ua, us = _sample_case(B, gamma, V, seed=B * 131 + gamma, sharp=sharp)
    a, o = _gpu_accept_sample(draft, pd, pt, ua, us)
    ea, eo = orc.accept_sample(draft.numpy(), pd.numpy(), pt.numpy(), ua.numpy(), us.numpy())
    assert np.array_equal(a, ea)                       # the keep tests are exact on both sides
    assert a.min() >= 1 and a.max() <= gamma + 1
    if gamma >= 5 and B >= 64:
        assert len(np.unique(a)) >= 3                  # the case exercises several lengths
    for b in range(B):
        n = ea[b] - 1
        assert np.array_equal(o[b, :n], eo[b, :n]) and np.all(o[b, n + 1:] == -1)
        if o[b, n] != eo[b, n]:                        # only legitimate on a rounding boundary
            wts = np.maximum(pt[b, n].double().numpy() - pd[b, n].double().numpy(), 0) \
                if n < gamma else pt[b, n].double().numpy()
            assert _draw_is_valid(wts, us[b].item(), int(o[b, n])), (b, o[b, n], eo[b, n])


def test_accept_sample_special_cases():
    _say("spec_accept_sample special cases")
    # point masses: the rule is the greedy rule (worked example of Fig. 4 included)
    V, gamma = 40, 5
    rng = np.random.default_rng(9)
    draft = rng.integers(0, V, size=(50, gamma)).astype(np.int32)
    target = rng.integers(0, V, size=(50, gamma + 1)).astype(np.int32)
    keep = rng.random(size=(50, gamma)) < 0.75
    target[:, :gamma] = np.where(keep, draft, target[:, :gamma])
    draft[0] = [10, 11, 12, 13, 14]
    target[0] = [10, 11, 12, 20, 21, 22]
    oh = lambda ids: torch.nn.functional.one_hot(torch.from_numpy(ids).long(), V).float()
    a, o = _gpu_accept_sample(torch.from_numpy(draft), oh(draft), oh(target),
                              torch.rand(50, gamma), torch.rand(50))
    ga, go = orc.accept(draft, target)
    assert np.array_equal(a, ga) and np.array_equal(o, go)
    assert a[0] == 4 and o[0].tolist() == [10, 11, 12, 20, -1, -1]
    # identical distributions: nothing can be rejected
    d2, pd, pt, ua, us = _sample_case(20, 4, 64, seed=77)
    pt[:, :4] = pd
    a, o = _gpu_accept_sample(d2, pd, pt, ua, us)
    assert np.all(a == 5) and np.array_equal(o[:, :4], d2.numpy())
    # a draft id outside the vocabulary is rejected at once
    d3 = d2.clone()
    d3[:, 0] = 64
    a, o = _gpu_accept_sample(d3, pd, pt, ua, us)
    assert np.all(a == 1) and np.all((o[:, 0] >= 0) & (o[:, 0] < 64)) and np.all(o[:, 1:] == -1)


# ------------------------------------------------------------------ n4 greedy head, active volume
@pytest.mark.parametrize("R,V,dtype", [(64, 32000, torch.bfloat16), (7, 1001, torch.bfloat16),
                                       (33, 4096, torch.float32), (5, 13, torch.float32),
                                       (2048, 32000, torch.bfloat16)])
def test_greedy_tokens_match_oracle(R, V, dtype):
    _say(f"spec_greedy_tokens R={R} V={V} {dtype}")
    g = torch.Generator(device="cuda").manual_seed(R + V)
    logits = (torch.randn(R, V, generator=g, device="cuda") * 3).to(dtype)
    if R <= 64:
        logits = torch.round(logits * 2) / 2            # coarse grid: many exact ties at the top
        logits = logits.to(dtype)
    tok = torch.full((R,), -5, dtype=I32, device="cuda")
    sm.spec_greedy_tokens(logits, tok)
    torch.cuda.synchronize()
    rows = range(R) if R <= 64 else range(0, R, 37)
    lf = logits.float().cpu().numpy()
    want = orc.greedy_tokens(lf[list(rows)])
    assert np.array_equal(tok.cpu().numpy()[list(rows)], want)
    # property at any size: the chosen logit is the row maximum and no lower id attains it
    mx = lf.max(axis=1)
    t = tok.cpu().numpy()
    assert np.all(lf[np.arange(R), t] == mx)
    assert np.all(t == (lf == mx[:, None]).argmax(axis=1))


@pytest.mark.parametrize("R,V,dtype", [(1100, 48008, torch.bfloat16), (1030, 24308, torch.float32),
                                       (1400, 48008, torch.float32)])
def test_greedy_tokens_of_many_long_rows(R, V, dtype):
    """From 100 MB (bf16) or 256 MiB (fp32) on the logits are read with the non-temporal hint."""
    _say(f"spec_greedy_tokens R={R} V={V} {dtype}")
    g = torch.Generator(device="cuda").manual_seed(R + V)
    logits = (torch.randn(R, V, generator=g, device="cuda") * 6).round().to(dtype) / 2       # ties at the top
    tok = torch.full((R,), -5, dtype=I32, device="cuda")
    sm.spec_greedy_tokens(logits, tok)
    ids = torch.arange(V, device="cuda")
    want = torch.where(logits == logits.amax(dim=1, keepdim=True), ids, V).amin(dim=1)
    assert torch.equal(tok.long(), want)


def test_active_expert_bytes_and_greedy_accept_chain():
    _say("active expert bytes + greedy head feeding spec_accept")
    for counts in ([3, 0, 5, 0, 0, 1, 2, 9], [0] * 64, list(range(130))):
        off = torch.from_numpy(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)).cuda()
        out = torch.full((1,), -1, dtype=torch.int64, device="cuda")
        per = 3 * 4096 * 14336 * 2
        sm.moe_active_expert_bytes(off, per, out)
        torch.cuda.synchronize()
        assert int(out.item()) == orc.active_expert_bytes(counts, per)
    # logits -> greedy target tokens -> greedy acceptance, against the oracle's chain
    B, gamma, V = 32, 4, 500
    g = torch.Generator(device="cpu").manual_seed(5)
    logits = torch.randn(B * (gamma + 1), V, generator=g)
    tgt_want = orc.greedy_tokens(logits.numpy()).reshape(B, gamma + 1)
    draft = torch.from_numpy(tgt_want[:, :gamma].copy())
    flip = torch.rand(B, gamma, generator=g) < 0.3
    draft = torch.where(flip, (draft + 1) % V, draft).to(I32)
    tok = torch.empty((B * (gamma + 1),), dtype=I32, device="cuda")
    sm.spec_greedy_tokens(logits.cuda(), tok)
    alen = torch.empty((B,), dtype=I32, device="cuda")
    out = torch.empty((B, gamma + 1), dtype=I32, device="cuda")
    sm.spec_accept(draft.cuda(), tok.view(B, gamma + 1), alen, out)
    torch.cuda.synchronize()
    ea, eo = orc.accept(draft.numpy(), tgt_want)
    assert np.array_equal(alen.cpu().numpy(), ea) and np.array_equal(out.cpu().numpy(), eo)


# ------------------------------------------------------------------ affinity table: edges
@pytest.mark.parametrize("E,d,f,dtype", [
    (1, 64, 64, torch.bfloat16), (2, 64, 64, torch.bfloat16), (4, 72, 40, torch.bfloat16),
    (8, 264, 24, torch.bfloat16), (9, 256, 64, torch.bfloat16), (16, 128, 72, torch.bfloat16),
    (33, 64, 192, torch.bfloat16), (49, 64, 128, torch.float32), (65, 64, 64, torch.bfloat16),
    (140, 24, 32, torch.float32), (3, 4, 1, torch.float32)])
def test_affinity_table_operand_edges(E, d, f, dtype):
    """One to four 16-expert row blocks per wave, column slices for 4 and 8 experts, a second and
    third group of 64 experts, and column counts that end inside a unit of 16 or 32 columns."""
    _say(f"affinity edges E={E} d={d} f={f} {dtype}")
    wg, wu, wd = _weights(E, d, f, dtype, seed=200 + E, planted=E >= 9)
    got = _gpu_affinity(wg, wu, wd)
    want = orc.affinity_table(f64(wg), f64(wu), f64(wd))
    assert np.all(np.diag(got) == 0) and np.array_equal(got, got.T)
    np.testing.assert_allclose(got, want, rtol=AFFINITY_RTOL, atol=0)


def test_affinity_table_close_pairs_and_non_finite_weights():
    """Pairs far below their norms (a copy, one element off by one bf16 step, a 1e-4 relative
    offset; with and without a common part in all experts) keep the accuracy of a direct sum, and
    an infinite or NaN weight reaches exactly the pairs of its expert."""
    _say("affinity close pairs, non-finite weights")
    E, d, f = 12, 128, 192
    for common in (0.0, 1.0):
        wg, wu, wd = (w.float() for w in _weights(E, d, f, torch.float32, seed=7, planted=False))
        for w in (wg, wu, wd):
            w += common * w[0].clone() * 50
            w[5] = w[4]
            w[7] = w[6]
            w[9] = w[8] * (1 + 1e-4)
        wg[7, 3, 5] *= 1 + 2.0 ** -7
        got = _gpu_affinity(wg, wu, wd)
        want = orc.affinity_table(f64(wg), f64(wu), f64(wd))
        assert got[4, 5] == 0 and got[6, 7] > 0
        np.testing.assert_allclose(got, want, rtol=AFFINITY_RTOL, atol=0)
    for bad in (float("inf"), float("nan")):
        for e in (0, 6):
            w2 = wu.clone()
            w2[e, 1, 2] = bad
            got = _gpu_affinity(wg, w2, wd)
            hit = np.zeros((E, E), dtype=bool)
            hit[e, :] = hit[:, e] = True
            hit[e, e] = False
            assert np.array_equal(~np.isfinite(got), hit) and (not np.isinf(bad) or np.all(got[hit] == np.inf))
            np.testing.assert_allclose(got[~hit], want[~hit], rtol=AFFINITY_RTOL, atol=0)
    w2 = wu.clone()
    w2[2, 1, 2] = w2[3, 1, 3] = float("inf")       # both infinite, at different places
    assert _gpu_affinity(wg, w2, wd)[2, 3] == np.inf


# fp32 rounds a distance by at most 2^-24; the integer products may move it by 2^-27
EXACT_RTOL = 2.0 ** -24 + 4 * 2.0 ** -27


@pytest.mark.parametrize("kind", ["normal", "heavy tails", "spikes", "scales", "sparse", "steps", "huge and tiny"])
@pytest.mark.parametrize("E,d,f", [(9, 520, 561), (16, 264, 601), (17, 376, 401), (33, 264, 288), (49, 256, 200),
                                   (64, 512, 128)])
def test_affinity_table_integer_products(E, d, f, kind):
    """The integer form (from 2.5 million weights per matrix on), one to four row blocks, whole and ragged
    last units, and values that change the scale of a row again and again."""
    assert E * d * f >= 2500000
    _say(f"affinity, integer products E={E} d={d} f={f} {kind}")
    g = torch.Generator().manual_seed(E + d)
    W = []
    for shape in ((E, f, d), (E, f, d), (E, d, f)):
        w = torch.randn(shape, generator=g) * 0.02
        if kind == "heavy tails":
            w = w * torch.exp(2 * torch.randn(shape, generator=g))
        elif kind == "spikes":
            w = torch.where(torch.rand(shape, generator=g) < 0.01, w * 3000, w)
        elif kind == "scales":                     # experts of different magnitude
            w = w * (10.0 ** torch.linspace(-3, 3, E)).view(-1, 1, 1)
        elif kind == "sparse":
            w = w * (torch.rand(shape, generator=g) < 0.03)
        elif kind == "steps":                      # magnitude changes along the columns
            w = w * 2.0 ** (torch.arange(w[0].numel()) // 100 % 7 * 4 - 12).view(1, *shape[1:])
        elif kind == "huge and tiny":              # more than 2^100 apart, in one unit
            w = w * torch.where(torch.rand(shape, generator=g) < 0.5, 1e-34, 1.0)
            w[:, 0, :2] *= 1e32
        W.append(w.to(torch.bfloat16))
    got = _gpu_affinity(*W)
    want = orc.affinity_table(*(f64(w) for w in W))
    assert np.all(np.diag(got) == 0) and np.array_equal(got, got.T)
    np.testing.assert_allclose(got, want, rtol=EXACT_RTOL, atol=0)


def _structured(kind, E, d, f):
    """Weights whose low bits are alike from column to column or row to row (d, f: multiples of 64)."""
    g = torch.Generator().manual_seed(E)
    W = []
    for shape in ((E, f, d), (E, f, d), (E, d, f)):
        col = torch.arange(shape[2])
        odd = torch.isin(col % 8, torch.tensor([1, 3, 4, 6]))
        if kind == "half the columns":             # and a large value in one of 64
            sign = torch.randint(0, 2, shape, generator=g) * 2.0 - 1
            w = torch.where(col % 64 == 1, torch.ones(shape), torch.where(odd, sign * 255 * 2.0 ** -20, 0.0))
            w[0] = 0
        elif kind == "outlier channels":           # of expert 0, larger still in its first rows
            w = torch.randn(shape, generator=g) * 0.02 * odd
            w[0, :, torch.isin(col % 64, torch.tensor([1, 9, 17, 25]))] = 20
            if not W:
                w[0, :shape[1] // 11, torch.isin(col % 64, torch.tensor([1, 9, 17, 25]))] = 280
        else:                                      # expert 0 small and constant, the others zero or positive
            w = (torch.rand(shape, generator=g) + 1) * (torch.rand(shape, generator=g) < 0.5)
            w[0] = 0.4 * 2.0 ** -19
            if kind == "one sign, larger at first" and not W:
                w[1:, :shape[1] // 4] *= 4
        W.append(w.to(torch.bfloat16))
    return W


@pytest.mark.parametrize("kind", ["half the columns", "outlier channels", "one sign", "one sign, larger at first"])
@pytest.mark.parametrize("E,d,f", [(9, 512, 576), (64, 256, 192)])
def test_affinity_table_structured_residuals(E, d, f, kind):
    """Whatever the integer form cannot hold of a weight, in whichever columns and with whatever signs: D moves
    by at most 2^-27 of it, then by the rounding to fp32."""
    assert E * d * f >= 2500000
    _say(f"affinity, structured residuals E={E} d={d} f={f} {kind}")
    W = _structured(kind, E, d, f)
    got = _gpu_affinity(*W)
    want = orc.affinity_table(*(f64(w) for w in W))
    assert np.all(np.diag(got) == 0) and np.array_equal(got, got.T)
    np.testing.assert_allclose(got, want, rtol=2.0 ** -24 + 2.0 ** -27, atol=0)


@pytest.mark.parametrize("E,d,f", [(9, 520, 561), (17, 376, 401), (33, 264, 288), (64, 512, 128)])
def test_affinity_table_integer_products_non_finite(E, d, f):
    """The integer form with infinite and NaN weights, in expert 0, in the middle and in the last row block, in the
    first columns and in the last (ragged) unit: exactly the pairs of their experts are reached."""
    assert E * d * f >= 2500000
    _say(f"affinity, integer products, non-finite E={E} d={d} f={f}")
    wg, wu, wd = _weights(E, d, f, torch.bfloat16, seed=E, planted=False)
    want = orc.affinity_table(f64(wg), f64(wu), f64(wd))
    for bad in (float("inf"), -float("inf"), float("nan")):
        for e, at in ((0, (0, 0)), (E // 2, (f - 1, d - 1)), (E - 1, (f // 2, d // 2))):
            w2 = wu.clone()
            w2[(e,) + at] = bad
            got = _gpu_affinity(wg, w2, wd)
            hit = np.zeros((E, E), dtype=bool)
            hit[e, :] = hit[:, e] = True
            hit[e, e] = False
            assert np.array_equal(~np.isfinite(got), hit), (bad, e)
            assert np.all(got[hit] == np.inf) if np.isinf(bad) else np.all(np.isnan(got[hit]))
            np.testing.assert_allclose(got[~hit], want[~hit], rtol=EXACT_RTOL, atol=0)
    w2 = wu.clone()
    w2[1, 3, 5] = w2[E - 1, 4, 6] = float("inf")       # two experts, at different places: infinite
    w2[2, 7, 9] = w2[3, 7, 9] = float("inf")           # at the same place: no difference
    got = _gpu_affinity(wg, w2, wd)
    assert got[1, E - 1] == np.inf and got[1, 2] == np.inf and np.isnan(got[2, 3])
    ok = [e for e in range(E) if e not in (1, 2, 3, E - 1)]
    np.testing.assert_allclose(got[np.ix_(ok, ok)], want[np.ix_(ok, ok)], rtol=EXACT_RTOL, atol=0)


def test_affinity_table_integer_products_long_sums():
    """More columns per team than the int32 sums hold (28672), all products of one sign."""
    E, d, f = 9, 4096, 14336
    assert 3 * d * f > 256 * 16 * 28672
    _say(f"affinity, integer products, long sums E={E} d={d} f={f}")
    g = torch.Generator(device="cuda").manual_seed(1)
    W = [torch.rand(s, generator=g, device="cuda", dtype=torch.bfloat16) + 1 for s in ((E, f, d), (E, f, d), (E, d, f))]
    table = torch.empty((E, E), dtype=torch.float32, device="cuda")
    ws = torch.empty((sm.moe_affinity_table_workspace_bytes(E),), dtype=torch.uint8, device="cuda")
    sm.moe_affinity_table(*W, table, ws)
    for i, j in ((0, 1), (0, 8), (3, 8), (5, 6)):
        sq = sum(float((w[i].double() - w[j].double()).square_().sum()) for w in W)
        assert abs(float(table[i, j]) - sq ** 0.5) <= EXACT_RTOL * sq ** 0.5, (i, j)


def _many_close(kind, wg, wu, wd):
    E = wg.shape[0]
    for w in (wg, wu, wd):
        if kind == "outlier":                      # expert 0 lies far from all others
            w[0] *= 5000.0
        elif kind == "clusters":                   # copies of the first eight
            w[:] = w[torch.arange(E, device=w.device) % 8]
        elif kind == "half":                       # copies of one expert, each off by a little
            w[E // 2:] = w[E // 2] * (1 + 1e-4 * torch.arange(E - E // 2, device=w.device)
                                      .view(-1, 1, 1)).to(w.dtype)
        elif kind == "last pair":
            w[E - 1] = w[E - 2]


@pytest.mark.parametrize("kind", ["outlier", "clusters", "half", "last pair"])
@pytest.mark.parametrize("E,d,f,dtype", [(9, 64, 64, torch.bfloat16), (17, 24, 20, torch.float32),
                                         (40, 64, 68, torch.float32), (64, 128, 96, torch.bfloat16),
                                         (70, 256, 512, torch.bfloat16)])
def test_affinity_table_many_close_pairs(E, d, f, dtype, kind):
    """Blocks of close pairs: whole, at the ragged end of the table, with fewer columns than
    partial sums and with slabs that cross from one matrix to the next."""
    _say(f"affinity {kind} E={E} d={d} f={f} {dtype}")
    W = _weights(E, d, f, dtype, seed=300 + E, planted=False)
    _many_close(kind, *W)
    got = _gpu_affinity(*W)
    want = orc.affinity_table(*(f64(w) for w in W))
    assert np.all(np.diag(got) == 0) and np.array_equal(got, got.T)
    np.testing.assert_allclose(got, want, rtol=AFFINITY_RTOL, atol=0)


def test_affinity_table_cost_of_close_pairs():
    """A table full of close pairs costs a few times one without (measured 3.6), not the tens
    of times that it takes to sum the pairs one after the other."""
    _say("affinity, cost of close pairs")
    g = torch.Generator(device="cuda").manual_seed(3)
    E, d, f = 64, 2048, 704
    W = [(torch.randn(s, generator=g, device="cuda") * 0.02).to(torch.bfloat16)
         for s in ((E, f, d), (E, f, d), (E, d, f))]
    table = torch.empty((E, E), dtype=torch.float32, device="cuda")
    ws = torch.empty((sm.moe_affinity_table_workspace_bytes(E),), dtype=torch.uint8, device="cuda")

    def median_ms():
        t = []
        for _ in range(7):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            sm.moe_affinity_table(*W, table, ws)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return sorted(t)[3]

    plain = median_ms()
    _many_close("outlier", *W)
    close = median_ms()
    print(f"   {plain:.3f} ms -> {close:.3f} ms")
    assert close <= 8 * plain


@pytest.mark.parametrize("B,gamma,V", [(9, 3, 4096), (9, 3, 4097), (3, 2, 32769), (5, 1, 40003), (2, 1, 524288),
                                       (2, 1, 540672)])
def test_accept_sample_vocabulary_edges(B, gamma, V):
    """One tile per wave and one more, a second burst of tiles, rows without 16-byte alignment, and
    the last vocabulary whose tile sums fit in LDS and a larger one; u_sample at both ends."""
    _say(f"spec_accept_sample edges B={B} gamma={gamma} V={V}")
    draft, pd, pt, ua, us = _sample_case(B, gamma, V, seed=V, sharp=3.0)
    us[0] = 0.0
    us[1] = 1.0 - 2.0 ** -24
    a, o = _gpu_accept_sample(draft, pd, pt, ua, us)
    ea, eo = orc.accept_sample(draft.numpy(), pd.numpy(), pt.numpy(), ua.numpy(), us.numpy())
    assert np.array_equal(a, ea)
    for b in range(B):
        n = ea[b] - 1
        assert np.array_equal(o[b, :n], eo[b, :n]) and np.all(o[b, n + 1:] == -1)
        if o[b, n] != eo[b, n]:                        # only legitimate on a rounding boundary
            wts = np.maximum(pt[b, n].double().numpy() - pd[b, n].double().numpy(), 0) \
                if n < gamma else pt[b, n].double().numpy()
            assert _draw_is_valid(wts, us[b].item(), int(o[b, n])), (b, o[b, n], eo[b, n])


@pytest.mark.parametrize("R,V,dtype", [(1024, 8192, torch.bfloat16), (1025, 8192, torch.bfloat16),
                                       (640, 8192, torch.bfloat16), (641, 8192, torch.bfloat16),
                                       (642, 49160, torch.float32),
                                       (3, 8200, torch.bfloat16), (2, 4100, torch.float32)])
def test_greedy_tokens_burst_edges(R, V, dtype):
    """Rows at the edge of the burst rule, and a burst whose last chunks lie beyond the row."""
    _say(f"spec_greedy_tokens edges R={R} V={V}")
    g = torch.Generator().manual_seed(R + V)
    logits = torch.round(torch.randn(R, V, generator=g) * 2).to(dtype)     # many exact ties
    logits[0] = 0
    logits[-1, -1] = 50
    tok = torch.full((R,), -5, dtype=I32, device="cuda")
    sm.spec_greedy_tokens(dev(logits), tok)
    torch.cuda.synchronize()
    assert np.array_equal(tok.cpu().numpy(), orc.greedy_tokens(logits.float().numpy()))


def _wave_scan_witnesses(m, n=30000):
    """Tile sums for which a log-step scan over 64 lanes passes half of its total on a tile that
    holds nothing: the first m tiles, zeros, and a permutation of the first m."""
    rng = np.random.default_rng(5)
    w = np.zeros((n, 64))
    w[:, :m] = (rng.random((n, m)) * 10.0 ** rng.uniform(-9, 0, (n, m))).astype(np.float32)
    w[:, 64 - m:] = rng.permuted(w[:, :m], axis=1)
    s = w.copy()
    for off in (1, 2, 4, 8, 16, 32):
        s[:, off:] = s[:, off:] + s[:, :-off].copy()
    first = (s > 0.5 * s[:, -1:]).argmax(axis=1)
    return w[w[np.arange(n), first] == 0]


def test_accept_sample_never_draws_from_empty_tiles():
    """Distributions with most ids at exactly zero (a truncated target, a residual): the running
    sums of the tiles move by a rounding over empty tiles, the draw must not land there."""
    _say("spec_accept_sample, empty tiles")
    w = np.concatenate([_wave_scan_witnesses(m)[:16] for m in (4, 8, 12, 20)])
    assert len(w) >= 16
    pt = torch.zeros(len(w), 1, 64 * 256)
    pt[:, 0, ::256] = torch.from_numpy(w.astype(np.float32))
    empty = torch.zeros(len(w), 0)
    a, o = _gpu_accept_sample(empty.to(I32), torch.zeros(len(w), 0, 64 * 256), pt, empty,
                              torch.full((len(w),), 0.5))
    assert np.all(a == 1)
    for b in range(len(w)):
        assert _draw_is_valid(pt[b, 0].double().numpy(), 0.5, int(o[b, 0])), (b, o[b, 0])


@pytest.mark.parametrize("V,keep", [(16384, 40), (40003, 300), (32000, 5), (4096, 17)])
def test_accept_sample_truncated_distributions(V, keep):
    """A few ids with weight among empty tiles and empty lanes, the uniform at their running sums."""
    _say(f"spec_accept_sample truncated V={V} keep={keep}")
    B = 64
    rng = np.random.default_rng(V + keep)
    pt = torch.zeros(B, 1, V)
    us = torch.zeros(B)
    for b in range(B):
        ids = np.sort(rng.choice(V, size=keep, replace=False))
        p = (rng.random(keep) * 10.0 ** rng.uniform(-9, 0, keep)).astype(np.float32)
        pt[b, 0, ids] = torch.from_numpy(p)
        c = np.cumsum(p.astype(np.float64))
        us[b] = min(float(np.float32(c[rng.integers(keep)] / c[-1])), 1.0 - 2.0 ** -24)
    empty = torch.zeros(B, 0)
    a, o = _gpu_accept_sample(empty.to(I32), torch.zeros(B, 0, V), pt, empty, us)
    assert np.all(a == 1)
    for b in range(B):
        assert _draw_is_valid(pt[b, 0].double().numpy(), us[b].item(), int(o[b, 0])), (b, o[b, 0])
