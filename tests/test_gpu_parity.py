"""GPU parity: every C-ABI entry point against the float64 oracle on the same seeded inputs.

Acceptance rules (float32 accumulation of 256 exact products bounds the score error by a few ulp of
sum |q k| * scale; everything downstream inherits that resolution):
  * page statistics: min/max bit-exact; mean and variance within 1 ulp of the storage dtype (bf16) or
    2e-6 relative to the page's value range (f32);
  * page scores: |gpu - oracle| <= 1e-5 * max(1, |score|);
  * selected page sets: identical, except pages whose score lies within 1e-5*max(1,|cut|) of the cut;
  * tau, tau_hat: |gpu - oracle| <= 4e-6 * max(1, |tau|);
  * supports: identical token lists; a token with |z - tau| <= 2e-6*max(1,|tau|) (float32 resolution
    of the score) may fall on either side -- the float32-cache inputs contain none (asserted);
  * outputs: ||gpu - oracle||_2 / ||oracle||_2 <= 1e-5 (f32 cache) or 2e-3 (bf16 cache);
  * dropped mass delta: 1e-4 absolute.
"""
import math
import numpy as np
import pytest
import torch

from oracle import entmaxkv_oracle as orc
from paper_2605_21649_amd import binding as ekv
from paper_2605_21649_amd import synth
from tests.helpers import (DeviceState, unit_kv, oracle_stats, storage_ulp, sets_equal_up_to_cut, rel_err,
                           to_f64, OUT_TOL, check_decode_unit, check_decode_of_gpu_list, pre_groups)

pytestmark = pytest.mark.gpu

W1 = synth.C1
W1S = synth.C1.scaled(name="C1-soft", scale=0.5 / math.sqrt(128.0))
W1R = synth.C1.scaled(name="C1-ragged", ragged=5, scale=0.5 / math.sqrt(128.0))
W2 = synth.C2.scaled(name="C2-8k", context=8192 + 16, ragged=3)
W3 = synth.C3.scaled(name="C3-small", batch=2, context=4096)
W5 = synth.C5.scaled(name="C5-small", batch=2, context=8192, alpha=1.25)
W5B = synth.C5.scaled(name="C5-small-a2", batch=2, context=4096, alpha=2.0, ragged=17)
W3A = synth.C3.scaled(name="C3-small-a43", batch=1, context=4096 + 32, ragged=9, alpha=4.0 / 3.0)   # beta = 3
ALL = [W1, W1S, W1R, W2, W3, W3A, W5, W5B]
IDS = [w.name for w in ALL]

_cache = {}


def get_inputs(w, seed=0):
    key = (w.name, seed)
    if key not in _cache:
        cfg_id = ["C1", "C2", "C3", "C4", "C5"].index(w.name[:2]) + 1
        _cache[key] = synth.make_inputs(w, 1000 * cfg_id + seed, device="cpu")
    return _cache[key]


def sample_units(w, k=6):
    units = [(b, h) for b in range(w.batch) for h in range(w.n_q_heads)]
    rng = np.random.default_rng(5)
    if len(units) > k:
        units = [units[i] for i in sorted(rng.choice(len(units), k, replace=False))]
    return units


def topk_budget(w):
    return max(2, min(w.pages_per_seq // 4, 2048 // w.page_size))


# ---------------------------------------------------------------------------- a1 / a2
@pytest.mark.parametrize("w", ALL, ids=IDS)
def test_stats_build(w):
    inp = get_inputs(w)
    st = DeviceState(w, inp)
    ekv.ekv_stats_build(st.cfg, st.cache(), st.stats())
    torch.cuda.synchronize()
    box = to_f64(st.box_stats); gauss = to_f64(st.gauss_stats)
    for b in range(w.batch):
        for h in range(0, w.n_kv_heads, 3):
            kmin, kmax, kavg, kstd, cnt = oracle_stats(inp, w, b, h)
            M = len(cnt)
            np.testing.assert_array_equal(box[b, h, :M, 0], kmin)
            np.testing.assert_array_equal(box[b, h, :M, 1], kmax)
            kvar = kstd ** 2                               # the variance is what the library stores
            if w.kv_dtype == "bf16":
                tol_avg = storage_ulp(kavg, "bf16"); tol_var = storage_ulp(kvar, "bf16")
            else:
                rng_ = (kmax - kmin) + 1e-30
                tol_avg = 2e-6 * np.maximum(np.abs(kavg), rng_); tol_var = 4e-6 * rng_ ** 2
            assert np.all(np.abs(gauss[b, h, :M, 0] - kavg) <= tol_avg)
            assert np.all(np.abs(gauss[b, h, :M, 1] - kvar) <= tol_var)


@pytest.mark.parametrize("w", [W1R, W2], ids=["C1-ragged", "C2-8k"])
def test_stats_append_equals_rebuild(w):
    inp = get_inputs(w)
    st = DeviceState(w, inp)
    dev = st.box.device
    n_final = int(inp["seq_lens"][0])
    steps = w.page_size + 3                         # crosses a page boundary
    n0 = n_final - steps
    # the tokens to append are the ones already sitting in the cache; wipe their slots first
    B, Hkv, d = w.batch, w.n_kv_heads, w.head_dim
    k_log = torch.stack([torch.stack([synth.logical_kv(inp, w, b, h)[0] for h in range(Hkv)]) for b in range(B)])
    v_log = torch.stack([torch.stack([synth.logical_kv(inp, w, b, h)[1] for h in range(Hkv)]) for b in range(B)])
    st.inp["seq_lens"].fill_(n0)
    for b in range(B):
        for t in range(n0, n_final):
            phys = int(inp["block_table"][b, t // w.page_size])
            st.inp["k_pool"][phys, :, t % w.page_size] = 7.0
            st.inp["v_pool"][phys, :, t % w.page_size] = 7.0
    ekv.ekv_stats_build(st.cfg, st.cache(), st.stats())
    for t in range(n0, n_final):
        k_new = k_log[:, :, t].contiguous().to(dev); v_new = v_log[:, :, t].contiguous().to(dev)
        ekv.ekv_stats_append(st.cfg, st.cache(), st.stats(), k_new, v_new)
        st.inp["seq_lens"] += 1
    torch.cuda.synchronize()
    assert torch.equal(st.inp["k_pool"].cpu(), inp["k_pool"]) and torch.equal(st.inp["v_pool"].cpu(), inp["v_pool"])
    box_a, gauss_a = st.box_stats.clone(), st.gauss_stats.clone()
    st.box_stats.zero_(); st.gauss_stats.zero_()
    ekv.ekv_stats_build(st.cfg, st.cache(), st.stats())
    torch.cuda.synchronize()
    M = -(-n_final // w.page_size)
    assert torch.equal(box_a[:, :, :M].view(torch.uint8), st.box_stats[:, :, :M].view(torch.uint8))
    assert torch.equal(gauss_a[:, :, :M].view(torch.uint8), st.gauss_stats[:, :, :M].view(torch.uint8))


# ---------------------------------------------------------------------------- a3 / a4
def upload_oracle_stats(st, w, inp):
    """Oracle statistics, rounded to the storage dtype by the oracle, uploaded to the device."""
    dt = synth.torch_dtype(w.kv_dtype)
    stats = {}
    for b in range(w.batch):
        for h in range(w.n_kv_heads):
            kmin, kmax, kavg, kstd, cnt = oracle_stats(inp, w, b, h)
            kavg, kstd = orc.stored_gauss_stats(kavg, kstd, w.kv_dtype)
            kvar = orc.round_to_storage(kstd ** 2, w.kv_dtype)     # exactly the stored variance again
            M = len(cnt)
            st.box_stats[b, h, :M, 0] = torch.from_numpy(kmin).to(dt).to(st.box.device)
            st.box_stats[b, h, :M, 1] = torch.from_numpy(kmax).to(dt).to(st.box.device)
            st.gauss_stats[b, h, :M, 0] = torch.from_numpy(kavg).to(dt).to(st.box.device)
            st.gauss_stats[b, h, :M, 1] = torch.from_numpy(kvar).to(dt).to(st.box.device)
            stats[(b, h)] = (kmin, kmax, kavg, kstd, cnt)
    return stats


@pytest.mark.parametrize("w", ALL + [synth.C2.scaled(name="C2-short", context=8192, ragged=8192 - 1000)],
                         ids=IDS + ["C2-short"])
def test_score_pages(w):
    inp = get_inputs(w)
    st = DeviceState(w, inp)
    stats = upload_oracle_stats(st, w, inp)
    ekv.ekv_score_pages(st.cfg, st.inp["q"], st.stats(), st.inp["seq_lens"], ekv.EKV_SCORE_BOTH, st.box, st.mu,
                        st.sigma)
    torch.cuda.synchronize()
    box, mu, sigma = st.box.cpu().numpy(), st.mu.cpu().numpy(), st.sigma.cpu().numpy()
    worst = 0.0
    for b in range(w.batch):
        for hq in range(w.n_q_heads):
            kmin, kmax, kavg, kstd, cnt = stats[(b, hq // w.group)]
            M = len(cnt)
            q = to_f64(inp["q"][b, hq])
            ref_box = orc.box_scores(q, kmin, kmax, w.score_scale)
            ref_mu, ref_sig = orc.gauss_moments(q, kavg, kstd, w.score_scale)
            for got, ref in ((box[b, hq, :M], ref_box), (mu[b, hq, :M], ref_mu), (sigma[b, hq, :M], ref_sig)):
                err = np.abs(got - ref) / np.maximum(1.0, np.abs(ref))
                worst = max(worst, err.max())
            assert np.all(np.isneginf(box[b, hq, M:])) and np.all(np.isneginf(mu[b, hq, M:]))
            assert np.all(sigma[b, hq, M:] == 0)
    assert worst <= 1e-5, worst


# ---------------------------------------------------------------------------- a5
@pytest.mark.parametrize("w", ALL, ids=IDS)
def test_select_topk_on_shared_scores(w):
    """Index work on identical float32 scores: the sets must be bit-exact, ties included."""
    inp = get_inputs(w)
    k = topk_budget(w)
    st = DeviceState(w, inp, cap=k)
    rng = np.random.default_rng(3)
    M = -(-int(inp["seq_lens"][0]) // w.page_size)
    scores = rng.normal(size=(w.batch, w.n_q_heads, st.Mmax)).astype(np.float32)
    scores[0, 0, :] = 1.25                                   # all equal: lowest indices win
    scores[0, 1, : M // 2] = np.round(scores[0, 1, : M // 2], 1)   # many ties around the cut
    st.box.copy_(torch.from_numpy(scores))
    ekv.ekv_select_topk(st.cfg, st.box, st.inp["seq_lens"], k, st.page_idx, st.n_sel, st.workspace(ekv.EKV_OP_SELECT_TOPK))
    torch.cuda.synchronize()
    idx, ns = st.page_idx.cpu().numpy(), st.n_sel.cpu().numpy()
    for b in range(w.batch):
        for hq in range(w.n_q_heads):
            ref, _, _ = orc.topk_pages(scores[b, hq, :M].astype(np.float64), k)
            assert ns[b, hq] == len(ref)
            np.testing.assert_array_equal(idx[b, hq, : ns[b, hq]], ref)


@pytest.mark.parametrize("M,k", [(40000 - 3, 1311), (65536, 2622), (20000, 20000), (17000, 1),
                                 (270000, 5400)])       # beyond 64 slices: one workgroup per head reads the keys from memory
def test_select_topk_long_context(M, k):
    """More than 16384 pages: the selection is split over slices of 4096 pages and several launches.
    Synthetic float32 scores (no cache needed); heads with massive ties at the cut: one value (known without ranking),
    thousands of near-equal values inside one histogram bin (ranked inside a sub-bin), two values with thousands of
    pages each inside one bin (a sub-bin filled by one value), thousands of pages on a handful of adjacent float32
    values (the single-workgroup fallback)."""
    P, B, Hq = 16, 1, 11
    Mmax = -(-M // 64) * 64
    cfg = ekv.make_config(B, Hq, Hq, 128, P, "bf16", 1.5, 0.1, Mmax, k)
    dev = torch.device("cuda")
    rng = np.random.default_rng(M + k)
    scores = (rng.normal(size=(B, Hq, Mmax)) * 3.0 + 17.0).astype(np.float32)
    scores[0, 1] = 2.5                                             # all equal -> redo path
    scores[0, 2] = np.round(scores[0, 2], 1)                       # ~100 distinct values, heavy ties
    scores[0, 3, :1024] = 1.0; scores[0, 3, 1024:] += 40.0         # range estimate from the first pages is off
    scores[0, 4] = np.abs(scores[0, 4]) * 1e-3 * rng.choice([-1.0, 1.0], size=Mmax)   # both signs
    scores[0, 5, ::2] = scores[0, 5, 1::2]                         # every value twice
    scores[0, 6] += np.linspace(0.0, 18.0, Mmax, dtype=np.float32)  # trend along the sequence: the top pages crowd the last slices
    scores[0, 7, rng.choice(M, 40, replace=False)] += 60.0         # a few pages far above the sampled range
    n_cl = min(5000, M // 3)
    scores[0, 8, rng.choice(M, n_cl, replace=False)] = (25.0 + 1e-3 * rng.random(n_cl)).astype(np.float32)   # a dense cluster
    two = rng.choice(M, 2 * (n_cl // 2), replace=False)
    scores[0, 9, two[: n_cl // 2]] = 25.0; scores[0, 9, two[n_cl // 2:]] = 25.001              # two crowded values
    scores[0, 10, rng.choice(M, n_cl, replace=False)] = (25.0 + 3e-5 * rng.random(n_cl)).astype(np.float32)  # ~16 adjacent values
    box = torch.from_numpy(scores).to(dev)
    seq_lens = torch.full((B,), M * P - 5, dtype=torch.int32, device=dev)
    page_idx = torch.full((B, Hq, k), -1, dtype=torch.int32, device=dev)
    n_sel = torch.zeros(B, Hq, dtype=torch.int32, device=dev)
    ws = torch.empty(ekv.ekv_workspace_bytes(cfg, ekv.EKV_OP_SELECT_TOPK), dtype=torch.uint8, device=dev)
    for rep in range(2):                                           # second call reuses a dirty workspace
        ekv.ekv_select_topk(cfg, box, seq_lens, k, page_idx, n_sel, ws)
        torch.cuda.synchronize()
        idx, ns = page_idx.cpu().numpy(), n_sel.cpu().numpy()
        for hq in range(Hq):
            ref, _, _ = orc.topk_pages(scores[0, hq, :M].astype(np.float64), k)
            assert ns[0, hq] == len(ref)
            np.testing.assert_array_equal(idx[0, hq, : ns[0, hq]], ref)


@pytest.mark.parametrize("alpha", [1.5, 1.25, 2.0, 4.0 / 3.0], ids=["a1.5", "a1.25", "a2", "a4/3"])
def test_select_gauss_long_context(alpha):
    """Gaussian selector with 65536 pages per head (keys held in registers, 64 per lane), page populations of several
    shapes, every order beta = 1/(alpha-1) of the moments."""
    P, B, Hq, M = 16, 1, 8, 65536
    cap = 3000
    cfg = ekv.make_config(B, Hq, Hq, 128, P, "bf16", alpha, 0.1, M, cap)
    dev = torch.device("cuda")
    rng = np.random.default_rng(99)
    mu = (rng.normal(size=(B, Hq, M)) * 0.25 + 1.0).astype(np.float32)
    sg = (np.abs(rng.normal(size=(B, Hq, M))) * 0.1 + 0.9).astype(np.float32)
    mu[0, 1, rng.choice(M, 50, replace=False)] += 3.0              # a few hot pages
    mu[0, 2, : M // 2] -= 12.0                                      # bimodal: the pooled start is far off
    sg[0, 2, : M // 2] *= 0.05
    mu[0, 3, rng.choice(M, 3, replace=False)] += 9.0; sg[0, 3] *= 0.02   # three pages carry all the mass
    sg[0, 4] = (np.abs(rng.normal(size=M)) * 0.6 + 0.05).astype(np.float32)   # page deviations from 0.05 to ~2
    mu[0, 5] = (1.0 + 0.25 * rng.standard_t(3, size=M)).astype(np.float32)   # heavy-tailed page means
    # two populations interleaved at random (no slice of the sequence sees one alone), and a trend along the sequence
    hi6 = rng.random(M) < 0.5
    mu[0, 6] = np.where(hi6, 4.0 + 0.125 * rng.normal(size=M), 1.0 + 0.25 * rng.normal(size=M)).astype(np.float32)
    mu[0, 7] += np.linspace(0.0, 1.5, M, dtype=np.float32)
    seq_lens = torch.full((B,), M * P - 7, dtype=torch.int32, device=dev)
    t = lambda a: torch.from_numpy(a).to(dev)
    tau_hat = torch.zeros(B, Hq, device=dev); page_idx = torch.zeros(B, Hq, cap, dtype=torch.int32, device=dev)
    n_sel = torch.zeros(B, Hq, dtype=torch.int32, device=dev); ovf = torch.zeros_like(n_sel)
    ws = torch.empty(ekv.ekv_workspace_bytes(cfg, ekv.EKV_OP_SELECT_GAUSS), dtype=torch.uint8, device=dev)
    cnt = np.full(M, P); cnt[-1] = P - 7
    for q_page, margin in ((0.99, 0.0), (0.999, 0.02)):
        ekv.ekv_select_gauss(cfg, t(mu), t(sg), seq_lens, q_page, margin, tau_hat, page_idx, n_sel, ovf, ws)
        torch.cuda.synchronize()
        for hq in range(Hq):
            pages, th, o, g = orc.gauss_select(mu[0, hq].astype(np.float64), sg[0, hq].astype(np.float64), cnt, alpha,
                                               q_page, margin, cap=cap)
            assert abs(float(tau_hat[0, hq]) - th) <= 4e-6 * max(1.0, abs(th)), (float(tau_hat[0, hq]), th)
            assert int(ovf[0, hq]) == int(o)
            got = page_idx[0, hq, : int(n_sel[0, hq])].cpu().numpy()
            if not o:
                cut = th - margin
                ok, bad = sets_equal_up_to_cut(got, pages, g, cut, 1e-5 * max(1.0, abs(cut)))
                assert ok, (hq, bad[:5], len(pages), len(got))
            else:                                              # the cap best estimates, up to ties at the cut
                assert len(got) == cap
                cut = float(np.min(g[pages]))
                ok, bad = sets_equal_up_to_cut(got, pages, g, cut, 1e-5 * max(1.0, abs(cut)))
                assert ok, (hq, bad[:5])
            assert np.all(np.diff(got) > 0)


# ---------------------------------------------------------------------------- a6
WP64 = synth.C2.scaled(name="C2-p64-g8", context=4096 + 64, ragged=21, page_size=64, n_q_heads=16, n_kv_heads=2)
WP8 = synth.C2.scaled(name="C2-p8-g2", context=2048 + 8, ragged=3, page_size=8, n_q_heads=4, n_kv_heads=2)


@pytest.mark.parametrize("w", [W1S, W2, W3, W3A, W5, W5B, WP64, WP8],
                         ids=["C1-soft", "C2-8k", "C3-small", "C3-small-a43", "C5-small", "C5-small-a2", "C2-p64-g8",
                              "C2-p8-g2"])
@pytest.mark.parametrize("q_page,margin", [(0.99, 0.0), (0.9, 0.05)])
def test_select_gauss_on_shared_moments(w, q_page, margin):
    inp = get_inputs(w)
    st = DeviceState(w, inp)
    stats = upload_oracle_stats(st, w, inp)
    mus, sigs = {}, {}
    for b in range(w.batch):
        for hq in range(w.n_q_heads):
            kmin, kmax, kavg, kstd, cnt = stats[(b, hq // w.group)]
            m, s = orc.gauss_moments(to_f64(inp["q"][b, hq]), kavg, kstd, w.score_scale)
            m32, s32 = m.astype(np.float32), s.astype(np.float32)
            M = len(cnt)
            st.mu[b, hq, :M] = torch.from_numpy(m32).to(st.mu.device)
            st.sigma[b, hq, :M] = torch.from_numpy(s32).to(st.mu.device)
            mus[(b, hq)], sigs[(b, hq)] = m32.astype(np.float64), s32.astype(np.float64)
    ws = st.workspace(ekv.EKV_OP_SELECT_GAUSS)
    ekv.ekv_select_gauss(st.cfg, st.mu, st.sigma, st.inp["seq_lens"], q_page, margin, st.tau_hat, st.page_idx,
                         st.n_sel, st.overflow, ws)
    torch.cuda.synchronize()
    idx, ns, th = st.page_idx.cpu().numpy(), st.n_sel.cpu().numpy(), st.tau_hat.cpu().numpy()
    assert not st.overflow.cpu().numpy().any()
    for (b, hq) in sample_units(w, 8):
        cnt = stats[(b, hq // w.group)][4]
        pages, tau_hat, ovf, g = orc.gauss_select(mus[(b, hq)], sigs[(b, hq)], cnt, w.alpha, q_page, margin)
        assert abs(th[b, hq] - tau_hat) <= 4e-6 * max(1.0, abs(tau_hat)), (th[b, hq], tau_hat)
        cut = tau_hat - margin
        ok, bad = sets_equal_up_to_cut(idx[b, hq, : ns[b, hq]], pages, g, cut, 1e-5 * max(1.0, abs(cut)))
        assert ok, (b, hq, bad[:5], len(pages), ns[b, hq])
        assert np.all(np.diff(idx[b, hq, : ns[b, hq]]) > 0)


def test_select_gauss_empty_and_overflow():
    w = W3
    inp = get_inputs(w)
    cap = 5
    st = DeviceState(w, inp, cap=cap)
    rng = np.random.default_rng(1)
    M = w.pages_per_seq
    mu = rng.normal(size=(w.batch, w.n_q_heads, M)).astype(np.float32)
    sg = (np.abs(rng.normal(size=mu.shape)) * 0.3 + 0.05).astype(np.float32)
    st.mu.copy_(torch.from_numpy(mu)); st.sigma.copy_(torch.from_numpy(sg))
    ws = st.workspace(ekv.EKV_OP_SELECT_GAUSS)
    cnt = np.full(M, w.page_size)
    # tiny q_page pushes every page estimate far below tau_hat: empty -> best single page
    ekv.ekv_select_gauss(st.cfg, st.mu, st.sigma, st.inp["seq_lens"], 1e-6, 0.0, st.tau_hat, st.page_idx, st.n_sel,
                         st.overflow, ws)
    torch.cuda.synchronize()
    for (b, hq) in sample_units(w, 4):
        pages, _, ovf, g = orc.gauss_select(mu[b, hq].astype(np.float64), sg[b, hq].astype(np.float64), cnt, w.alpha,
                                            1e-6, 0.0, cap=cap)
        assert int(st.n_sel[b, hq]) == len(pages) == 1 and int(st.page_idx[b, hq, 0]) == pages[0]
        assert int(st.overflow[b, hq]) == 0
    # a huge margin selects everything: overflow -> the cap best pages
    ekv.ekv_select_gauss(st.cfg, st.mu, st.sigma, st.inp["seq_lens"], 0.9, 50.0, st.tau_hat, st.page_idx, st.n_sel,
                         st.overflow, ws)
    torch.cuda.synchronize()
    for (b, hq) in sample_units(w, 4):
        pages, _, ovf, g = orc.gauss_select(mu[b, hq].astype(np.float64), sg[b, hq].astype(np.float64), cnt, w.alpha,
                                            0.9, 50.0, cap=cap)
        assert ovf and int(st.overflow[b, hq]) == 1 and int(st.n_sel[b, hq]) == cap
        np.testing.assert_array_equal(st.page_idx[b, hq].cpu().numpy(), pages)


# ---------------------------------------------------------------------------- a7 / a8 / metrics
@pytest.mark.parametrize("w", ALL, ids=IDS)
def test_decode_sparse_and_full_on_shared_page_lists(w):
    inp = get_inputs(w)
    k = topk_budget(w)
    st = DeviceState(w, inp, cap=k)
    dev = st.box.device
    units = sample_units(w, 6)
    refs = {}
    for (b, hq) in [(b, h) for b in range(w.batch) for h in range(w.n_q_heads)]:
        # page list: oracle top-k on the oracle's box scores
        kmin, kmax, *_ = oracle_stats(inp, w, b, hq // w.group)
        boxs = orc.box_scores(to_f64(inp["q"][b, hq]), kmin, kmax, w.score_scale)
        pages, _, _ = orc.topk_pages(boxs, k)
        st.page_idx[b, hq, : len(pages)] = torch.from_numpy(pages.astype(np.int32)).to(dev)
        st.n_sel[b, hq] = len(pages)
        refs[(b, hq)] = pages
    supp_tok = torch.full((w.batch, w.n_q_heads, 4096), -1, device=dev, dtype=torch.int32)
    tau_ref = torch.zeros(w.batch, w.n_q_heads, device=dev)
    kept_mass = torch.zeros_like(tau_ref); kept_supp = torch.zeros_like(st.supp)
    # dense first (gives tau_full for the dropped-mass side outputs)
    wsf = st.workspace(ekv.EKV_OP_DECODE_FULL)
    out_f, tau_f, supp_f = torch.zeros_like(st.out), torch.zeros_like(st.tau), torch.zeros_like(st.supp)
    lse = torch.zeros_like(tau_ref)
    ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), out_f, tau_f, supp_f, wsf,
                        extras=ekv.decode_extras(support_tokens=supp_tok, lse=lse))
    torch.cuda.synchronize()
    full_tokens = supp_tok.cpu().numpy().copy()
    full = {}
    for (b, hq) in units:
        q, K, V = unit_kv(inp, w, b, hq)
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        full[(b, hq)] = ref
        check_decode_unit(w, out_f[b, hq].cpu().numpy(), float(tau_f[b, hq]), int(supp_f[b, hq]),
                          full_tokens[b, hq], ref)
        sm = orc.softmax_attention(q, K, V, w.score_scale)
        assert abs(float(lse[b, hq]) - sm["lse"]) <= 2e-5 * max(1.0, abs(sm["lse"]))
        tau_ref[b, hq] = ref["tau"]                   # oracle value -> GPU input (never the reverse)
    # sparse
    supp_tok.fill_(-1)
    wss = st.workspace(ekv.EKV_OP_DECODE_SPARSE)
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp, wss,
                          extras=ekv.decode_extras(support_tokens=supp_tok, tau_ref=tau_ref, kept_mass_ref=kept_mass,
                                                   kept_supp_ref=kept_supp))
    torch.cuda.synchronize()
    sp_tokens = supp_tok.cpu().numpy()
    for (b, hq) in units:
        q, K, V = unit_kv(inp, w, b, hq)
        tok = orc.pages_to_tokens(refs[(b, hq)], w.page_size, K.shape[0])
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale, tok)
        check_decode_unit(w, st.out[b, hq].cpu().numpy(), float(st.tau[b, hq]), int(st.supp[b, hq]),
                          sp_tokens[b, hq], ref)
        delta = orc.dropped_mass(full[(b, hq)]["p"], tok)
        assert abs((1.0 - float(kept_mass[b, hq])) - delta) <= 1e-4
        assert int(kept_supp[b, hq]) == int(np.isin(full[(b, hq)]["support"], tok).sum())


def test_sparse_equals_full_when_support_is_covered():
    """Prop. 2 on the GPU: candidates that contain the support reproduce the dense result."""
    w = W1S
    inp = get_inputs(w)
    st = DeviceState(w, inp)
    dev = st.box.device
    wsf = st.workspace(ekv.EKV_OP_DECODE_FULL)
    out_f, tau_f, supp_f = torch.zeros_like(st.out), torch.zeros_like(st.tau), torch.zeros_like(st.supp)
    ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), out_f, tau_f, supp_f, wsf)
    rng = np.random.default_rng(0)
    for hq in range(w.n_q_heads):
        q, K, V = unit_kv(inp, w, 0, hq)
        S = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)["support"]      # oracle support
        pages = np.union1d(np.unique(S // w.page_size), rng.choice(w.pages_per_seq, 7, replace=False))
        st.page_idx[0, hq, : len(pages)] = torch.from_numpy(pages.astype(np.int32)).to(dev)
        st.n_sel[0, hq] = len(pages)
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                          st.workspace(ekv.EKV_OP_DECODE_SPARSE))
    torch.cuda.synchronize()
    assert torch.equal(st.supp, supp_f)
    assert float((st.tau - tau_f).abs().max()) <= 1e-6
    assert rel_err(st.out.cpu().numpy().ravel(), out_f.cpu().numpy().ravel().astype(np.float64)) <= 2e-6


def seeded(base, kind, rng):
    """Seeds for the warm start, from the oracle's tau (float64 array [B, Hq])."""
    if kind == "exact": return base
    if kind == "slightly-low": return base - 1e-3
    if kind == "slightly-high": return base + 1e-3
    if kind == "far-low": return base - 0.7
    if kind == "far-high": return base + 0.7
    if kind == "garbage":
        vals = np.array([np.nan, np.inf, -np.inf, 1e30, -1e30, 0.0])
        return vals[rng.integers(0, len(vals), size=base.shape)]
    raise ValueError(kind)


@pytest.mark.parametrize("w", [W1S, W2, W3A, W5, W5B], ids=["C1-soft", "C2-8k", "C3-small-a43", "C5-small", "C5-small-a2"])
def test_warm_started_solve_gives_the_same_result(w):
    """tau_seed only moves the starting point: whatever the seed (the exact tau, near it on either side,
    far off, NaN/inf), threshold, support and output are those of the unseeded solve and of the oracle; a
    good seed takes fewer evaluations of the mass.  Sparse decode on top-k lists and dense decode."""
    inp = get_inputs(w)
    k = topk_budget(w)
    st = DeviceState(w, inp, cap=k)
    dev = st.box.device
    run_step(st, w, "topk", k=k)
    torch.cuda.synchronize()
    idx, ns = st.page_idx.cpu().numpy(), st.n_sel.cpu().numpy()
    B, Hq = w.batch, w.n_q_heads
    units = [(b, h) for b in range(B) for h in range(Hq)]
    ref_s = np.zeros((B, Hq)); ref_d = np.zeros((B, Hq))
    refs = {}
    for (b, hq) in units:
        q, K, V = unit_kv(inp, w, b, hq)
        tok = orc.pages_to_tokens(idx[b, hq, : ns[b, hq]], w.page_size, K.shape[0])
        rs = orc.entmax_attention(q, K, V, w.alpha, w.score_scale, tok)
        rd = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        ref_s[b, hq], ref_d[b, hq] = rs["tau"], rd["tau"]
        refs[(b, hq)] = (rs, rd)
    evals = torch.zeros(B, Hq, dtype=torch.int32, device=dev)
    ws_s, ws_d = st.workspace(ekv.EKV_OP_DECODE_SPARSE), st.workspace(ekv.EKV_OP_DECODE_FULL)
    rng = np.random.default_rng(3)

    def run(dense, seed):
        t = None if seed is None else torch.from_numpy(seed.astype(np.float32)).to(dev)
        ex = ekv.decode_extras(tau_seed=t, solve_evals=evals)
        if dense:
            ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), st.out, st.tau, st.supp, ws_d, extras=ex)
        else:
            ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                                  ws_s, extras=ex)
        torch.cuda.synchronize()
        return st.tau.cpu().numpy().copy(), st.supp.cpu().numpy().copy(), st.out.cpu().numpy().copy(), \
            evals.cpu().numpy().copy()

    for dense, base in ((False, ref_s), (True, ref_d)):
        tau0, supp0, out0, ev0 = run(dense, None)
        assert ev0.min() >= 1
        for kind in ("exact", "slightly-low", "slightly-high", "far-low", "far-high", "garbage"):
            tau1, supp1, out1, ev1 = run(dense, seeded(base, kind, rng))
            assert np.all(np.abs(tau1 - base) <= 4e-6 * np.maximum(1.0, np.abs(base))), kind
            for (b, hq) in units:
                ref = refs[(b, hq)][1 if dense else 0]
                z = (w.alpha - 1.0) * ref["s"]
                n_boundary = int(np.sum(np.abs(z - ref["tau"]) <= 2e-6 * max(1.0, abs(ref["tau"]))))
                assert abs(int(supp1[b, hq]) - len(ref["support"])) <= n_boundary, (kind, b, hq)
                if n_boundary == 0:
                    assert supp1[b, hq] == supp0[b, hq]
                assert rel_err(out1[b, hq], ref["o"]) <= OUT_TOL[w.kv_dtype], (kind, b, hq)
            if kind == "exact":
                assert ev1.mean() <= ev0.mean() and ev1.max() <= 3, (ev0.mean(), ev1.mean(), ev1.max())


# ---------------------------------------------------------------------------- a9
@pytest.mark.parametrize("w", [W1S, W5, synth.C2.scaled(name="C2-p64-g8", context=4096 + 64, ragged=21, page_size=64,
                                                        n_q_heads=16, n_kv_heads=2),
                               synth.C2.scaled(name="C2-p8-g2", context=2048 + 8, ragged=3, page_size=8, n_q_heads=4,
                                               n_kv_heads=2)],
                         ids=["C1-soft", "C5-small", "C2-p64-g8", "C2-p8-g2"])
def test_decode_sparse_softmax(w):
    inp = get_inputs(w)
    k = topk_budget(w)
    st = DeviceState(w, inp, cap=k)
    dev = st.box.device
    rng = np.random.default_rng(2)
    lists = {}
    for b in range(w.batch):
        for hq in range(w.n_q_heads):
            pages = np.sort(rng.choice(-(-int(inp["seq_lens"][b]) // w.page_size), k, replace=False))
            pages[-1] = -(-int(inp["seq_lens"][b]) // w.page_size) - 1          # include the (partial) last page
            pages = np.unique(pages)
            st.page_idx[b, hq, : len(pages)] = torch.from_numpy(pages.astype(np.int32)).to(dev)
            st.n_sel[b, hq] = len(pages)
            lists[(b, hq)] = pages
    lse = torch.zeros_like(st.tau)
    ekv.ekv_decode_sparse_softmax(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, lse,
                                  st.workspace(ekv.EKV_OP_DECODE_SPARSE_SOFTMAX))
    torch.cuda.synchronize()
    for (b, hq) in sample_units(w, 6):
        q, K, V = unit_kv(inp, w, b, hq)
        tok = orc.pages_to_tokens(lists[(b, hq)], w.page_size, K.shape[0])
        ref = orc.softmax_attention(q, K, V, w.score_scale, tok)
        assert rel_err(st.out[b, hq].cpu().numpy(), ref["o"]) <= max(OUT_TOL[w.kv_dtype], 2e-5)
        assert abs(float(lse[b, hq]) - ref["lse"]) <= 2e-5 * max(1.0, abs(ref["lse"]))
        # kept softmax mass against the full-cache normaliser (Eq. 8's delta^sm)
        full = orc.softmax_attention(q, K, V, w.score_scale)
        d_sm = orc.dropped_mass(full["p"], tok)
        assert abs((1.0 - math.exp(float(lse[b, hq]) - full["lse"])) - d_sm) <= 1e-4


# ---------------------------------------------------------------------------- whole step
def run_step(st, w, selector, k=None, q_page=0.99, margin=0.0):
    ekv.ekv_stats_build(st.cfg, st.cache(), st.stats())
    if selector == "topk":
        ekv.ekv_score_pages(st.cfg, st.inp["q"], st.stats(), st.inp["seq_lens"], ekv.EKV_SCORE_BOX, st.box)
        ekv.ekv_select_topk(st.cfg, st.box, st.inp["seq_lens"], k, st.page_idx, st.n_sel, st.workspace(ekv.EKV_OP_SELECT_TOPK))
    else:
        ekv.ekv_score_pages(st.cfg, st.inp["q"], st.stats(), st.inp["seq_lens"], ekv.EKV_SCORE_GAUSS, None, st.mu,
                            st.sigma)
        ekv.ekv_select_gauss(st.cfg, st.mu, st.sigma, st.inp["seq_lens"], q_page, margin, st.tau_hat, st.page_idx,
                             st.n_sel, st.overflow, st.workspace(ekv.EKV_OP_SELECT_GAUSS))
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                          st.workspace(ekv.EKV_OP_DECODE_SPARSE))
    torch.cuda.synchronize()


@pytest.mark.parametrize("w", ALL, ids=IDS)
def test_end_to_end_topk_step(w):
    inp = get_inputs(w)
    k = topk_budget(w)
    st = DeviceState(w, inp, cap=k)
    run_step(st, w, "topk", k=k)
    idx, ns = st.page_idx.cpu().numpy(), st.n_sel.cpu().numpy()
    for (b, hq) in sample_units(w, 6):
        q, K, V = unit_kv(inp, w, b, hq)
        ref = orc.decode_step_unit(q, K, V, w.page_size, w.alpha, w.score_scale, "topk", w.kv_dtype, k_pages=k)
        cuts = [ref["cut_in"], ref["cut_out"]]
        band = 1e-5 * max(1.0, abs(ref["cut_in"]))
        ok, bad = sets_equal_up_to_cut(idx[b, hq, : ns[b, hq]], ref["pages"], ref["box"], cuts, band)
        assert ok, (b, hq, bad)
        # the decode is checked for the list the GPU chose, whether or not it equals the oracle's (tie band)
        check_decode_of_gpu_list(w, q, K, V, idx[b, hq, : ns[b, hq]], st.out[b, hq].cpu().numpy(), st.tau[b, hq],
                                 st.supp[b, hq])


@pytest.mark.parametrize("w", [W1S, W2, W5B], ids=["C1-soft", "C2-8k", "C5-small-a2"])
def test_end_to_end_gauss_step_is_deterministic_and_consistent(w):
    """Whole Gaussian-selector step on GPU-built statistics.  bf16 storage of k_avg/k_std may differ
    from the oracle's rounding by one ulp in rare elements, which moves individual page estimates by
    far more than the 1e-5 rule; page-set parity of this selector is therefore asserted on shared
    moments (test_select_gauss_on_shared_moments) and this test checks what is unique: the decode
    result for the page list the GPU itself chose, and bitwise reproducibility."""
    inp = get_inputs(w)
    st = DeviceState(w, inp)
    run_step(st, w, "gauss", q_page=0.99)
    first = (st.out.clone(), st.tau.clone(), st.page_idx.clone(), st.n_sel.clone(), st.tau_hat.clone())
    idx, ns = st.page_idx.cpu().numpy(), st.n_sel.cpu().numpy()
    for (b, hq) in sample_units(w, 4):
        q, K, V = unit_kv(inp, w, b, hq)
        tok = orc.pages_to_tokens(idx[b, hq, : ns[b, hq]], w.page_size, K.shape[0])
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale, tok)
        assert abs(float(st.tau[b, hq]) - ref["tau"]) <= 4e-6 * max(1.0, abs(ref["tau"]))
        assert rel_err(st.out[b, hq].cpu().numpy(), ref["o"]) <= OUT_TOL[w.kv_dtype]
        full = orc.decode_step_unit(q, K, V, w.page_size, w.alpha, w.score_scale, "gauss", w.kv_dtype, q_page=0.99)
        assert abs(float(st.tau_hat[b, hq]) - full["tau_hat"]) <= 2e-3 * max(1.0, abs(full["tau_hat"]))
    run_step(st, w, "gauss", q_page=0.99)
    for a, bb in zip(first, (st.out, st.tau, st.page_idx, st.n_sel, st.tau_hat)):
        assert torch.equal(a.view(torch.uint8), bb.view(torch.uint8))


# ---------------------------------------------------------------------------- edge cases
def test_tiny_sequences_and_all_pages_selected():
    for n in (1, 3, 16, 17):
        w = synth.C1.scaled(name="C1-edge", context=n, n_planted=0, scale=0.1)
        inp = synth.make_inputs(w, 77 + n, device="cpu")
        st = DeviceState(w, inp, cap=w.pages_per_seq)
        run_step(st, w, "topk", k=w.pages_per_seq)           # k >= M: every page
        for hq in (0, 5):
            q, K, V = unit_kv(inp, w, 0, hq)
            ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
            assert int(st.n_sel[0, hq]) == w.pages_per_seq
            assert int(st.supp[0, hq]) == len(ref["support"])
            assert rel_err(st.out[0, hq].cpu().numpy(), ref["o"]) <= 1e-5
        # the Gaussian-aware selector on the same few pages (one page per wavefront of its single slice)
        run_step(st, w, "gauss", q_page=0.99, margin=0.0)
        for hq in (0, 5):
            q, K, V = unit_kv(inp, w, 0, hq)
            ref = orc.decode_step_unit(q, K, V, w.page_size, w.alpha, w.score_scale, "gauss", w.kv_dtype, q_page=0.99,
                                       margin=0.0, cap=w.pages_per_seq)
            assert abs(float(st.tau_hat[0, hq]) - ref["tau_hat"]) <= 4e-6 * max(1.0, abs(ref["tau_hat"]))
            got = st.page_idx[0, hq, : int(st.n_sel[0, hq])].cpu().numpy()
            band = 1e-5 * max(1.0, abs(ref["tau_hat"]))
            ok, bad = sets_equal_up_to_cut(got, ref["pages"], ref["g"], ref["tau_hat"], band)
            assert ok, (n, hq, bad)


def test_candidate_list_larger_than_lds_uses_the_streaming_path():
    """Nearly flat scores: every token is within 1 of the maximum, so 8192 candidates exceed the LDS
    list (4096) and the solver must stream the score row instead."""
    w = synth.C1.scaled(name="C1-flat", context=8192, n_planted=0, scale=0.02 / math.sqrt(128.0), n_q_heads=2,
                        n_kv_heads=2)
    inp = synth.make_inputs(w, 4242, device="cpu")
    st = DeviceState(w, inp)
    out_f, tau_f, supp_f = torch.zeros_like(st.out), torch.zeros_like(st.tau), torch.zeros_like(st.supp)
    ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), out_f, tau_f, supp_f, st.workspace(ekv.EKV_OP_DECODE_FULL))
    torch.cuda.synchronize()
    for hq in range(2):
        q, K, V = unit_kv(inp, w, 0, hq)
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        z = (w.alpha - 1.0) * ref["s"]
        assert np.sum(z > z.max() - 1.0) > 4096 and len(ref["support"]) > 4096
        # same rule as everywhere: tau 4e-6, output 1e-5, support exact up to tokens within float32 resolution of tau
        check_decode_unit(w, out_f[0, hq].cpu().numpy(), float(tau_f[0, hq]), int(supp_f[0, hq]), None, ref,
                          boundary_expected=True)


LONG = [synth.C2.scaled(name="C2-long-bf16", context=100000, ragged=7, n_q_heads=4, n_kv_heads=2),
        synth.C1.scaled(name="C1-long-f32", context=70000, ragged=3, n_q_heads=2, n_kv_heads=2,
                        scale=1.0 / math.sqrt(128.0)),
        synth.C5.scaled(name="C5-long-p32-a2", batch=2, context=98304 + 64, ragged=33, n_q_heads=2, n_kv_heads=1,
                        alpha=2.0),
        # nearly flat scores: more than 4096 tokens above the certified bound -> the solve cannot take the
        # filtered lists and falls back to streaming the row from that bound
        synth.C1.scaled(name="C1-long-flat", context=66000, n_planted=0, scale=0.02 / math.sqrt(128.0),
                        n_q_heads=2, n_kv_heads=2),
        # rows of more than 16384 groups: these take the multi-workgroup filter passes (the rows above are solved from
        # the group maxima by one workgroup); one page of 36, 40 or 48 tokens is a group
        synth.C2.scaled(name="C2-filter-bf16", context=790000, ragged=11, n_q_heads=2, n_kv_heads=1, page_size=48),
        synth.C1.scaled(name="C1-filter-f32", context=592000, ragged=3, n_q_heads=2, n_kv_heads=1, page_size=36,
                        scale=1.0 / math.sqrt(128.0)),
        synth.C1.scaled(name="C1-filter-flat", context=592000, n_planted=0, scale=0.02 / math.sqrt(128.0),
                        n_q_heads=2, n_kv_heads=1, page_size=36),
        # moderately flat rows, supports of hundreds to thousands of tokens: the candidates stay in the segments of the
        # solve or continue in the row's one list, and the row of 660 000 tokens reaches that list through the filter
        # passes' per-slice lists.
        synth.C1.scaled(name="C1-wide-900", context=100000, ragged=5, n_planted=0, scale=0.15 / math.sqrt(128.0),
                        n_q_heads=2, n_kv_heads=2),
        synth.C1.scaled(name="C1-wide-5000", context=100000, ragged=5, n_planted=0, scale=0.05 / math.sqrt(128.0),
                        n_q_heads=2, n_kv_heads=2),
        synth.C1.scaled(name="C1-filter-wide-6000", context=660000, ragged=9, n_planted=0, scale=0.05 / math.sqrt(128.0),
                        n_q_heads=2, n_kv_heads=1, page_size=40),
        # the same through the matrix-core score pass: bf16 cache, pages of 32, two query heads per KV head, beta = 4
        synth.C5.scaled(name="C5-wide-a125-6000", batch=1, context=100000, ragged=5, n_planted=0,
                        scale=0.5 / math.sqrt(128.0), n_q_heads=2, n_kv_heads=1, alpha=1.25)]


@pytest.mark.parametrize("w", LONG, ids=[w.name for w in LONG])
def test_decode_long_rows_take_the_filter_passes(w):
    """Long rows: up to 16384 groups one workgroup solves them from the group maxima, several per thread; longer ones
    are pre-filtered by the multi-workgroup passes (dense, and sparse with a large selection).  Results must meet the
    same bars as the short-row path."""
    inp = get_inputs(w)
    M = w.pages_per_seq
    n = w.context - w.ragged
    n_pages = -(-n // w.page_size)
    filtered = "filter" in w.name
    cap = pre_groups() + 1 if filtered else min(M, -(-66000 // w.page_size))     # pages of a selection
    assert not filtered or (w.page_size > 32 and cap < M)                        # a page is a group of its own
    st = DeviceState(w, inp, cap=cap)
    dev = st.box.device
    supp_tok = torch.full((w.batch, w.n_q_heads, 8192), -1, device=dev, dtype=torch.int32)
    out_f, tau_f, supp_f = torch.zeros_like(st.out), torch.zeros_like(st.tau), torch.zeros_like(st.supp)
    ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), out_f, tau_f, supp_f, st.workspace(ekv.EKV_OP_DECODE_FULL),
                        extras=ekv.decode_extras(support_tokens=supp_tok))
    torch.cuda.synchronize()
    full_tokens = supp_tok.cpu().numpy().copy()
    # sparse: a seeded random page list of `cap` pages that always holds the last (partial) page
    rng = np.random.default_rng(77)
    lists = {}
    for b in range(w.batch):
        for hq in range(w.n_q_heads):
            pages = np.sort(rng.choice(n_pages - 1, cap - 1, replace=False))
            pages = np.append(pages, n_pages - 1)
            lists[(b, hq)] = pages
            st.page_idx[b, hq, :cap] = torch.from_numpy(pages.astype(np.int32)).to(dev)
            st.n_sel[b, hq] = cap
    supp_tok.fill_(-1)
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                          st.workspace(ekv.EKV_OP_DECODE_SPARSE), extras=ekv.decode_extras(support_tokens=supp_tok))
    torch.cuda.synchronize()
    sp_tokens = supp_tok.cpu().numpy()
    flat = "flat" in w.name
    for (b, hq) in [(0, 0), (w.batch - 1, w.n_q_heads - 1)]:
        q, K, V = unit_kv(inp, w, b, hq)
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        tok = orc.pages_to_tokens(lists[(b, hq)], w.page_size, K.shape[0])
        ref_s = orc.entmax_attention(q, K, V, w.alpha, w.score_scale, tok)
        if "wide" in w.name:
            lo, hi = {"900": (500, 2000), "5000": (4096, 8192), "6000": (4096, 8192)}[w.name.rsplit("-", 1)[1]]
            assert lo < len(ref["support"]) < hi and (hi < 4096 or len(ref_s["support"]) > 2500)
            check_decode_unit(w, out_f[b, hq].cpu().numpy(), float(tau_f[b, hq]), int(supp_f[b, hq]),
                              full_tokens[b, hq], ref, boundary_expected=True)
            check_decode_unit(w, st.out[b, hq].cpu().numpy(), float(st.tau[b, hq]), int(st.supp[b, hq]),
                              sp_tokens[b, hq], ref_s, boundary_expected=True)
        elif flat:
            assert len(ref["support"]) > 4096 and len(ref_s["support"]) > 4096
            # supports larger than the token list the test asked for: counts, tau and outputs under the usual rule
            for got_tau, got_supp, got_out, r in ((tau_f, supp_f, out_f, ref), (st.tau, st.supp, st.out, ref_s)):
                check_decode_unit(w, got_out[b, hq].cpu().numpy(), float(got_tau[b, hq]), int(got_supp[b, hq]), None, r,
                                  boundary_expected=True)
        else:
            check_decode_unit(w, out_f[b, hq].cpu().numpy(), float(tau_f[b, hq]), int(supp_f[b, hq]),
                              full_tokens[b, hq], ref)
            check_decode_unit(w, st.out[b, hq].cpu().numpy(), float(st.tau[b, hq]), int(st.supp[b, hq]),
                              sp_tokens[b, hq], ref_s)


# ---------------------------------------------------------------------------- box-threshold refinement
@pytest.mark.parametrize("M,cap,alpha", [(300, 300, 1.5), (40000 - 3, 9000, 1.5), (8192, 700, 2.0),
                                         (5000, 5000, 1.25)])
def test_select_box_threshold_on_shared_scores(M, cap, alpha):
    """Union of a given list with the pages above the threshold, on identical float32 scores: sets,
    counts and flags must match the oracle (pages within 1e-5 of the threshold may differ)."""
    P = 16
    w = synth.C1.scaled(name=f"C1-boxthr-{M}-{alpha}", context=M * P, ragged=5, n_q_heads=6, n_kv_heads=6, alpha=alpha)
    inp = get_inputs(w)
    st = DeviceState(w, inp, cap=cap)
    dev = st.box.device
    rng = np.random.default_rng(11)
    scores = rng.normal(size=(1, 6, M)).astype(np.float32)
    a = alpha - 1.0
    tau_lo = np.array([[np.quantile(a * scores[0, 0], 0.98), np.quantile(a * scores[0, 1], 0.5), np.inf, -np.inf,
                        np.quantile(a * scores[0, 4], 0.999), float(a * scores[0, 5].max())]], dtype=np.float32)
    lists = []
    for h in range(6):
        n_in = [0, 17, 40, 3, min(cap, 257), 1][h]
        lst = rng.choice(M, n_in, replace=False).astype(np.int32)
        if h == 1:
            lst = np.concatenate([lst, lst[:5], np.array([M + 3, -1], dtype=np.int32)])   # duplicates, out of range
        lists.append(lst)
        st.page_idx[0, h, : len(lst)] = torch.from_numpy(lst).to(dev)
        st.n_sel[0, h] = len(lst)
    st.box.copy_(torch.from_numpy(scores))
    tau_d = torch.from_numpy(tau_lo).to(dev)
    out_idx = torch.full_like(st.page_idx, -7)
    out_n, added, ovf = torch.zeros_like(st.n_sel), torch.zeros_like(st.n_sel), torch.zeros_like(st.n_sel)
    ekv.ekv_select_box_threshold(st.cfg, st.box, st.inp["seq_lens"], tau_d, st.page_idx, st.n_sel, out_idx, out_n,
                                 added, ovf, st.workspace(ekv.EKV_OP_SELECT_BOX_THRESHOLD))
    torch.cuda.synchronize()
    oi, on, ad, ov = out_idx.cpu().numpy(), out_n.cpu().numpy(), added.cpu().numpy(), ovf.cpu().numpy()
    for h in range(6):
        given = np.array(sorted(set(int(p) for p in lists[h] if 0 <= p < M)), dtype=np.int64)
        union, new = orc.refine_selection(scores[0, h].astype(np.float64), alpha, float(tau_lo[0, h]), given)
        band = 1e-5 * max(1.0, abs(float(tau_lo[0, h]))) if np.isfinite(tau_lo[0, h]) else 0.0
        near = int(np.sum(np.abs(a * scores[0, h].astype(np.float64) - float(tau_lo[0, h])) <= band)) if band else 0
        assert abs(int(ad[0, h]) - len(new)) <= near
        if len(union) > cap + near:
            assert ov[0, h] == 1 and on[0, h] == cap
            if near == 0:
                np.testing.assert_array_equal(oi[0, h, :cap], union[:cap])
        elif len(union) <= cap - near:
            assert ov[0, h] == 0
            got = oi[0, h, : on[0, h]]
            assert np.all(np.diff(got) > 0)
            ok, bad = sets_equal_up_to_cut(got, union, a * scores[0, h].astype(np.float64), float(tau_lo[0, h]), band)
            assert ok, bad
    # no input list at all: pure threshold selection
    ekv.ekv_select_box_threshold(st.cfg, st.box, st.inp["seq_lens"], tau_d, None, None, out_idx, out_n, added, ovf,
                                 st.workspace(ekv.EKV_OP_SELECT_BOX_THRESHOLD))
    torch.cuda.synchronize()
    oi, on, ad = out_idx.cpu().numpy(), out_n.cpu().numpy(), added.cpu().numpy()
    for h in (0, 2, 4, 5):
        ref = orc.box_threshold_pages(scores[0, h].astype(np.float64), alpha, float(tau_lo[0, h]))
        if len(ref) <= cap:
            np.testing.assert_array_equal(oi[0, h, : on[0, h]], ref)
            assert ad[0, h] == len(ref)


@pytest.mark.parametrize("w", [W1S, W2, W5B], ids=["C1-soft", "C2-8k", "C5-small-a2"])
def test_one_refinement_after_topk_reaches_the_full_cache_result(w):
    """top-k with a small budget -> sparse decode -> box-threshold refinement with the sparse tau -> sparse
    decode again: the second result is the full-cache result (oracle), and refining once more adds nothing."""
    inp = get_inputs(w)
    st = DeviceState(w, inp)                                   # cap = every page
    k = max(2, w.pages_per_seq // 64)
    ekv.ekv_stats_build(st.cfg, st.cache(), st.stats())
    ekv.ekv_score_pages(st.cfg, st.inp["q"], st.stats(), st.inp["seq_lens"], ekv.EKV_SCORE_BOX, st.box)
    ekv.ekv_select_topk(st.cfg, st.box, st.inp["seq_lens"], k, st.page_idx, st.n_sel, st.workspace(ekv.EKV_OP_SELECT_TOPK))
    wsd = st.workspace(ekv.EKV_OP_DECODE_SPARSE)
    wsb = st.workspace(ekv.EKV_OP_SELECT_BOX_THRESHOLD)
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp, wsd)
    tau_first = st.tau.clone()
    added, ovf = torch.zeros_like(st.n_sel), torch.zeros_like(st.n_sel)
    ekv.ekv_select_box_threshold(st.cfg, st.box, st.inp["seq_lens"], st.tau, st.page_idx, st.n_sel, st.page_idx,
                                 st.n_sel, added, ovf, wsb)                      # in place
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp, wsd)
    added2 = torch.zeros_like(st.n_sel)
    ekv.ekv_select_box_threshold(st.cfg, st.box, st.inp["seq_lens"], st.tau, st.page_idx, st.n_sel, st.page_idx,
                                 st.n_sel, added2, ovf, wsb)
    torch.cuda.synchronize()
    assert int(ovf.sum()) == 0
    assert int(added.sum()) > 0                                # the small budget did miss pages
    assert bool((st.tau >= tau_first - 1e-6).all())            # sparse thresholds only rise towards the full one
    # the refined threshold is exact, so at most pages whose bound sits on it can still be "added"
    assert int(added2.sum()) <= 2
    for (b, hq) in sample_units(w, 4):
        q, K, V = unit_kv(inp, w, b, hq)
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        check_decode_unit(w, st.out[b, hq].cpu().numpy(), float(st.tau[b, hq]), int(st.supp[b, hq]), None, ref)


# ---------------------------------------------------------------------------- page lists shared per KV head
def group_cfg(st, w, cap):
    """Selection calls have batch x n_q_heads rows: for one list per KV head they get n_q_heads = n_kv_heads."""
    return ekv.make_config(w.batch, w.n_kv_heads, w.n_kv_heads, w.head_dim, w.page_size, w.kv_dtype, w.alpha,
                           w.score_scale, st.Mmax, cap)


@pytest.mark.parametrize("w", [W1S, W2, W3, W5], ids=["C1-soft", "C2-8k", "C3-small", "C5-small"])
def test_group_shared_step(w):
    """Group-maximum page score -> top-k per KV head -> grouped sparse decode, stage by stage against the
    oracle: scores on oracle statistics, the selected set up to cut ties, every query head's entmax over
    the shared list."""
    inp = get_inputs(w)
    k = topk_budget(w)
    st = DeviceState(w, inp, cap=k)
    dev = st.box.device
    stats = upload_oracle_stats(st, w, inp)
    gbox = torch.zeros(w.batch, w.n_kv_heads, st.Mmax, device=dev)
    ekv.ekv_score_pages(st.cfg, st.inp["q"], st.stats(), st.inp["seq_lens"], ekv.EKV_SCORE_BOX | ekv.EKV_SCORE_GROUP_MAX,
                        gbox)
    gcfg = group_cfg(st, w, k)
    g_idx = torch.zeros(w.batch, w.n_kv_heads, k, device=dev, dtype=torch.int32)
    g_n = torch.zeros(w.batch, w.n_kv_heads, device=dev, dtype=torch.int32)
    ws_sel = torch.empty(max(256, ekv.ekv_workspace_bytes(gcfg, ekv.EKV_OP_SELECT_TOPK)), device=dev, dtype=torch.uint8)
    ekv.ekv_select_topk(gcfg, gbox, st.inp["seq_lens"], k, g_idx, g_n, ws_sel)
    supp_tok = torch.full((w.batch, w.n_q_heads, 4096), -1, device=dev, dtype=torch.int32)
    ekv.ekv_decode_sparse_group(st.cfg, st.inp["q"], st.cache(), g_idx, g_n, st.out, st.tau, st.supp,
                                st.workspace(ekv.EKV_OP_DECODE_SPARSE), extras=ekv.decode_extras(support_tokens=supp_tok))
    torch.cuda.synchronize()
    gb, gi, gn, toks = gbox.cpu().numpy(), g_idx.cpu().numpy(), g_n.cpu().numpy(), supp_tok.cpu().numpy()
    G = w.group
    for b in range(w.batch):
        for hkv in range(w.n_kv_heads):
            kmin, kmax, _, _, cnt = stats[(b, hkv)]
            M = len(cnt)
            heads = np.stack([orc.box_scores(to_f64(inp["q"][b, hkv * G + g]), kmin, kmax, w.score_scale)
                              for g in range(G)])
            ref_g = orc.group_max_scores(heads)
            assert np.max(np.abs(gb[b, hkv, :M] - ref_g) / np.maximum(1.0, np.abs(ref_g))) <= 1e-5
            assert np.all(np.isneginf(gb[b, hkv, M:]))
            pages, cut_in, cut_out = orc.topk_pages(ref_g, k)
            ok, bad = sets_equal_up_to_cut(gi[b, hkv, : gn[b, hkv]], pages, ref_g, [cut_in, cut_out],
                                           1e-5 * max(1.0, abs(cut_in)))
            assert ok, (b, hkv, bad)
            # every head of the group decodes the list the GPU wrote for its KV head (equal to the oracle's or not)
            for g in range(G if (b, hkv) in ((0, 0), (w.batch - 1, w.n_kv_heads - 1)) else 0):
                hq = hkv * G + g
                q, K, V = unit_kv(inp, w, b, hq)
                check_decode_of_gpu_list(w, q, K, V, gi[b, hkv, : gn[b, hkv]], st.out[b, hq].cpu().numpy(),
                                         st.tau[b, hq], st.supp[b, hq], toks[b, hq])


def test_group_decode_equals_per_head_decode_on_the_same_lists():
    """The same page list given once per KV head, or copied to each of its query heads, must give
    bit-identical results: only the way K is read differs."""
    w = W2
    inp = get_inputs(w)
    k = 96
    st = DeviceState(w, inp, cap=k)
    dev = st.box.device
    rng = np.random.default_rng(9)
    n_pages = -(-int(inp["seq_lens"][0]) // w.page_size)
    g_idx = torch.zeros(w.batch, w.n_kv_heads, k, device=dev, dtype=torch.int32)
    g_n = torch.zeros(w.batch, w.n_kv_heads, device=dev, dtype=torch.int32)
    for hkv in range(w.n_kv_heads):
        cnt = k - (hkv % 3) * 7                                     # ragged list lengths
        pages = np.sort(rng.choice(n_pages, cnt, replace=False)).astype(np.int32)
        g_idx[0, hkv, :cnt] = torch.from_numpy(pages).to(dev)
        g_n[0, hkv] = cnt
        for g in range(w.group):
            st.page_idx[0, hkv * w.group + g, :cnt] = torch.from_numpy(pages).to(dev)
            st.n_sel[0, hkv * w.group + g] = cnt
    wsd = st.workspace(ekv.EKV_OP_DECODE_SPARSE)
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp, wsd)
    out_g, tau_g, supp_g = torch.zeros_like(st.out), torch.zeros_like(st.tau), torch.zeros_like(st.supp)
    ekv.ekv_decode_sparse_group(st.cfg, st.inp["q"], st.cache(), g_idx, g_n, out_g, tau_g, supp_g, wsd)
    torch.cuda.synchronize()
    assert torch.equal(tau_g, st.tau) and torch.equal(supp_g, st.supp) and torch.equal(out_g, st.out)


def test_results_do_not_depend_on_where_pages_live():
    """The same logical cache in three physical arrangements -- a random permutation of exactly the mapped
    pages (the generator's), the identity, and a larger pool with unused pages of garbage between the
    mapped ones -- gives bit-identical statistics, scores, selections and outputs (and the first of them is
    checked against the oracle by the other tests)."""
    w = W2
    inp = get_inputs(w)
    k = topk_budget(w)
    dev = torch.device("cuda")
    P, M = w.page_size, w.pages_per_seq
    n_phys = inp["k_pool"].shape[0]
    results = []
    g = torch.Generator().manual_seed(3)
    for arrangement in ("generated", "identity", "sparse-pool"):
        i2 = dict(inp)
        if arrangement != "generated":
            bt = inp["block_table"].long()                                   # [B, M] -> old physical page
            if arrangement == "identity":
                new_of_logical = torch.arange(w.batch * M).view(w.batch, M)
                pool_pages = w.batch * M
            else:
                pool_pages = 3 * n_phys + 5
                new_of_logical = torch.randperm(pool_pages, generator=g)[: w.batch * M].view(w.batch, M)
            k2 = torch.full((pool_pages,) + tuple(inp["k_pool"].shape[1:]), 1e4).to(inp["k_pool"].dtype)
            v2 = torch.full_like(k2, -1e4)
            k2[new_of_logical.reshape(-1)] = inp["k_pool"][bt.reshape(-1)]
            v2[new_of_logical.reshape(-1)] = inp["v_pool"][bt.reshape(-1)]
            i2.update(k_pool=k2, v_pool=v2, block_table=new_of_logical.to(torch.int32).contiguous())
        st = DeviceState(w, i2, cap=k, device=dev)
        run_step(st, w, "topk", k=k)
        out_f, tau_f, supp_f = torch.zeros_like(st.out), torch.zeros_like(st.tau), torch.zeros_like(st.supp)
        ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), out_f, tau_f, supp_f, st.workspace(ekv.EKV_OP_DECODE_FULL))
        torch.cuda.synchronize()
        results.append([t.clone() for t in (st.box_stats, st.gauss_stats, st.box, st.page_idx, st.n_sel, st.out, st.tau,
                                            st.supp, out_f, tau_f, supp_f)])
    for other in results[1:]:
        for a, b_ in zip(results[0], other):
            assert torch.equal(a.view(torch.uint8), b_.view(torch.uint8))


# ---------------------------------------------------------------------------- multi-step decode loop
def test_multi_step_decode_loop_with_ragged_batch():
    """append -> score -> select -> decode for 40 consecutive steps on a batch whose two sequences have
    different lengths and cross page boundaries at different steps (the lengths are bumped on the device
    between steps, nothing is synchronised inside the loop); the step's results are checked against the
    oracle at several steps, and the statistics at the end against a rebuild."""
    w = synth.C2.scaled(name="C2-loop", batch=2, context=4096, n_q_heads=8, n_kv_heads=2)
    inp = get_inputs(w)
    k = 24
    st = DeviceState(w, inp, cap=k)
    dev = st.box.device
    P, T = w.page_size, 40
    start = torch.tensor([4096 - T - 3, 4096 - T - 14], dtype=torch.int32)       # mid-page, different phases
    B, Hkv = w.batch, w.n_kv_heads
    k_log = torch.stack([torch.stack([synth.logical_kv(inp, w, b, h)[0] for h in range(Hkv)]) for b in range(B)])
    v_log = torch.stack([torch.stack([synth.logical_kv(inp, w, b, h)[1] for h in range(Hkv)]) for b in range(B)])
    st.inp["seq_lens"].copy_(start)
    for b in range(B):                                       # wipe the slots that the loop will fill
        for t in range(int(start[b]), 4096):
            phys = int(inp["block_table"][b, t // P])
            st.inp["k_pool"][phys, :, t % P] = -3.0
            st.inp["v_pool"][phys, :, t % P] = -3.0
    ekv.ekv_stats_build(st.cfg, st.cache(), st.stats())
    check_at = {0, 13, 14, 39}
    snaps = {}
    ws_t, ws_d = st.workspace(ekv.EKV_OP_SELECT_TOPK), st.workspace(ekv.EKV_OP_DECODE_SPARSE)
    for step in range(T):
        pos = (start + step).long()
        k_new = torch.stack([k_log[b, :, pos[b]] for b in range(B)]).contiguous().to(dev)
        v_new = torch.stack([v_log[b, :, pos[b]] for b in range(B)]).contiguous().to(dev)
        ekv.ekv_stats_append(st.cfg, st.cache(), st.stats(), k_new, v_new)
        st.inp["seq_lens"] += 1
        ekv.ekv_score_pages(st.cfg, st.inp["q"], st.stats(), st.inp["seq_lens"], ekv.EKV_SCORE_BOX, st.box)
        ekv.ekv_select_topk(st.cfg, st.box, st.inp["seq_lens"], k, st.page_idx, st.n_sel, ws_t)
        ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp, ws_d)
        if step in check_at:                                 # device-side copies, read after the loop
            snaps[step] = (st.page_idx.clone(), st.n_sel.clone(), st.out.clone(), st.tau.clone(), st.supp.clone())
    torch.cuda.synchronize()
    for step, (idx, ns, out, tau, supp) in snaps.items():
        idx, ns = idx.cpu().numpy(), ns.cpu().numpy()
        for (b, hq) in [(0, 0), (1, 5), (1, 7)]:
            n_b = int(start[b]) + step + 1
            q = to_f64(inp["q"][b, hq])
            K, V = to_f64(k_log[b, hq // w.group, :n_b]), to_f64(v_log[b, hq // w.group, :n_b])
            ref = orc.decode_step_unit(q, K, V, P, w.alpha, w.score_scale, "topk", w.kv_dtype, k_pages=k)
            ok, bad = sets_equal_up_to_cut(idx[b, hq, : ns[b, hq]], ref["pages"], ref["box"],
                                           [ref["cut_in"], ref["cut_out"]], 1e-5 * max(1.0, abs(ref["cut_in"])))
            assert ok, (step, b, hq, bad)
            check_decode_of_gpu_list(w, q, K, V, idx[b, hq, : ns[b, hq]], out[b, hq].cpu().numpy(), tau[b, hq],
                                     supp[b, hq])
    box_a, gauss_a = st.box_stats.clone(), st.gauss_stats.clone()
    ekv.ekv_stats_build(st.cfg, st.cache(), st.stats())
    torch.cuda.synchronize()
    for b in range(B):
        M = -(-(int(start[b]) + T) // P)
        assert torch.equal(box_a[b, :, :M].view(torch.uint8), st.box_stats[b, :, :M].view(torch.uint8))
        assert torch.equal(gauss_a[b, :, :M].view(torch.uint8), st.gauss_stats[b, :, :M].view(torch.uint8))


# ---------------------------------------------------------------------------- shape matrix
SHAPES = [
    synth.C2.scaled(name="C2-p64-g8", context=4096 + 64, ragged=21, page_size=64, n_q_heads=16, n_kv_heads=2),
    synth.C2.scaled(name="C2-p8-g2", context=2048 + 8, ragged=3, page_size=8, n_q_heads=4, n_kv_heads=2),
    synth.C2.scaled(name="C2-p48-g1", context=2400, ragged=11, page_size=48, n_q_heads=2, n_kv_heads=2),
    synth.C1.scaled(name="C1-f32-g4-p32", context=2048 + 32, ragged=5, page_size=32, n_q_heads=8, n_kv_heads=2,
                    scale=0.5 / math.sqrt(128.0)),
    synth.C1.scaled(name="C1-f32-p4-b3", batch=3, context=1024, ragged=1, page_size=4, n_q_heads=2, n_kv_heads=1,
                    scale=0.5 / math.sqrt(128.0)),
    synth.C5.scaled(name="C5-p32-g2-b2", batch=2, context=4096, ragged=31, n_q_heads=4, n_kv_heads=2, alpha=1.25),
    # page sizes that do not divide 64: a group of the decode's score pass is 5 pages of 12 (60 tokens), 2 of 24
    synth.C2.scaled(name="C2-p12-g2", context=12 * 260, ragged=7, page_size=12, n_q_heads=4, n_kv_heads=2),
    synth.C2.scaled(name="C2-p24-g4", context=24 * 150, ragged=23, page_size=24, n_q_heads=8, n_kv_heads=2),
    synth.C1.scaled(name="C1-f32-p20", context=20 * 120, ragged=19, page_size=20, n_q_heads=2, n_kv_heads=2,
                    scale=0.5 / math.sqrt(128.0)),
]


@pytest.mark.parametrize("w", SHAPES, ids=[w.name for w in SHAPES])
def test_shape_matrix_whole_step_and_dense(w):
    """Page sizes 4..64 (matrix-core and plain-FMA paths), group sizes 1..8, both cache dtypes, batches:
    statistics -> box and Gaussian scores -> top-k -> sparse decode, and the dense decode, against the oracle."""
    inp = get_inputs(w)
    k = max(2, w.pages_per_seq // 8)
    st = DeviceState(w, inp, cap=k)
    ekv.ekv_stats_build(st.cfg, st.cache(), st.stats())
    ekv.ekv_score_pages(st.cfg, st.inp["q"], st.stats(), st.inp["seq_lens"], ekv.EKV_SCORE_BOTH, st.box, st.mu, st.sigma)
    ekv.ekv_select_topk(st.cfg, st.box, st.inp["seq_lens"], k, st.page_idx, st.n_sel, st.workspace(ekv.EKV_OP_SELECT_TOPK))
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                          st.workspace(ekv.EKV_OP_DECODE_SPARSE))
    out_f, tau_f, supp_f = torch.zeros_like(st.out), torch.zeros_like(st.tau), torch.zeros_like(st.supp)
    ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), out_f, tau_f, supp_f, st.workspace(ekv.EKV_OP_DECODE_FULL))
    torch.cuda.synchronize()
    idx, ns = st.page_idx.cpu().numpy(), st.n_sel.cpu().numpy()
    box, mu, sigma = st.box.cpu().numpy(), st.mu.cpu().numpy(), st.sigma.cpu().numpy()
    for (b, hq) in sample_units(w, 5):
        q, K, V = unit_kv(inp, w, b, hq)
        ref = orc.decode_step_unit(q, K, V, w.page_size, w.alpha, w.score_scale, "topk", w.kv_dtype, k_pages=k)
        M = len(ref["box"])
        assert np.max(np.abs(box[b, hq, :M] - ref["box"]) / np.maximum(1.0, np.abs(ref["box"]))) <= 1e-5
        _, _, kavg, kstd, cnt = orc.page_stats(K, w.page_size)
        kavg_s, kstd_s = orc.stored_gauss_stats(kavg, kstd, w.kv_dtype)
        ref_mu, ref_sig = orc.gauss_moments(q, kavg_s, kstd_s, w.score_scale)
        # the GPU's own stored mean/variance may sit one storage ulp from the oracle's: compare loosely here
        # (score parity on shared statistics is test_score_pages)
        assert np.max(np.abs(mu[b, hq, :M] - ref_mu)) <= 5e-2 and np.max(np.abs(sigma[b, hq, :M] - ref_sig)) <= 5e-2
        ok, bad = sets_equal_up_to_cut(idx[b, hq, : ns[b, hq]], ref["pages"], ref["box"],
                                       [ref["cut_in"], ref["cut_out"]], 1e-5 * max(1.0, abs(ref["cut_in"])))
        assert ok, (b, hq, bad)
        check_decode_of_gpu_list(w, q, K, V, idx[b, hq, : ns[b, hq]], st.out[b, hq].cpu().numpy(), st.tau[b, hq],
                                 st.supp[b, hq])
        full = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        check_decode_unit(w, out_f[b, hq].cpu().numpy(), float(tau_f[b, hq]), int(supp_f[b, hq]), None, full)


# ---------------------------------------------------------------------------- fused append + score
WSHORT = synth.C2.scaled(name="C2-short", context=8192, ragged=8192 - 1000)      # most score tiles lie past the end


@pytest.mark.parametrize("w", [W1R, W2, W5, WP8, WSHORT], ids=["C1-ragged", "C2-8k", "C5-small", "C2-p8-g2", "C2-short"])
@pytest.mark.parametrize("mode", ["box", "gauss", "both", "group"])
def test_fused_append_score_equals_the_two_calls(w, mode):
    """ekv_append_score_pages == ekv_stats_append then ekv_score_pages with the lengths + 1, bit for bit
    (cache, statistics, scores), over steps that fill a page, cross into a new one and continue."""
    inp = get_inputs(w)
    P, B, Hkv = w.page_size, w.batch, w.n_kv_heads
    n_final = int(inp["seq_lens"][0])
    steps = P + 2
    n0 = n_final - steps
    k_log = torch.stack([torch.stack([synth.logical_kv(inp, w, b, h)[0] for h in range(Hkv)]) for b in range(B)])
    v_log = torch.stack([torch.stack([synth.logical_kv(inp, w, b, h)[1] for h in range(Hkv)]) for b in range(B)])
    flags = {"box": ekv.EKV_SCORE_BOX, "gauss": ekv.EKV_SCORE_GAUSS, "both": ekv.EKV_SCORE_BOTH,
             "group": ekv.EKV_SCORE_BOX | ekv.EKV_SCORE_GROUP_MAX}[mode]
    results = []
    for fused in (False, True):
        st = DeviceState(w, inp)
        dev = st.box.device
        box = torch.zeros(B, Hkv if mode == "group" else w.n_q_heads, st.Mmax, device=dev)
        st.inp["seq_lens"].fill_(n0)
        for b in range(B):                                   # wipe the slots that will be appended
            for t in range(n0, n_final):
                phys = int(inp["block_table"][b, t // P])
                st.inp["k_pool"][phys, :, t % P] = 5.0
                st.inp["v_pool"][phys, :, t % P] = 5.0
        ekv.ekv_stats_build(st.cfg, st.cache(), st.stats())
        snaps = []
        for t in range(n0, n_final):
            k_new = k_log[:, :, t].contiguous().to(dev); v_new = v_log[:, :, t].contiguous().to(dev)
            args = dict(box=box if mode != "gauss" else None, mu=st.mu if mode in ("gauss", "both") else None,
                        sigma=st.sigma if mode in ("gauss", "both") else None)
            if fused:
                ekv.ekv_append_score_pages(st.cfg, st.cache(), st.stats(), k_new, v_new, st.inp["q"], flags, **args)
                st.inp["seq_lens"] += 1
            else:
                ekv.ekv_stats_append(st.cfg, st.cache(), st.stats(), k_new, v_new)
                st.inp["seq_lens"] += 1
                ekv.ekv_score_pages(st.cfg, st.inp["q"], st.stats(), st.inp["seq_lens"], flags, **args)
            snaps.append((box.clone(), st.mu.clone(), st.sigma.clone()))
        torch.cuda.synchronize()
        results.append((st.inp["k_pool"].cpu(), st.inp["v_pool"].cpu(), st.box_stats.cpu(), st.gauss_stats.cpu(), snaps))
    a, b_ = results
    M = -(-n_final // P)
    assert torch.equal(a[0], b_[0]) and torch.equal(a[1], b_[1])
    assert torch.equal(a[0], inp["k_pool"]) and torch.equal(a[1], inp["v_pool"])
    assert torch.equal(a[2][:, :, :M].view(torch.uint8), b_[2][:, :, :M].view(torch.uint8))
    assert torch.equal(a[3][:, :, :M].view(torch.uint8), b_[3][:, :, :M].view(torch.uint8))
    for (ba, ma, sa), (bb, mb, sb) in zip(a[4], b_[4]):
        assert torch.equal(ba.view(torch.int32), bb.view(torch.int32))
        assert torch.equal(ma.view(torch.int32), mb.view(torch.int32))
        assert torch.equal(sa.view(torch.int32), sb.view(torch.int32))


# ---------------------------------------------------------------------------- trend of the paper's selector table
def test_gauss_selector_on_plain_random_inputs_follows_the_papers_trend():
    """q, K, V ~ N(0,1), batch 8, page 16 (the setting of the paper's selector-quality table, App. E): the
    estimated threshold is close to the exact full-cache one, the fraction of pages kept falls as the
    context grows, and at 4K/8K tokens almost nothing of the mass is dropped.  (The table's own numbers
    depend on hyper-parameters the paper does not state; only the trend is checked.)"""
    dev = torch.device("cuda")
    cov, delta, gap = [], [], []
    for n in (4096, 8192, 16384, 32768):
        w = synth.Workload("randn", 8, 8, 8, 128, n, 16, "bf16")
        inp = synth.make_inputs(w, 9000 + n, device=dev)
        st = DeviceState(w, inp, cap=w.pages_per_seq, device=dev)
        ekv.ekv_stats_build(st.cfg, st.cache(), st.stats())
        ekv.ekv_score_pages(st.cfg, inp["q"], st.stats(), inp["seq_lens"], ekv.EKV_SCORE_GAUSS, None, st.mu, st.sigma)
        ekv.ekv_select_gauss(st.cfg, st.mu, st.sigma, inp["seq_lens"], 0.99, 0.0, st.tau_hat, st.page_idx, st.n_sel,
                             st.overflow, st.workspace(ekv.EKV_OP_SELECT_GAUSS))
        out_f, tau_f, supp_f = torch.zeros_like(st.out), torch.zeros_like(st.tau), torch.zeros_like(st.supp)
        ekv.ekv_decode_full(st.cfg, inp["q"], st.cache(), out_f, tau_f, supp_f, st.workspace(ekv.EKV_OP_DECODE_FULL))
        km = torch.zeros_like(st.tau)
        ekv.ekv_decode_sparse(st.cfg, inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                              st.workspace(ekv.EKV_OP_DECODE_SPARSE),
                              extras=ekv.decode_extras(tau_ref=tau_f, kept_mass_ref=km))
        torch.cuda.synchronize()
        cov.append(float(st.n_sel.float().mean()) / w.pages_per_seq)
        delta.append(float((1.0 - km).mean()))
        gap.append(float((st.tau_hat - tau_f).abs().mean()))
        assert float((st.tau - tau_f).max()) <= 1e-6          # a sparse threshold never exceeds the full one
    assert all(a > b for a, b in zip(cov, cov[1:])), cov
    assert delta[0] <= 0.01 and delta[1] <= 0.02, delta
    assert all(a <= b + 1e-3 for a, b in zip(delta, delta[1:])), delta
    assert max(gap) <= 0.1, gap


# ---------------------------------------------------------------------------- an idle batch slot
@pytest.mark.parametrize("kv_dtype,context,lens", [("bf16", 2048, [2048 - 5, 0, 37]), ("f32", 2048, [2048 - 5, 0, 37]),
                                                  ("bf16", 70000, [70000 - 3, 0])],
                         ids=["bf16", "f32", "bf16-long-rows"])
def test_batch_slot_with_zero_tokens(kv_dtype, context, lens):
    """A sequence of length 0 (an idle slot of a serving batch) next to live ones: every entry point runs,
    the idle slot gets the documented empty results (no page, zero output, tau = +inf, empty support,
    log-sum-exp = -inf, tau-hat = 0), and the live sequences match the oracle as if the slot were not there.
    Then a first token is appended to the idle slot and the step serves it.  (Beside rows that take the filter passes:
    test_filter_passes_beside_short_and_empty_rows.)"""
    w = synth.C2.scaled(name="C2-idle-slot", batch=len(lens), context=context, n_q_heads=4, n_kv_heads=2,
                        kv_dtype=kv_dtype)
    inp = {key: v.clone() for key, v in synth.make_inputs(w, 2000 + 31, device="cpu").items()}
    inp["seq_lens"] = torch.tensor(lens, dtype=torch.int32)
    live = [b for b, n_b in enumerate(lens) if n_b > 0]
    k = 8
    st = DeviceState(w, inp, cap=16)
    dev = st.box.device
    P = w.page_size

    def run(selector):
        run_step(st, w, selector, k=k, q_page=0.9, margin=0.02)
        full = dict(out=torch.zeros_like(st.out), tau=torch.zeros_like(st.tau), supp=torch.zeros_like(st.supp),
                    lse=torch.zeros_like(st.tau))
        ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), full["out"], full["tau"], full["supp"],
                            st.workspace(ekv.EKV_OP_DECODE_FULL), extras=ekv.decode_extras(lse=full["lse"]))
        sm_out, sm_lse = torch.full_like(st.out, 7.0), torch.full_like(st.tau, 7.0)
        ekv.ekv_decode_sparse_softmax(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, sm_out, sm_lse,
                                      st.workspace(ekv.EKV_OP_DECODE_SPARSE_SOFTMAX))
        ref_idx, ref_n = torch.zeros_like(st.page_idx), torch.full_like(st.n_sel, 7)
        added, ovf = torch.full_like(st.n_sel, 7), torch.full_like(st.n_sel, 7)
        ekv.ekv_select_box_threshold(st.cfg, st.box, st.inp["seq_lens"], st.tau, st.page_idx, st.n_sel, ref_idx, ref_n,
                                     added, ovf, st.workspace(ekv.EKV_OP_SELECT_BOX_THRESHOLD))
        km, kn = torch.full_like(st.tau, 7.0), torch.full_like(st.supp, 7)
        ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                              st.workspace(ekv.EKV_OP_DECODE_SPARSE),
                              extras=ekv.decode_extras(tau_ref=full["tau"], kept_mass_ref=km, kept_supp_ref=kn))
        torch.cuda.synchronize()
        assert torch.all(km[1] == 0) and torch.all(kn[1] == 0)
        assert torch.all((km[live] >= 0) & (km[live] <= 1.0 + 1e-5)) and torch.all((kn[live] >= 0) & (kn[live] <= full["supp"][live]))
        return full, sm_out, sm_lse, ref_n, added

    for selector in ("topk", "gauss"):
        st.out.fill_(7.0); st.tau.fill_(7.0); st.supp.fill_(7); st.n_sel.fill_(7); st.tau_hat.fill_(7.0)
        if selector == "topk":
            st.box.fill_(7.0)
        full, sm_out, sm_lse, ref_n, added = run(selector)
        # the idle slot
        assert torch.all(st.n_sel[1] == 0) and torch.all(st.supp[1] == 0) and torch.all(full["supp"][1] == 0)
        assert torch.all(st.out[1] == 0) and torch.all(full["out"][1] == 0) and torch.all(sm_out[1] == 0)
        assert torch.all(torch.isposinf(st.tau[1])) and torch.all(torch.isposinf(full["tau"][1]))
        assert torch.all(torch.isneginf(full["lse"][1])) and torch.all(torch.isneginf(sm_lse[1]))
        assert torch.all(ref_n[1] == 0) and torch.all(added[1] == 0)
        if selector == "topk":
            assert torch.all(torch.isneginf(st.box[1]))
        else:
            assert torch.all(st.tau_hat[1] == 0) and torch.all(torch.isneginf(st.mu[1])) and torch.all(st.sigma[1] == 0)
        # the live sequences
        for b in live:
            for hq in (0, 3):
                q, K, V = unit_kv(inp, w, b, hq)
                if selector == "topk":
                    ref = orc.decode_step_unit(q, K, V, P, w.alpha, w.score_scale, "topk", w.kv_dtype, k_pages=k)
                else:
                    ref = orc.decode_step_unit(q, K, V, P, w.alpha, w.score_scale, "gauss", w.kv_dtype, q_page=0.9,
                                               margin=0.02, cap=16)
                    if ref["overflow"]:
                        continue
                got = st.page_idx[b, hq, : int(st.n_sel[b, hq])].cpu().numpy()
                check_decode_of_gpu_list(w, q, K, V, got, st.out[b, hq].cpu().numpy(), st.tau[b, hq], st.supp[b, hq])
                dense = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
                check_decode_unit(w, full["out"][b, hq].cpu().numpy(), float(full["tau"][b, hq]),
                                  int(full["supp"][b, hq]), None, dense)

    # the idle slot receives its first token
    g = torch.Generator().manual_seed(5)
    k_new = torch.randn(w.batch, w.n_kv_heads, w.head_dim, generator=g).to(st.inp["k_pool"].dtype).to(dev)
    v_new = torch.randn(w.batch, w.n_kv_heads, w.head_dim, generator=g).to(st.inp["k_pool"].dtype).to(dev)
    ekv.ekv_append_score_pages(st.cfg, st.cache(), st.stats(), k_new, v_new, st.inp["q"], ekv.EKV_SCORE_BOX, st.box,
                               None, None)
    st.inp["seq_lens"] += 1
    ekv.ekv_select_topk(st.cfg, st.box, st.inp["seq_lens"], k, st.page_idx, st.n_sel, st.workspace(ekv.EKV_OP_SELECT_TOPK))
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                          st.workspace(ekv.EKV_OP_DECODE_SPARSE))
    torch.cuda.synchronize()
    assert torch.all(st.n_sel[1] == 1) and torch.all(st.page_idx[1, :, 0] == 0) and torch.all(st.supp[1] == 1)
    # one token: p = (1), the output is its value row
    for hq in range(w.n_q_heads):
        np.testing.assert_allclose(st.out[1, hq].cpu().numpy(), v_new[1, hq // w.group].float().cpu().numpy(),
                                   rtol=1e-6, atol=0)


@pytest.mark.parametrize("Mmax,k", [(100, 7), (700, 14), (1024, 1024), (2048, 41)])
def test_select_topk_many_short_rows(Mmax, k):
    """More than 512 short rows take the one-wavefront-per-row kernel: ragged lengths (0 and 1 token
    included), ties, constant rows, both signs, k larger than a row."""
    P, B, Hq = 16, 20, 32
    cfg = ekv.make_config(B, Hq, Hq, 128, P, "bf16", 1.5, 0.1, Mmax, k)
    dev = torch.device("cuda")
    rng = np.random.default_rng(Mmax + k)
    scores = (rng.normal(size=(B, Hq, Mmax)) * 3.0 + 1.0).astype(np.float32)
    scores[:, 1] = 2.5                                             # all equal: the lowest indices win
    scores[:, 2] = np.round(scores[:, 2])                          # heavy ties
    scores[:, 3, ::2] = scores[:, 3, 1::2]                         # every value twice
    lens = rng.integers(1, Mmax * P + 1, size=B).astype(np.int32)
    lens[0], lens[1], lens[2], lens[3] = Mmax * P, 0, 1, Mmax * P - 5
    box = torch.from_numpy(scores).to(dev)
    seq_lens = torch.from_numpy(lens).to(dev)
    page_idx = torch.full((B, Hq, k), -1, dtype=torch.int32, device=dev)
    n_sel = torch.full((B, Hq), -1, dtype=torch.int32, device=dev)
    ws = torch.empty(max(256, ekv.ekv_workspace_bytes(cfg, ekv.EKV_OP_SELECT_TOPK)), dtype=torch.uint8, device=dev)
    ekv.ekv_select_topk(cfg, box, seq_lens, k, page_idx, n_sel, ws)
    torch.cuda.synchronize()
    idx, ns = page_idx.cpu().numpy(), n_sel.cpu().numpy()
    for b in range(B):
        M = -(-int(lens[b]) // P)
        for hq in (0, 1, 2, 3, 17, 31):
            if M == 0:
                assert ns[b, hq] == 0
                continue
            ref, _, _ = orc.topk_pages(scores[b, hq, :M].astype(np.float64), k)
            assert ns[b, hq] == len(ref)
            np.testing.assert_array_equal(idx[b, hq, : ns[b, hq]], ref)


@pytest.mark.parametrize("kv_dtype,ctx,k,scale,alpha", [("bf16", 2048, 8, 1.0, 1.5), ("bf16", 4096, 100, 1.0, 1.5),
                                                        ("f32", 1024, 20, 1.0, 1.5), ("bf16", 2048, 40, 0.02, 1.5),
                                                        ("bf16", 2048, 16, 1.0, 1.25), ("bf16", 2048, 16, 1.0, 2.0)],
                         ids=["bf16-8-pages", "bf16-100-pages", "f32-20-pages", "bf16-flat-scores", "alpha-1.25",
                              "alpha-2"])
def test_many_short_rows_step(kv_dtype, ctx, k, scale, alpha):
    """More than 512 (sequence, head) rows with short page lists take the one-wavefront-per-row selection, the one-launch
    decode and, as lists shared per KV head, the solve by one wavefront per row (by four, for the 100 pages): whole top-k
    step and the group-shared decode against the oracle on sampled rows, ragged lengths; the flat-score case has more
    candidates than one wavefront finishes in registers."""
    w = synth.C2.scaled(name="C2-many-rows", batch=24, context=ctx, n_q_heads=32, n_kv_heads=8, kv_dtype=kv_dtype,
                        n_planted=8, scale=scale / math.sqrt(128.0), alpha=alpha)
    inp = {key: v.clone() for key, v in synth.make_inputs(w, 2000 + 77, device="cpu").items()}
    rng = np.random.default_rng(3)
    lens = rng.integers(1, ctx + 1, size=w.batch).astype(np.int32)
    lens[0], lens[1] = ctx, 5
    inp["seq_lens"] = torch.from_numpy(lens)
    st = DeviceState(w, inp, cap=k)
    dev = st.box.device
    toks = torch.full((w.batch, w.n_q_heads, 2048), -1, dtype=torch.int32, device=dev)
    ekv.ekv_stats_build(st.cfg, st.cache(), st.stats())
    ekv.ekv_score_pages(st.cfg, st.inp["q"], st.stats(), st.inp["seq_lens"], ekv.EKV_SCORE_BOX, st.box)
    ekv.ekv_select_topk(st.cfg, st.box, st.inp["seq_lens"], k, st.page_idx, st.n_sel, st.workspace(ekv.EKV_OP_SELECT_TOPK))
    full = dict(out=torch.zeros_like(st.out), tau=torch.zeros_like(st.tau), supp=torch.zeros_like(st.supp))
    ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), full["out"], full["tau"], full["supp"],
                        st.workspace(ekv.EKV_OP_DECODE_FULL))
    km, kn = torch.zeros_like(st.tau), torch.zeros_like(st.supp)
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                          st.workspace(ekv.EKV_OP_DECODE_SPARSE),
                          extras=ekv.decode_extras(support_tokens=toks, tau_ref=full["tau"], kept_mass_ref=km,
                                                   kept_supp_ref=kn))
    torch.cuda.synchronize()
    P = w.page_size
    for (b, hq) in [(0, 0), (0, 31), (1, 5), (7, 12), (13, 20), (23, 9)]:
        q, K, V = unit_kv(inp, w, b, hq)
        ref = orc.decode_step_unit(q, K, V, P, w.alpha, w.score_scale, "topk", w.kv_dtype, k_pages=k)
        got = st.page_idx[b, hq, : int(st.n_sel[b, hq])].cpu().numpy()
        band = 1e-5 * max(1.0, abs(ref["cut_in"]))
        ok, bad = sets_equal_up_to_cut(got, ref["pages"], ref["box"], [ref["cut_in"], ref["cut_out"]], band)
        assert ok, (b, hq, bad)
        own = check_decode_of_gpu_list(w, q, K, V, got, st.out[b, hq].cpu().numpy(), st.tau[b, hq], st.supp[b, hq],
                                       toks[b, hq].cpu().numpy())
        dense = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        assert abs((1.0 - float(km[b, hq])) - orc.dropped_mass(dense["p"], own["tokens"])) <= 1e-4
    # a warm start (the exact thresholds as seeds) changes nothing but the number of evaluations
    out2, tau2, supp2 = torch.zeros_like(st.out), torch.zeros_like(st.tau), torch.zeros_like(st.supp)
    evals = torch.full_like(st.supp, -1)
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, out2, tau2, supp2,
                          st.workspace(ekv.EKV_OP_DECODE_SPARSE),
                          extras=ekv.decode_extras(tau_seed=st.tau, solve_evals=evals))
    torch.cuda.synchronize()
    assert torch.equal(supp2, st.supp)
    assert torch.allclose(tau2, st.tau, rtol=0, atol=4e-6)
    # (a threshold that moves within its tolerance moves the weights of a flat row by far more, relatively)
    assert float(((out2 - st.out).norm(dim=-1) / st.out.norm(dim=-1).clamp_min(1e-30)).max()) <= 2e-3
    assert int(evals.min()) >= 0 and int(evals.max()) <= 8
    # one list per KV head
    gcfg = group_cfg(st, w, k)
    gbox = torch.zeros(w.batch, w.n_kv_heads, st.Mmax, device=dev)
    g_idx = torch.zeros(w.batch, w.n_kv_heads, k, dtype=torch.int32, device=dev)
    g_n = torch.zeros(w.batch, w.n_kv_heads, dtype=torch.int32, device=dev)
    ekv.ekv_score_pages(st.cfg, st.inp["q"], st.stats(), st.inp["seq_lens"], ekv.EKV_SCORE_BOX | ekv.EKV_SCORE_GROUP_MAX, gbox)
    ekv.ekv_select_topk(gcfg, gbox, st.inp["seq_lens"], k, g_idx, g_n,
                        torch.empty(max(256, ekv.ekv_workspace_bytes(gcfg, ekv.EKV_OP_SELECT_TOPK)), device=dev, dtype=torch.uint8))
    ekv.ekv_decode_sparse_group(st.cfg, st.inp["q"], st.cache(), g_idx, g_n, st.out, st.tau, st.supp,
                                st.workspace(ekv.EKV_OP_DECODE_SPARSE))
    torch.cuda.synchronize()
    for (b, hq) in [(0, 3), (7, 12), (23, 30)]:
        q, K, V = unit_kv(inp, w, b, hq)
        pages = g_idx[b, hq // w.group, : int(g_n[b, hq // w.group])].cpu().numpy()
        tok = orc.pages_to_tokens(pages, P, K.shape[0])
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale, tok)
        check_decode_unit(w, st.out[b, hq].cpu().numpy(), float(st.tau[b, hq]), int(st.supp[b, hq]), None, ref)


@pytest.mark.parametrize("M,k,levels", [(21003, 400, 16), (299999, 777, 0), (299999, 5000, 64)])
def test_select_topk_memory_backed_rows_of_odd_length(M, k, levels):
    """The one-workgroup selection that reads its keys from memory (rows beyond the sliced kernels' range,
    and rows whose k-th key has thousands of exact ties) with a page count that leaves the last batch of
    key slots of a lane partly in the next wavefront's range."""
    P, B, Hq = 16, 1, 3
    Mmax = -(-M // 64) * 64
    cfg = ekv.make_config(B, Hq, Hq, 128, P, "bf16", 1.5, 0.1, Mmax, k)
    dev = torch.device("cuda")
    rng = np.random.default_rng(M + k)
    scores = (rng.normal(size=(B, Hq, Mmax)) * 3.0 + 17.0).astype(np.float32)
    if levels:
        scores[0, 1] = np.round(np.clip(scores[0, 1], 10, 10 + levels - 1))      # `levels` distinct values
        scores[0, 2] = 3.25                                                       # one value
    box = torch.from_numpy(scores).to(dev)
    seq_lens = torch.full((B,), M * P - 2, dtype=torch.int32, device=dev)
    page_idx = torch.full((B, Hq, k), -1, dtype=torch.int32, device=dev)
    n_sel = torch.zeros(B, Hq, dtype=torch.int32, device=dev)
    ws = torch.empty(max(256, ekv.ekv_workspace_bytes(cfg, ekv.EKV_OP_SELECT_TOPK)), dtype=torch.uint8, device=dev)
    ekv.ekv_select_topk(cfg, box, seq_lens, k, page_idx, n_sel, ws)
    torch.cuda.synchronize()
    idx, ns = page_idx.cpu().numpy(), n_sel.cpu().numpy()
    for hq in range(Hq):
        ref, _, _ = orc.topk_pages(scores[0, hq, :M].astype(np.float64), k)
        assert ns[0, hq] == len(ref)
        np.testing.assert_array_equal(idx[0, hq, : ns[0, hq]], ref)


def test_select_gauss_many_short_rows():
    """768 (sequence, head) rows of at most 200 pages, ragged lengths (0 and 1 token included): one slice per row,
    one page per wavefront lane at most; tau-hat and the page sets against the oracle on sampled rows."""
    P, B, Hq, Mmax = 16, 24, 32, 200
    cfg = ekv.make_config(B, Hq, Hq, 128, P, "bf16", 1.5, 0.1, Mmax, Mmax)
    dev = torch.device("cuda")
    rng = np.random.default_rng(5)
    mu = (rng.normal(size=(B, Hq, Mmax)) * 0.6 + 1.0).astype(np.float32)
    sg = (np.abs(rng.normal(size=(B, Hq, Mmax))) * 0.3 + 0.2).astype(np.float32)
    mu[:, 3, 7] += 6.0                                             # one hot page per row of head 3
    lens = rng.integers(1, Mmax * P + 1, size=B).astype(np.int32)
    lens[0], lens[1], lens[2] = Mmax * P, 0, 1
    seq_lens = torch.from_numpy(lens).to(dev)
    t = lambda a: torch.from_numpy(a).to(dev)
    tau_hat = torch.zeros(B, Hq, device=dev); page_idx = torch.zeros(B, Hq, Mmax, dtype=torch.int32, device=dev)
    n_sel = torch.full((B, Hq), -1, dtype=torch.int32, device=dev); ovf = torch.zeros_like(n_sel)
    ws = torch.empty(ekv.ekv_workspace_bytes(cfg, ekv.EKV_OP_SELECT_GAUSS), dtype=torch.uint8, device=dev)
    ekv.ekv_select_gauss(cfg, t(mu), t(sg), seq_lens, 0.9, 0.02, tau_hat, page_idx, n_sel, ovf, ws)
    torch.cuda.synchronize()
    assert int(ovf.sum()) == 0
    for b in range(B):
        n = int(lens[b]); M = -(-n // P)
        for hq in (0, 3, 17, 31):
            if M == 0:
                assert int(n_sel[b, hq]) == 0
                continue
            cnt = np.full(M, P); cnt[-1] = n - (M - 1) * P
            pages, th, o, g = orc.gauss_select(mu[b, hq, :M].astype(np.float64), sg[b, hq, :M].astype(np.float64), cnt, 1.5,
                                               0.9, 0.02, cap=Mmax)
            assert abs(float(tau_hat[b, hq]) - th) <= 4e-6 * max(1.0, abs(th)), (b, hq, float(tau_hat[b, hq]), th)
            got = page_idx[b, hq, : int(n_sel[b, hq])].cpu().numpy()
            cut = th - 0.02
            ok, bad = sets_equal_up_to_cut(got, pages, g, cut, 1e-5 * max(1.0, abs(cut)))
            assert ok, (b, hq, bad[:5], len(pages), len(got))
            assert np.all(np.diff(got) > 0)


# ---------------------------------------------------------------------------- list capacity
def test_decode_does_not_depend_on_the_capacity_of_the_page_lists():
    """The same page lists in buffers of 1x, 3x and 8x their length (max_sel_pages): the launches are sized by the
    device-side lengths, so every output is identical bit for bit -- per-head lists, one list per KV head, softmax
    over the lists -- and equal to the oracle's decode of those lists.  Ragged lengths, one empty list."""
    w = W2
    inp = get_inputs(w)
    k = 50
    dev = torch.device("cuda")
    rng = np.random.default_rng(21)
    n_pages = -(-int(inp["seq_lens"][0]) // w.page_size)
    lens = rng.integers(1, k + 1, size=(w.batch, w.n_q_heads)); lens[0, 3] = 0; lens[0, 0] = k
    lists = {(b, h): np.sort(rng.choice(n_pages, lens[b, h], replace=False)) for b in range(w.batch) for h in range(w.n_q_heads)}
    results = []
    for mult in (1, 3, 8):
        cap = k * mult
        st = DeviceState(w, inp, cap=cap)
        st.page_idx.fill_(n_pages + 7)                         # slots past the lengths hold an out-of-range page
        for (b, h), pg in lists.items():
            st.page_idx[b, h, : len(pg)] = torch.from_numpy(pg.astype(np.int32)).to(dev)
        st.n_sel.copy_(torch.from_numpy(lens.astype(np.int32)))
        toks = torch.full((w.batch, w.n_q_heads, 512), -1, device=dev, dtype=torch.int32)
        ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                              st.workspace(ekv.EKV_OP_DECODE_SPARSE), extras=ekv.decode_extras(support_tokens=toks))
        r = [st.out.clone(), st.tau.clone(), st.supp.clone(), toks.clone()]
        # one list per KV head: the lists of the group's first head
        g_idx = st.page_idx[:, :: w.group].contiguous(); g_n = st.n_sel[:, :: w.group].contiguous()
        ekv.ekv_decode_sparse_group(st.cfg, st.inp["q"], st.cache(), g_idx, g_n, st.out, st.tau, st.supp,
                                    st.workspace(ekv.EKV_OP_DECODE_SPARSE))
        r += [st.out.clone(), st.tau.clone(), st.supp.clone()]
        lse = torch.zeros_like(st.tau)
        ekv.ekv_decode_sparse_softmax(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, lse,
                                      st.workspace(ekv.EKV_OP_DECODE_SPARSE_SOFTMAX))
        r += [st.out.clone(), lse.clone()]
        torch.cuda.synchronize()
        results.append(r)
    for other in results[1:]:
        for i, (a, b_) in enumerate(zip(results[0], other)):
            assert torch.equal(a.view(torch.uint8), b_.view(torch.uint8)), i
    out, tau, supp, toks = [t.cpu().numpy() for t in results[0][:4]]
    assert supp[0, 3] == 0 and np.isposinf(tau[0, 3]) and not out[0, 3].any()
    for (b, hq) in [(0, 0), (0, 7), (0, 30)]:
        q, K, V = unit_kv(inp, w, b, hq)
        check_decode_of_gpu_list(w, q, K, V, lists[(b, hq)], out[b, hq], tau[b, hq], supp[b, hq], toks[b, hq])
