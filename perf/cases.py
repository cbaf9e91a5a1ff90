"""The decode hot path as a serving program calls it, over the sizes of this repository's workloads, tests and
benchmark: what is prepared once, one pass through the public entry points, and what the results are in 64 bits.

Kinds of a pass (all over a paged KV cache that is resident on the GPU):
  topk     append + box scores -> top-k pages -> sparse entmax decode          (the headline decode step)
  topk8    the same on the 8-bit page bounds
  group    append + group-maximum box scores -> one list per KV head -> sparse decode of the group
  group8   the same on the 8-bit page bounds
  gauss    append + Gaussian page moments -> Gaussian-aware selector -> sparse entmax decode
  softmax  append + box scores -> top-k pages -> softmax over the selection    (the comparison path)
  refine   append + box scores -> top-k -> decode -> box threshold -> decode   (the exactly recovered result)
  dense    full-cache entmax decode
  build    bulk page statistics, what a prefill ends with
"""
import math

import torch

from paper_2605_21649_amd import binding as ekv
from paper_2605_21649_amd import synth

D = 128
APPENDING = ("topk", "topk8", "group", "group8", "gauss", "softmax", "refine")


def _case(name, kind, batch, heads, tokens, page=16, dtype="bf16", alpha=1.5, flat=1.0, budget=0.02, stagger=0,
          planted=64, spans=0, outliers=4):
    """heads: (query heads, KV heads).  stagger: sequence b is b * stagger tokens shorter than the longest (a batch
    of requests is never level).  flat: factor on the score scale, below 1 a flatter attention with a larger support."""
    c = dict(kind=kind, batch=batch, q_heads=heads[0], kv_heads=heads[1], tokens=tokens, page=page, dtype=dtype,
             alpha=alpha, flat=flat, budget=budget, stagger=stagger, planted=planted, spans=spans, outliers=outliers)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one short sequence on a float32 cache without grouped heads, a chain of launches
        _case("topk-1x4k-f32", "topk", 1, (8, 8), 4096, dtype="f32", planted=32, outliers=0, budget=0.125, flat=0.5),
        # a single million-token sequence, the benchmark's step
        _case("topk-1x1m", "topk", 1, (32, 8), 1048576),
        # a serving batch of many short chats: thousands of short rows, every length different
        _case("topk-64x8k", "topk", 64, (32, 8), 8192, stagger=37),
        # eight long sequences, pages of 32, lists shared by the heads of a group, 8-bit bounds
        _case("group8-8x256k-p32", "group8", 8, (32, 8), 262144, page=32, budget=1.0 / 64),
        # the adaptive selector on one ordinary context, and on a batch of long ones with clustered support
        _case("gauss-1x32k", "gauss", 1, (32, 8), 32763),
        _case("gauss-4x128k", "gauss", 4, (32, 8), 131072, spans=8),
        # softmax over the same lists, the path entmax is compared with; uneven lengths
        _case("softmax-4x128k", "softmax", 4, (32, 8), 131072, stagger=9001, spans=8),
        # the certified exact result on a float32 cache, pages of 8 tokens, uneven lengths
        _case("refine-3x21k-f32-p8", "refine", 3, (16, 8), 21003, page=8, dtype="f32", stagger=1777),
        # full-cache decode: one ordinary context, a flat attention with thousands of support tokens, and the largest
        # call of all (eight sequences of 256K tokens, a smaller alpha)
        _case("dense-1x32k", "dense", 1, (32, 8), 32763),
        _case("dense-1x256k-flat", "dense", 1, (32, 8), 262144, flat=0.06),
        _case("dense-8x256k-p32-a125", "dense", 8, (32, 8), 262144, page=32, alpha=1.25),
        # statistics of freshly prefilled sequences
        _case("build-4x128k", "build", 4, (32, 8), 131072, stagger=4097),
    ]


def draw(rng):
    kind = rng.choice(("topk", "topk", "topk8", "group", "group8", "gauss", "gauss", "softmax", "refine", "dense", "dense",
                       "build"))
    dtype = "f32" if rng.random() < 0.25 and kind not in ("topk8", "group8") else "bf16"
    heads = rng.choice(((8, 8), (16, 8), (32, 8), (32, 8), (32, 8), (64, 8), (8, 1), (4, 4)))
    page = rng.choice((8, 16, 16, 16, 32, 32, 64, 12, 48))
    tokens = int(round(2.0 ** rng.uniform(11, 20))) - rng.choice((0, 0, 1, 5, 13))
    esz = 4 if dtype == "f32" else 2
    # bytes of K of the largest draw: below the largest listed case's, less where a pass reads them several times or
    # goes through the plain FMA path
    most = 3.0e9
    if kind == "build":
        most = 2.0e9
    if kind == "refine":
        most = 1.2e9 / (heads[0] // heads[1])
    if dtype == "f32" or page not in (16, 32, 64):
        most /= 3
    while tokens * heads[1] * D * esz > most:
        tokens = tokens // 2 + 1
    room = most / (tokens * heads[1] * D * esz)
    batch = max(1, min(64, int(2.0 ** rng.uniform(0, math.log2(max(room, 1.0)) + 1e-9))))
    stagger = 0 if batch == 1 or rng.random() < 0.3 else rng.randint(1, max(1, tokens // (2 * batch)))
    return _case(None, kind, batch, heads, tokens, page, dtype, rng.choice((1.25, 4.0 / 3.0, 1.5, 1.5, 1.5, 2.0)),
                 rng.choice((1.0, 1.0, 1.0, 0.25, 0.06)) if kind in ("topk", "dense") else 1.0,
                 rng.choice((0.01, 0.02, 0.04, 0.125)), stagger, rng.choice((32, 64)), rng.choice((0, 0, 8)),
                 rng.choice((0, 4)))


# ---- sizes --------------------------------------------------------------------------------------------------------
def _lens(c):
    return [c["tokens"] - b * c["stagger"] for b in range(c["batch"])]


def _pages(c):
    return -(-c["tokens"] // c["page"])


def _k_pages(c):
    return max(1, math.ceil(c["budget"] * _pages(c)))


def _cap(c):
    m, k = _pages(c), _k_pages(c)
    if c["kind"] == "refine":
        return m
    if c["kind"] == "gauss":
        return min(m, max(math.ceil(0.25 * m), 2048))
    return min(m, 2 * k)


def _scale(c):
    return c["flat"] / math.sqrt(D)


def work(case):
    """Each input read once, each output written once: statistics or K of every page the path has to look at, K of the
    selected pages once per list, scores and statistics it returns.  V rows of the support are a few kilobytes per
    head and counted as 32 rows; for the Gaussian selector, whose budget is adaptive, one page in fifty is counted."""
    c, kind = case, case["kind"]
    esz = 4 if c["dtype"] == "f32" else 2
    hq, hkv, p = c["q_heads"], c["kv_heads"], c["page"]
    tok = sum(_lens(c))
    pages = sum(-(-n // p) for n in _lens(c))
    if kind == "build":
        return {"bytes": tok * hkv * D * esz + pages * hkv * 4 * D * esz, "flops": 6 * tok * hkv * D}
    v_rows = 32 * c["batch"] * hq * D * esz
    if kind == "dense":
        return {"bytes": tok * hkv * D * esz + v_rows, "flops": 2 * tok * hq * D}
    stat = 2 * D * (1 if kind in ("topk8", "group8") else esz)
    lists = hkv if kind in ("group", "group8") else hq
    sel = sum(min(_k_pages(c), -(-n // p)) for n in _lens(c))
    if kind == "gauss":
        sel = pages / 50
    if kind == "refine":                        # K of a KV head at most once, however many of its heads ask for it
        lists, sel = hkv, pages
    values = 2 if kind == "softmax" else 1      # softmax needs V of every selected token
    score = 4 * (hkv if kind in ("group", "group8") else hq) * (2 if kind == "gauss" else 1)
    return {"bytes": pages * (hkv * stat + score) + values * sel * lists * p * D * esz + v_rows,
            "flops": 4 * pages * hq * D + 2 * sel * hq * p * D * values}


def tolerance(case):
    """Four times the distance from exact() that these sizes show: 7e-7 in outputs and scores (32-bit sums), and in
    16-bit stored means and variances 8e-6 (a step's one page) to 1.5e-5 (all pages), from values that lie on a
    rounding boundary of the stored type and move by its last place, 1/256 of themselves."""
    if case["dtype"] == "f32" or case["kind"] == "dense":
        return {"rel": 3e-6, "max": 2e-4, "differ": 0.01}
    return {"rel": 6e-5 if case["kind"] == "build" else 3e-5, "max": 8e-3, "differ": 0.01}


# ---- inputs -------------------------------------------------------------------------------------------------------
def _inputs(c, seed):
    w = synth.Workload("case", c["batch"], c["q_heads"], c["kv_heads"], D, c["tokens"], c["page"], c["dtype"],
                       alpha=c["alpha"], scale=_scale(c), n_planted=c["planted"], planted_spans=c["spans"],
                       n_outlier_channels=c["outliers"])
    inp = synth.make_inputs(w, seed, device="cuda")
    inp["seq_lens"] = torch.tensor(_lens(c), dtype=torch.int32, device="cuda")
    return inp


def _head(inp, b, h):
    """K or V of a sequence's KV head in token order: a function of the pool."""
    rows = inp["block_table"][b].long()
    return lambda pool: pool[rows, h]           # [pages, page, D]


def _moments(k, dt):
    """Stored statistics of pages k [.., tokens, D]: (min, max), (mean, variance), in the cache's type."""
    k = k.double()
    mean = k.mean(-2)
    var = (k - mean.unsqueeze(-2)).square().mean(-2)
    return (torch.stack((k.amin(-2), k.amax(-2)), -2).to(dt), torch.stack((mean, var), -2).to(dt))


def _statistics(c, inp):
    """Statistics of whole pages (what ran before left them so; the step's append brings the last page up to date)."""
    dt = inp["k_pool"].dtype
    b_, h_, m = c["batch"], c["kv_heads"], _pages(c)
    box = torch.empty(b_, h_, m, 2, D, device="cuda", dtype=dt)
    gauss = torch.empty_like(box)
    for b in range(b_):
        for h in range(h_):
            k = _head(inp, b, h)(inp["k_pool"])
            for lo in range(0, m, 8192):
                box[b, h, lo:lo + 8192], gauss[b, h, lo:lo + 8192] = _moments(k[lo:lo + 8192], dt)
    return box, gauss


def _e4m3_outward(x, up):
    """Codes of the 8-bit format's neighbour of x that is not below it (up) or not above it."""
    code = x.float().to(torch.float8_e4m3fn)
    v, code = code.float(), code.view(torch.uint8).to(torch.int16)
    off = (v < x.float()) if up else (v > x.float())
    away = (v > 0) | ((v == 0) & bool(up))     # the step goes towards larger values (up) or smaller ones
    if up:
        new = torch.where(away, torch.where(v == 0, torch.ones_like(code), code + 1), torch.where(v == -2.0 ** -9, torch.zeros_like(code), code - 1))
    else:
        new = torch.where(v > 0, code - 1, torch.where(v == 0, torch.full_like(code, 0x81), code + 1))
    return torch.where(off, new, code).to(torch.uint8)


def _box8(box):
    """8-bit bounds [.., D/8, 2, 8] of bounds [.., 2, D], rounded outward."""
    lo, hi = _e4m3_outward(box[..., 0, :], False), _e4m3_outward(box[..., 1, :], True)
    return torch.stack((lo.unflatten(-1, (D // 8, 8)), hi.unflatten(-1, (D // 8, 8))), -2).contiguous()


def prepare(case, seed):
    c, kind = case, case["kind"]
    inp = _inputs(c, seed)
    b_, hq, hkv, m, cap, p = c["batch"], c["q_heads"], c["kv_heads"], _pages(c), _cap(c), c["page"]
    f32, i32 = dict(device="cuda", dtype=torch.float32), dict(device="cuda", dtype=torch.int32)
    s = dict(inp, case=c, kind=kind, k=_k_pages(c))
    s["cfg"] = ekv.make_config(b_, hq, hkv, D, p, c["dtype"], c["alpha"], _scale(c), m, cap)
    s["cache"] = ekv.cache_view(inp["k_pool"], inp["v_pool"], inp["block_table"], inp["seq_lens"])
    if kind == "build":
        s["box_stats"] = torch.zeros(b_, hkv, m, 2, D, device="cuda", dtype=inp["k_pool"].dtype)
        s["gauss_stats"] = torch.zeros_like(s["box_stats"])
        s["stats"] = ekv.stats_view(s["box_stats"], s["gauss_stats"])
        return s

    def room(op, cfg=None):
        return torch.empty(max(256, ekv.ekv_workspace_bytes(cfg or s["cfg"], op)), device="cuda", dtype=torch.uint8)

    s["out"], s["tau"], s["supp"] = torch.zeros(b_, hq, D, **f32), torch.zeros(b_, hq, **f32), torch.zeros(b_, hq, **i32)
    if kind == "dense":
        s["ws_decode"] = room(ekv.EKV_OP_DECODE_FULL)
        return s
    s["box_stats"], s["gauss_stats"] = _statistics(c, inp)
    if kind in ("topk8", "group8"):
        s["box8_stats"] = _box8(s["box_stats"])
    s["stats"] = ekv.stats_view(s["box_stats"], s["gauss_stats"], s.get("box8_stats"))
    # the step's token: its slot is empty until the step appends it
    before = inp["seq_lens"] - 1
    s["before"] = before
    s["cache_before"] = ekv.cache_view(inp["k_pool"], inp["v_pool"], inp["block_table"], before)
    rows = inp["block_table"].long().gather(1, (before.long() // p)[:, None])[:, 0]
    slot = before.long() % p
    for new, pool in (("k_new", "k_pool"), ("v_new", "v_pool")):
        s[new] = inp[pool][rows, :, slot].contiguous()
        inp[pool][rows, :, slot] = 0
    lists = hkv if kind in ("group", "group8") else hq
    s["scfg"] = s["cfg"] if lists == hq else ekv.make_config(b_, hkv, hkv, D, p, c["dtype"], c["alpha"], _scale(c), m, cap)
    s["page_idx"], s["n_sel"] = torch.zeros(b_, lists, cap, **i32), torch.zeros(b_, lists, **i32)
    if kind == "gauss":
        s["mu"], s["sigma"] = torch.zeros(b_, hq, m, **f32), torch.zeros(b_, hq, m, **f32)
        s["tau_hat"], s["overflow"] = torch.zeros(b_, hq, **f32), torch.zeros(b_, hq, **i32)
        s["ws_select"] = room(ekv.EKV_OP_SELECT_GAUSS)
    else:
        s["box"] = torch.zeros(b_, lists, m, **f32)
        s["ws_select"] = room(ekv.EKV_OP_SELECT_TOPK, s["scfg"])
    s["ws_decode"] = room(ekv.EKV_OP_DECODE_SPARSE_SOFTMAX if kind == "softmax" else ekv.EKV_OP_DECODE_SPARSE)
    if kind == "softmax":
        s["lse"] = torch.zeros(b_, hq, **f32)
    if kind == "refine":
        s["n_added"], s["overflow"] = torch.zeros(b_, hq, **i32), torch.zeros(b_, hq, **i32)
        s["ws_refine"] = room(ekv.EKV_OP_SELECT_BOX_THRESHOLD)
    return s


# ---- one pass -----------------------------------------------------------------------------------------------------
def run(s):
    """Counts that a change of the last bit of a score moves by one (support tokens of a flat attention, pages at a
    threshold) are not among the outputs; tau and the output show what they stand for."""
    kind = s["kind"]
    if kind == "build":
        ekv.ekv_stats_build(s["cfg"], s["cache"], s["stats"])
        return {"box_stats": s["box_stats"], "gauss_stats": s["gauss_stats"]}
    got = {"out": s["out"]}
    if kind != "softmax":
        got["tau"] = s["tau"]
        if s["case"]["flat"] == 1.0 and s["case"]["alpha"] >= 1.5:
            got["supp"] = s["supp"]
    if kind == "dense":
        ekv.ekv_decode_full(s["cfg"], s["q"], s["cache"], s["out"], s["tau"], s["supp"], s["ws_decode"])
        return got
    got["box_stats"], got["gauss_stats"] = s["box_stats"], s["gauss_stats"]
    if kind == "gauss":
        ekv.ekv_append_score_pages(s["cfg"], s["cache_before"], s["stats"], s["k_new"], s["v_new"], s["q"],
                                   ekv.EKV_SCORE_GAUSS, mu=s["mu"], sigma=s["sigma"])
        ekv.ekv_select_gauss(s["cfg"], s["mu"], s["sigma"], s["seq_lens"], 0.99, 0.0, s["tau_hat"], s["page_idx"],
                             s["n_sel"], s["overflow"], s["ws_select"])
        ekv.ekv_decode_sparse(s["cfg"], s["q"], s["cache"], s["page_idx"], s["n_sel"], s["out"], s["tau"], s["supp"],
                              s["ws_decode"])
        return dict(got, mu=s["mu"], sigma=s["sigma"], tau_hat=s["tau_hat"])
    mode = ekv.EKV_SCORE_BOX8 if kind in ("topk8", "group8") else ekv.EKV_SCORE_BOX
    if kind in ("group", "group8"):
        mode |= ekv.EKV_SCORE_GROUP_MAX
    ekv.ekv_append_score_pages(s["cfg"], s["cache_before"], s["stats"], s["k_new"], s["v_new"], s["q"], mode, box=s["box"])
    ekv.ekv_select_topk(s["scfg"], s["box"], s["seq_lens"], s["k"], s["page_idx"], s["n_sel"], s["ws_select"])
    got["box"] = s["box"]
    if kind == "softmax":
        ekv.ekv_decode_sparse_softmax(s["cfg"], s["q"], s["cache"], s["page_idx"], s["n_sel"], s["out"], s["lse"],
                                      s["ws_decode"])
        return dict(got, lse=s["lse"], n_sel=s["n_sel"])
    decode = ekv.ekv_decode_sparse_group if kind in ("group", "group8") else ekv.ekv_decode_sparse
    decode(s["cfg"], s["q"], s["cache"], s["page_idx"], s["n_sel"], s["out"], s["tau"], s["supp"], s["ws_decode"])
    if kind == "refine":
        ekv.ekv_select_box_threshold(s["cfg"], s["box"], s["seq_lens"], s["tau"], s["page_idx"], s["n_sel"], s["page_idx"],
                                     s["n_sel"], s["n_added"], s["overflow"], s["ws_refine"])
        ekv.ekv_decode_sparse(s["cfg"], s["q"], s["cache"], s["page_idx"], s["n_sel"], s["out"], s["tau"], s["supp"],
                              s["ws_decode"])
    else:
        got["n_sel"] = s["n_sel"]
    return got


# ---- the same in 64 bits ------------------------------------------------------------------------------------------
def _entmax(z, keep, beta):
    """tau [G] and weights [G, n] of entmax over the kept entries of z [G, n] (z = (alpha - 1) * score)."""
    z = z.masked_fill(~keep, -math.inf)
    hi = z.amax(1)
    lo = hi - 1.0
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        over = (z - mid[:, None]).clamp_min(0).pow(beta).sum(1) >= 1.0
        lo, hi = torch.where(over, mid, lo), torch.where(over, hi, mid)
    return lo, (z - lo[:, None]).clamp_min(0).pow(beta)


def _gauss_tau(mu, sigma, cnt, a, beta):
    """Root of sum_p cnt_p E[(a S_p - tau)_+^beta] = 1 with S_p ~ N(mu_p, sigma_p^2), per row of mu [G, M]."""
    m, s = a * mu, a * sigma
    lo, hi = m.amax(1) - 1.0, (m + 40.0 * s).amax(1) + 1.0
    for _ in range(80):
        mid = 0.5 * (lo + hi)
        y = m - mid[:, None]
        t = (y / s.clamp_min(1e-300)).clamp(-38.0, 1e30)
        h0 = torch.special.ndtr(t)
        h1 = t * h0 + torch.exp(-0.5 * t * t) / math.sqrt(2 * math.pi)
        for n in range(2, beta + 1):
            h0, h1 = h1, (t * h1 + (n - 1) * h0).clamp_min(0)
        f = torch.where(s > 0, s.pow(beta) * h1, y.clamp_min(0).pow(beta))
        over = (f * cnt).sum(1) >= 1.0
        lo, hi = torch.where(over, mid, lo), torch.where(over, hi, mid)
    return lo


def _largest(x, k):
    """Mask of the k largest entries of each row, lower index first among equals."""
    at = torch.sort(x, dim=1, descending=True, stable=True).indices[:, :k]
    return torch.zeros_like(x, dtype=torch.bool).scatter_(1, at, True)


def exact(case, seed):
    c, kind = case, case["kind"]
    inp = _inputs(c, seed)
    dt, p, m_all = inp["k_pool"].dtype, c["page"], _pages(c)
    b_, hq, hkv = c["batch"], c["q_heads"], c["kv_heads"]
    g_, a, scale = hq // hkv, c["alpha"] - 1.0, _scale(c)
    beta = 1.0 / a
    f64 = dict(device="cuda", dtype=torch.float64)
    if kind == "build":
        box, gauss = torch.zeros(b_, hkv, m_all, 2, D, device="cuda", dtype=dt), torch.zeros(b_, hkv, m_all, 2, D, device="cuda", dtype=dt)
    elif kind in APPENDING:
        box, gauss = _statistics(c, inp)
    got = {"out": torch.zeros(b_, hq, D, **f64), "tau": torch.zeros(b_, hq, **f64), "lse": torch.zeros(b_, hq, **f64),
           "tau_hat": torch.zeros(b_, hq, **f64), "mu": torch.full((b_, hq, m_all), -math.inf, **f64),
           "sigma": torch.zeros(b_, hq, m_all, **f64),
           "box": torch.full((b_, hkv if kind in ("group", "group8") else hq, m_all), -math.inf, **f64)}
    for b, n in enumerate(_lens(c)):
        m, last = -(-n // p), n - (-(-n // p) - 1) * p
        cnt = torch.full((m,), p, **f64)
        cnt[-1] = last
        for h in range(hkv):
            head = _head(inp, b, h)
            k = head(inp["k_pool"])
            if kind == "build":
                for lo in range(0, m, 8192):
                    hi = min(m, lo + 8192)
                    box[b, h, lo:hi], gauss[b, h, lo:hi] = _moments(k[lo:hi], dt)
            if kind != "dense":
                box[b, h, m - 1], gauss[b, h, m - 1] = _moments(k[m - 1, :last], dt)
            if kind == "build":
                continue
            q = inp["q"][b, h * g_:(h + 1) * g_].double()
            heads = slice(h * g_, (h + 1) * g_)
            z = torch.empty(g_, n, **f64)
            flat_k = k.reshape(-1, D)[:n]
            for lo in range(0, n, 1 << 18):
                z[:, lo:lo + (1 << 18)] = a * scale * (q @ flat_k[lo:lo + (1 << 18)].double().t().contiguous())
            keep = torch.ones(g_, m, device="cuda", dtype=torch.bool)
            if kind == "gauss":
                mean, var = gauss[b, h, :m, 0].double(), gauss[b, h, :m, 1].double()
                mu = scale * (q @ mean.t().contiguous())
                sigma = scale * (q.square() @ var.t().contiguous()).sqrt()
                tau_hat = _gauss_tau(mu, sigma, cnt, a, round(beta))
                est = a * (mu + sigma * torch.special.ndtri(0.99 ** (1.0 / cnt)))
                keep = est > tau_hat[:, None]
                keep |= _largest(est, 1) & ~keep.any(1, keepdim=True)
                keep &= _largest(est, _cap(c))
                got["mu"][b, heads, :m], got["sigma"][b, heads, :m], got["tau_hat"][b, heads] = mu, sigma, tau_hat
            elif kind != "dense":
                bounds = box[b, h, :m]
                if kind in ("topk8", "group8"):
                    u = _box8(bounds)
                    bounds = torch.stack((u[:, :, 0].reshape(m, D), u[:, :, 1].reshape(m, D)), 1).view(torch.float8_e4m3fn)
                    bounds = bounds.float()
                bounds = bounds.double()
                score = scale * (q.clamp_max(0) @ bounds[:, 0].t().contiguous() + q.clamp_min(0) @ bounds[:, 1].t().contiguous())
                if kind in ("group", "group8"):
                    top = score.amax(0, keepdim=True)
                    got["box"][b, h, :m] = top[0]
                    keep = _largest(top, _k_pages(c)).expand(g_, m)
                else:
                    got["box"][b, heads, :m] = score
                    keep = _largest(score, _k_pages(c))
            v = head(inp["v_pool"]).reshape(-1, D)[:n]
            if kind == "refine":
                first, _ = _entmax(z, keep.repeat_interleave(p, 1)[:, :n], beta)
                keep = keep | (a * score > first[:, None])
            tokens = keep.repeat_interleave(p, 1)[:, :n]
            if kind == "softmax":
                s = (z / a).masked_fill(~tokens, -math.inf)
                got["lse"][b, heads] = torch.logsumexp(s, 1)
                weight = torch.softmax(s, 1)
            else:
                got["tau"][b, heads], weight = _entmax(z, tokens, beta)
            for lo in range(0, n, 1 << 18):
                got["out"][b, heads] += weight[:, lo:lo + (1 << 18)].contiguous() @ v[lo:lo + (1 << 18)].double()
    wanted = {"build": (), "dense": ("out", "tau"), "gauss": ("out", "tau", "mu", "sigma", "tau_hat"),
              "softmax": ("out", "lse", "box")}.get(kind, ("out", "tau", "box"))
    got = {k: got[k] for k in wanted}
    if kind != "dense":
        got["box_stats"], got["gauss_stats"] = box.double(), gauss.double()
    return got
