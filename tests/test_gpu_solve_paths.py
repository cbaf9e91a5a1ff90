"""The end of the entmax decode (threshold, support, value sum) at the sizes where its branches meet: one group of
scores, a wavefront's 512 and 1024 group maxima and one more of each, groups of fewer than 64 tokens, a partial last
group, and candidate lists of a lane's one entry, its four, the wavefronts' segments and beyond them.

Results against the float64 oracle under the rules of tests/helpers.py (tau 4e-6, output 1e-5 / 2e-3, support exact up
to tokens within float32 resolution of tau)."""
import math

import numpy as np
import pytest
import torch

from oracle import entmaxkv_oracle as orc
from paper_2605_21649_amd import binding as ekv
from paper_2605_21649_amd import synth
from tests.helpers import DeviceState, unit_kv, check_decode_unit, pre_groups

pytestmark = pytest.mark.gpu

# tokens, page, dtype, score scale (times 1/sqrt(128)), alpha
CASES = [(1, 16, "bf16", 1.0, 1.5), (4, 4, "f32", 1.0, 2.0), (61, 16, "f32", 1.0, 1.5),
         (512 * 64, 16, "bf16", 1.0, 1.5), (512 * 64 + 1, 16, "bf16", 1.0, 1.25),
         (1024 * 64 - 15, 32, "bf16", 0.5, 1.5), (1024 * 64 + 1, 64, "bf16", 1.0, 2.0),
         (513 * 60 - 7, 12, "bf16", 0.5, 4.0 / 3.0), (1025 * 48 - 3, 48, "bf16", 1.0, 1.5),
         # candidates after the bound: a few hundred, a few thousand (segments), more than the segments hold
         (20000, 16, "f32", 0.3, 1.5), (40000, 8, "f32", 0.1, 1.25), (30000, 16, "f32", 0.05, 1.5),
         (40000, 16, "f32", 0.01, 2.0), (70000, 16, "f32", 0.15, 1.7), (3000, 20, "f32", 0.6, 3.0), (70000, 16, "f32", 0.1, 2.5)]


@pytest.mark.parametrize("tokens,page,dtype,scale,alpha", CASES)
def test_solve_at_the_edges_of_its_paths(tokens, page, dtype, scale, alpha):
    w = synth.Workload("edge", 1, 2, 1, 128, tokens, page, dtype, alpha=alpha, scale=scale / math.sqrt(128.0))
    inp = synth.make_inputs(w, 77 + tokens, device="cpu")
    st = DeviceState(w, inp)
    toks = torch.full((1, 2, 65536), -1, device="cuda", dtype=torch.int32)
    ex = ekv.decode_extras(support_tokens=toks)
    ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), st.out, st.tau, st.supp, st.workspace(ekv.EKV_OP_DECODE_FULL),
                        extras=ex)
    dense = [x.clone() for x in (st.out, st.tau, st.supp, toks)]
    # the same pages as lists: the sparse decode of every page is the dense one, bit for bit
    st.page_idx.copy_(torch.arange(st.cap, device="cuda", dtype=torch.int32).expand(1, 2, st.cap))
    st.n_sel.fill_(st.cap)
    toks.fill_(-1)
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                          st.workspace(ekv.EKV_OP_DECODE_SPARSE), extras=ex)
    torch.cuda.synchronize()
    for a, b in zip(dense, (st.out, st.tau, st.supp, toks)):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    for hq in range(2):
        q, K, V = unit_kv(inp, w, 0, hq)
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        check_decode_unit(w, st.out[0, hq].cpu().numpy(), float(st.tau[0, hq]), int(st.supp[0, hq]),
                          toks[0, hq].cpu().numpy(), ref, boundary_expected=True)


@pytest.mark.parametrize("lens", [(1, 64, 0), (2048, 1, 700)])
def test_solve_side_outputs_of_short_and_flat_rows(lens):
    """Mass and count above a reference threshold and the log-sum-exp cover all candidates, whichever path a row took."""
    for scale in (1.0, 0.05):
        w = synth.Workload("edge", 3, 2, 1, 128, 2048, 16, "f32", scale=scale / math.sqrt(128.0))
        inp = synth.make_inputs(w, 5, device="cpu")
        inp["seq_lens"] = torch.tensor(lens, dtype=torch.int32)
        st = DeviceState(w, inp)
        f = dict(device="cuda", dtype=torch.float32)
        lse, mass, cnt = torch.zeros(3, 2, **f), torch.zeros(3, 2, **f), torch.zeros(3, 2, device="cuda", dtype=torch.int32)
        refs = {}
        for b in range(3):
            for hq in range(2):
                if lens[b]:
                    q, K, V = unit_kv(inp, w, b, hq)
                    refs[b, hq] = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        tau_ref = torch.zeros(3, 2, **f)
        for (b, hq), r in refs.items():
            tau_ref[b, hq] = r["tau"] - 0.01
        ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), st.out, st.tau, st.supp, st.workspace(ekv.EKV_OP_DECODE_FULL),
                            extras=ekv.decode_extras(tau_ref=tau_ref, kept_mass_ref=mass, kept_supp_ref=cnt, lse=lse))
        torch.cuda.synchronize()
        for b in range(3):
            for hq in range(2):
                if not lens[b]:
                    assert torch.isposinf(st.tau[b, hq]) and not st.out[b, hq].any() and int(st.supp[b, hq]) == 0
                    assert torch.isneginf(lse[b, hq]) and float(mass[b, hq]) == 0 and int(cnt[b, hq]) == 0
                    continue
                r = refs[b, hq]
                check_decode_unit(w, st.out[b, hq].cpu().numpy(), float(st.tau[b, hq]), int(st.supp[b, hq]), None, r,
                                  boundary_expected=True)
                z, t = (w.alpha - 1.0) * r["s"], float(tau_ref[b, hq])
                assert abs(float(lse[b, hq]) - (r["s"].max() + np.log(np.exp(r["s"] - r["s"].max()).sum()))) < 1e-5 * 10
                over = np.clip(z - t, 0, None)
                assert abs(float(mass[b, hq]) - (over ** 2).sum()) < 1e-4
                assert abs(int(cnt[b, hq]) - int((over > 0).sum())) <= int((np.abs(z - t) < 2e-6).sum())


# batch, query heads, KV heads, page, dtype, pages per list: lists at the edges of the one-launch decode (a workgroup of
# sixteen wavefronts, of four, and the two-launch path just beyond), page sizes of both score paths
LISTS = [(1, 4, 2, 16, "bf16", 128), (1, 4, 2, 16, "bf16", 129), (1, 4, 2, 4, "f32", 256), (1, 4, 2, 36, "f32", 28),
         (3, 32, 8, 36, "bf16", 113), (3, 32, 8, 32, "bf16", 128), (3, 32, 8, 64, "bf16", 64), (9, 32, 8, 12, "bf16", 85),
         (9, 32, 8, 64, "bf16", 32), (9, 32, 8, 16, "bf16", 64), (9, 32, 32, 4, "f32", 512), (9, 32, 8, 16, "f32", 1),
         (8, 32, 8, 64, "bf16", 64), (8, 32, 8, 64, "bf16", 65),
         (5, 8, 2, 16, "bf16", 64)]                                                  # rows left over from whole rounds of the XCDs


@pytest.mark.parametrize("batch,hq,hkv,page,dtype,k", LISTS)
@pytest.mark.parametrize("scale", [1.0, 0.05])
def test_short_lists_in_one_launch(batch, hq, hkv, page, dtype, k, scale):
    """Ragged lists (one empty, one full) against the oracle, and, bit for bit, against the same lists in buffers so much
    longer that they go through the two-launch path; the flat scale leaves most of a list in the support."""
    n_pages = 2 * k + 3
    w = synth.Workload("lists", batch, hq, hkv, 128, n_pages * page, page, dtype, scale=scale / math.sqrt(128.0))
    inp = synth.make_inputs(w, 9 + k, device="cpu")
    inp["seq_lens"] = inp["seq_lens"] - torch.arange(batch, dtype=torch.int32) * 3
    rng = np.random.default_rng(k)
    lens = rng.integers(1, k + 1, size=(batch, hq))
    lens[0, 0], lens[0, 1], lens[-1, -1] = k, 0, max(1, k - 1)
    pages = [[np.sort(rng.choice(n_pages - 1, lens[b, h], replace=False)) for h in range(hq)] for b in range(batch)]
    got = []
    wide = w.scaled(context=max(w.context, 20000))                          # room for a capacity beyond the short lists'
    for ww, cap in ((w, k), (wide, wide.pages_per_seq)):
        big = dict(inp, block_table=torch.nn.functional.pad(inp["block_table"], (0, ww.pages_per_seq - w.pages_per_seq)))
        st = DeviceState(ww, big, cap=cap)
        for b in range(batch):
            for h in range(hq):
                st.page_idx[b, h, :lens[b, h]] = torch.from_numpy(pages[b][h].astype(np.int32)).to(st.page_idx.device)
        st.n_sel.copy_(torch.from_numpy(lens.astype(np.int32)))
        toks = torch.full((batch, hq, 4096), -1, device="cuda", dtype=torch.int32)
        tau_ref = torch.full_like(st.tau, 0.5)
        mass, cnt = torch.zeros_like(st.tau), torch.zeros_like(st.supp)
        for extras in (ekv.decode_extras(support_tokens=toks), ekv.decode_extras(tau_ref=tau_ref, kept_mass_ref=mass, kept_supp_ref=cnt)):
            ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                                  st.workspace(ekv.EKV_OP_DECODE_SPARSE), extras=extras)
        torch.cuda.synchronize()
        got.append([x.cpu() for x in (st.out, st.tau, st.supp, toks, cnt)])
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    out, tau, supp, toks, _ = [x.numpy() for x in got[0]]
    assert supp[0, 1] == 0 and np.isposinf(tau[0, 1]) and not out[0, 1].any()
    for b, h in ((0, 0), (batch - 1, hq - 1), (batch // 2, hq // 2)):
        q, K, V = unit_kv(inp, w, b, h)
        tok = orc.pages_to_tokens(pages[b][h], page, K.shape[0])
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale, tok)
        check_decode_unit(w, out[b, h], float(tau[b, h]), int(supp[b, h]), toks[b, h], ref, boundary_expected=True)


# batch, query heads, KV heads, page, dtype, pages per list: more rows than compute units, to twice as many and beyond,
# lists of up to 1024 and 2048 tokens, groups of 64, 60, 48 and 36 tokens
GROUPED = [(9, 64, 8, 16, "bf16", 64), (9, 64, 8, 16, "bf16", 128), (9, 32, 8, 12, "bf16", 170), (9, 64, 8, 24, "bf16", 85),
           (9, 64, 16, 36, "f32", 56), (17, 32, 8, 64, "bf16", 32), (67, 8, 2, 16, "bf16", 32), (1, 32, 8, 16, "bf16", 128), (5, 32, 8, 16, "bf16", 256),
           # lists beyond the one launch: the last number of units that is split over the XCDs, and the next
           (12, 128, 16, 16, "bf16", 136), (25, 64, 8, 16, "bf16", 136), (25, 64, 8, 8, "f32", 260)]


@pytest.mark.parametrize("batch,hq,hkv,page,dtype,k", GROUPED)
@pytest.mark.parametrize("scale", [1.0, 0.3, 0.05])
def test_group_lists_and_the_same_lists_per_head_agree_bit_for_bit(batch, hq, hkv, page, dtype, k, scale):
    """A list per KV head gives every head of the group what the same list gives it as its own, side outputs included,
    however many rows the call has and however flat they are."""
    n_pages = 2 * k + 3
    w = synth.Workload("grouped", batch, hq, hkv, 128, n_pages * page, page, dtype, scale=scale / math.sqrt(128.0))
    inp = synth.make_inputs(w, 21 + k, device="cuda")
    inp["seq_lens"] = inp["seq_lens"] - torch.arange(batch, dtype=torch.int32, device="cuda") * 3
    rng = np.random.default_rng(k)
    lens = rng.integers(1, k + 1, size=(batch, hkv))
    lens[0, 0], lens[0, 1], lens[-1, -1] = k, 0, max(1, k - 1)
    lists = np.zeros((batch, hkv, k), dtype=np.int32)
    for b in range(batch):
        for h in range(hkv):
            lists[b, h, :lens[b, h]] = np.sort(rng.choice(n_pages - 1, lens[b, h], replace=False))
    lists, counts = torch.from_numpy(lists).cuda(), torch.from_numpy(lens.astype(np.int32)).cuda()
    st = DeviceState(w, inp, cap=k)
    ws = st.workspace(ekv.EKV_OP_DECODE_SPARSE)
    g = hq // hkv
    got = []
    for decode, idx, n in ((ekv.ekv_decode_sparse_group, lists, counts),
                           (ekv.ekv_decode_sparse, lists.repeat_interleave(g, 1).contiguous(), counts.repeat_interleave(g, 1).contiguous())):
        toks = torch.full((batch, hq, 2 * page * k), -1, device="cuda", dtype=torch.int32)
        mass, cnt, evals = torch.zeros_like(st.tau), torch.zeros_like(st.supp), torch.zeros_like(st.supp)
        decode(st.cfg, st.inp["q"], st.cache(), idx, n, st.out, st.tau, st.supp, ws,
               extras=ekv.decode_extras(support_tokens=toks, solve_evals=evals))
        plain = [x.clone() for x in (st.out, st.tau, st.supp, toks, evals)]
        decode(st.cfg, st.inp["q"], st.cache(), idx, n, st.out, st.tau, st.supp, ws,
               extras=ekv.decode_extras(tau_ref=plain[1] - 0.01, kept_mass_ref=mass, kept_supp_ref=cnt, tau_seed=plain[1] - 0.001))
        got.append(plain + [x.clone() for x in (st.out, st.tau, st.supp, mass, cnt)])
    torch.cuda.synchronize()
    names = ("out", "tau", "support size", "support", "evaluations", "seeded out", "seeded tau", "seeded support size", "mass", "count")
    assert not [n for n, a, b in zip(names, *got) if not torch.equal(a.view(torch.uint8), b.view(torch.uint8))]
    out, tau, supp, toks, _, out2, tau2, supp2, mass, cnt = [x.cpu().numpy() for x in got[0]]
    assert not out[0, g].any() and np.isposinf(tau[0, g]) and supp[0, g] == 0
    inp = {key: x.cpu() for key, x in inp.items()}
    for b, h in ((0, 0), (batch - 1, hq - 1)):
        q, K, V = unit_kv(inp, w, b, h)
        tok = orc.pages_to_tokens(lists[b, h // g, :lens[b, h // g]].cpu().numpy(), page, K.shape[0])
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale, tok)
        check_decode_unit(w, out[b, h], float(tau[b, h]), int(supp[b, h]), toks[b, h], ref, boundary_expected=True)
        check_decode_unit(w, out2[b, h], float(tau2[b, h]), int(supp2[b, h]), None, ref, boundary_expected=True)
        z = (w.alpha - 1.0) * ref["s"]
        over = np.clip(z - float(np.float32(tau[b, h]) - np.float32(0.01)), 0, None)
        assert abs(float(mass[b, h]) - (over ** 2).sum()) < 1e-4
        assert abs(int(cnt[b, h]) - int((over > 0).sum())) <= int((np.abs(z - tau[b, h] + 0.01) < 4e-6).sum())


@pytest.mark.parametrize("tokens,page,scale", [(4000, 16, 1.0), (4000, 16, 0.05), (192 * 64, 16, 0.05), (192 * 64 + 1, 16, 0.05),
                                               (16384, 16, 1.0), (16384, 32, 0.05),
                                               (16385, 16, 1.0), (1024 * 64, 64, 1.0), (20000, 32, 0.03),
                                               (1024 * 64 + 80, 16, 1.0), (1024 * 64 + 80, 16, 0.1), (70000, 12, 0.04)])
def test_more_rows_than_compute_units(tokens, page, scale):
    """288 rows (36 sequences over one shared set of pages, every length different): up to 192 groups a row is solved by
    four wavefronts, beyond by sixteen, and rows too flat for their LDS lists continue in the workspace.  Sampled rows against the oracle;
    dense and the same pages as lists agree bit for bit, and rows whose candidates fit all variants' segments with the same
    sequence decoded alone."""
    B, Hq = 36, 8
    one = synth.Workload("rows", 1, Hq, 1, 128, tokens, page, "bf16", scale=scale / math.sqrt(128.0))
    inp = synth.make_inputs(one, 3 + tokens, device="cpu")
    w = one.scaled(batch=B)
    g = torch.Generator().manual_seed(tokens)
    inp["q"] = torch.randn(B, Hq, 128, generator=g).to(torch.bfloat16)
    inp["block_table"] = inp["block_table"].expand(B, -1).contiguous()
    inp["seq_lens"] = torch.tensor([tokens - 7 * b for b in range(B)], dtype=torch.int32)
    st = DeviceState(w, inp)
    toks = torch.full((B, Hq, 32768), -1, device="cuda", dtype=torch.int32)
    ex = ekv.decode_extras(support_tokens=toks)
    ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), st.out, st.tau, st.supp, st.workspace(ekv.EKV_OP_DECODE_FULL), extras=ex)
    dense = [x.clone() for x in (st.out, st.tau, st.supp, toks)]
    st.page_idx.copy_(torch.arange(st.cap, device="cuda", dtype=torch.int32).expand(B, Hq, st.cap))
    st.n_sel.copy_(((st.inp["seq_lens"] + page - 1) // page)[:, None].expand(B, Hq))
    toks.fill_(-1)
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                          st.workspace(ekv.EKV_OP_DECODE_SPARSE), extras=ex)
    torch.cuda.synchronize()
    for a, b in zip(dense, (st.out, st.tau, st.supp, toks)):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    for b, h in ((0, 0), (17, 5), (35, 7)):
        q, K, V = unit_kv(inp, w, b, h)
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        check_decode_unit(w, st.out[b, h].cpu().numpy(), float(st.tau[b, h]), int(st.supp[b, h]), toks[b, h].cpu().numpy(),
                          ref, boundary_expected=True)
    if scale == 1.0:
        alone = DeviceState(one, dict(inp, q=inp["q"][17:18], block_table=inp["block_table"][17:18], seq_lens=inp["seq_lens"][17:18]))
        ekv.ekv_decode_full(alone.cfg, alone.inp["q"], alone.cache(), alone.out, alone.tau, alone.supp,
                            alone.workspace(ekv.EKV_OP_DECODE_FULL))
        torch.cuda.synchronize()
        for a, b in zip((alone.out, alone.tau, alone.supp), (st.out, st.tau, st.supp)):
            assert torch.equal(a[0].view(torch.uint8), b[17].view(torch.uint8))


@pytest.mark.parametrize("tokens,scale", [(4096 * 64 + 1, 1.0), (16384 * 64 - 30, 1.0), (16384 * 64 + 1, 1.0), (16384 * 64 + 1, 0.05)])
def test_long_rows_at_the_ends_of_the_group_bound(tokens, scale):
    """Rows of more than four maxima per thread, of sixteen, and one more group (which takes the filter passes, dense and as
    a list); the flat one hands thousands of candidates over through them."""
    w = synth.Workload("long", 1, 2, 1, 128, tokens, 16, "bf16", scale=scale / math.sqrt(128.0))
    inp = synth.make_inputs(w, tokens, device="cpu")
    st = DeviceState(w, inp)
    toks = torch.full((1, 2, 65536), -1, device="cuda", dtype=torch.int32)
    ex = ekv.decode_extras(support_tokens=toks)
    ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), st.out, st.tau, st.supp, st.workspace(ekv.EKV_OP_DECODE_FULL), extras=ex)
    dense = [x.clone() for x in (st.out, st.tau, st.supp, toks)]
    st.page_idx.copy_(torch.arange(st.cap, device="cuda", dtype=torch.int32).expand(1, 2, st.cap))
    st.n_sel.fill_(st.cap)
    toks.fill_(-1)
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                          st.workspace(ekv.EKV_OP_DECODE_SPARSE), extras=ex)
    torch.cuda.synchronize()
    for a, b in zip(dense, (st.out, st.tau, st.supp, toks)):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    q, K, V = unit_kv(inp, w, 0, 1)
    ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
    check_decode_unit(w, st.out[0, 1].cpu().numpy(), float(st.tau[0, 1]), int(st.supp[0, 1]), toks[0, 1].cpu().numpy(), ref,
                      boundary_expected=True)


# page, dtype, alpha, score scale (times 1/sqrt(128)): every group is one page, so the rows are as short as rows of more than
# kPreGroups groups can be; the flattest leaves a slice of the filter more candidates than its list holds
BEYOND = [(36, "f32", 2.0, 1.0), (36, "f32", 1.25, 0.5), (48, "bf16", 1.7, 0.1), (40, "f32", 4.0 / 3.0, 0.3), (36, "f32", 1.5, 0.01)]


@pytest.mark.parametrize("page,dtype,alpha,scale", BEYOND)
def test_filter_passes_beside_short_and_empty_rows(page, dtype, alpha, scale):
    """A row one group beyond the solve's own, an empty one and a short one over the same pages: dense, as lists of every
    page (bit for bit the dense result), and a short list in the long capacity."""
    pages = pre_groups() + 1
    one = synth.Workload("beyond", 1, 2, 1, 128, pages * page, page, dtype, alpha=alpha, scale=scale / math.sqrt(128.0))
    inp = synth.make_inputs(one, page, device="cuda")
    w = one.scaled(batch=3)
    g = torch.Generator(device="cuda").manual_seed(page)
    inp["q"] = torch.randn(3, 2, 128, generator=g, device="cuda").to(inp["k_pool"].dtype)
    inp["block_table"] = inp["block_table"].expand(3, -1).contiguous()
    lens = (pages * page - 5, 0, 7003)
    inp["seq_lens"] = torch.tensor(lens, dtype=torch.int32, device="cuda")
    st = DeviceState(w, inp)
    toks = torch.full((3, 2, pages * page), -1, device="cuda", dtype=torch.int32)
    ex = ekv.decode_extras(support_tokens=toks)
    ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), st.out, st.tau, st.supp, st.workspace(ekv.EKV_OP_DECODE_FULL), extras=ex)
    dense = [x.clone() for x in (st.out, st.tau, st.supp, toks)]
    st.page_idx.copy_(torch.arange(st.cap, device="cuda", dtype=torch.int32).expand(3, 2, st.cap))
    st.n_sel.copy_(((st.inp["seq_lens"] + page - 1) // page)[:, None].expand(3, 2))
    toks.fill_(-1)
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                          st.workspace(ekv.EKV_OP_DECODE_SPARSE), extras=ex)
    torch.cuda.synchronize()
    for a, b in zip(dense, (st.out, st.tau, st.supp, toks)):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    assert torch.isposinf(st.tau[1]).all() and not st.out[1].any() and not st.supp[1].any()
    st.n_sel[0, 1] = 300                                       # sequence 0, head 1: a short list beside a long one
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, st.tau, st.supp,
                          st.workspace(ekv.EKV_OP_DECODE_SPARSE), extras=ex)
    torch.cuda.synchronize()
    assert torch.equal(st.out[0, 0], dense[0][0, 0]) and torch.equal(st.tau[0, 0], dense[1][0, 0])
    inp = {key: x.cpu() for key, x in inp.items()}
    q, K, V = unit_kv(inp, w, 0, 0)
    q1 = unit_kv({**inp, "seq_lens": inp["seq_lens"] * 0}, w, 0, 1)[0]
    cases = [(0, 0, q, K, V), (0, 1, q1, K[:300 * page], V[:300 * page]), (2, 1, *unit_kv(inp, w, 2, 1))]
    for b, h, qq, kk, vv in cases:
        ref = orc.entmax_attention(qq, kk, vv, w.alpha, w.score_scale)
        check_decode_unit(w, st.out[b, h].cpu().numpy(), float(st.tau[b, h]), int(st.supp[b, h]), toks[b, h].cpu().numpy(), ref,
                          boundary_expected=True)
