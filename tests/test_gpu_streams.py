"""Calls large enough to read their streams past the caches (32 MiB of statistics, 128 MiB of K of decodes over all pages and of
builds, 64 MiB of K of lists that a group shares or a head without one has) against the same sequences one by one, which are
small enough not to: bit for bit, since only the kind of the loads differs."""
import pytest
import torch

from paper_2605_21649_amd import binding as ekv
from paper_2605_21649_amd import synth
from tests.helpers import DeviceState

pytestmark = pytest.mark.gpu


def same(a, b):
    return torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))


def alone(w, inp, b, **kw):
    """Sequence b of a batch as a problem of its own, on the same pools."""
    one = {key: (x if key.endswith("pool") else x[b:b + 1].contiguous()) for key, x in inp.items()}
    return DeviceState(w.scaled(batch=1), one, **kw)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("heads", [(8, 8), (16, 8), (32, 8), (64, 8)])
def test_scores_of_large_statistics(heads, dtype):
    # 5 x 8 x 3876 pages: 39.7 MB of 8-bit bounds, 79 MB of bf16 ones, 159 of float32; a fifth of it per sequence
    w = synth.Workload("streams", 5, heads[0], heads[1], 128, 62011, 16, dtype)
    bounds8 = dtype == "bf16"
    inp = synth.make_inputs(w, 5, device="cuda")
    inp["seq_lens"] = torch.tensor([62010, 61000, 1, 50000 + 15, 62010], device="cuda", dtype=torch.int32)
    big = DeviceState(w, inp, cap=64)
    if bounds8:
        big.enable_box8()
    ekv.ekv_stats_build(big.cfg, big.cache(), big.stats())
    new = [torch.randn(5, heads[1], 128, device="cuda").to(synth.torch_dtype(dtype)) for _ in range(2)]

    def scores(st, k_new, v_new):
        lens, cfg, q = st.inp["seq_lens"], st.cfg, st.inp["q"]
        box8, got = torch.zeros_like(st.box), []
        ekv.ekv_score_pages(cfg, q, st.stats(), lens, ekv.EKV_SCORE_BOTH, st.box, st.mu, st.sigma)
        if bounds8:
            ekv.ekv_score_pages(cfg, q, st.stats(), lens, ekv.EKV_SCORE_BOX8, box8)
        got += [x.clone() for x in (st.box, st.mu, st.sigma, box8)]
        for mode in (ekv.EKV_SCORE_BOTH, ekv.EKV_SCORE_BOX8)[:1 + bounds8]:     # the same token twice at one length: idempotent
            ekv.ekv_append_score_pages(cfg, st.cache(), st.stats(), k_new, v_new, q, mode,
                                       box=st.box if mode == ekv.EKV_SCORE_BOTH else box8, mu=st.mu, sigma=st.sigma)
        torch.cuda.synchronize()
        return got + [x.clone() for x in (st.box, st.mu, st.sigma, box8)]

    singles = []
    for b in range(5):                                  # before the batch appends: the pools are shared
        st = alone(w, inp, b, cap=64)
        st.box_stats, st.gauss_stats = big.box_stats[b:b + 1].clone(), big.gauss_stats[b:b + 1].clone()
        if bounds8:
            st.box8_stats = big.box8_stats[b:b + 1].clone()
        singles.append(scores(st, new[0][b:b + 1].contiguous(), new[1][b:b + 1].contiguous()))
    for whole, *parts in zip(scores(big, *new), *singles):
        for b in range(5):
            assert same(whole[b:b + 1], parts[b])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("page", [12, 16, 32, 64])
@pytest.mark.parametrize("heads", [(8, 8), (16, 8), (32, 8), (64, 8)])
def test_decode_of_large_calls(heads, page, dtype):
    # K of five sequences 143 MB (float32: 287), of one 29 MB (57)
    w = synth.Workload("streams", 5, heads[0], heads[1], 128, 14001, page, dtype)
    inp = synth.make_inputs(w, 6 + page, device="cuda")
    inp["seq_lens"] = torch.tensor([14001, 13990, 1, 4097, 14001], device="cuda", dtype=torch.int32)
    pages = w.pages_per_seq

    def decode(st, lens):
        st.out.zero_()
        ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), st.out, st.tau, st.supp, st.workspace(ekv.EKV_OP_DECODE_FULL))
        got = [x.clone() for x in (st.out, st.tau, st.supp)]
        idx = torch.arange(pages, device="cuda", dtype=torch.int32).expand(st.w.batch, heads[1], pages).contiguous()
        cnt = ((lens + page - 1) // page)[:, None].expand(st.w.batch, heads[1]).contiguous()
        ekv.ekv_decode_sparse_group(st.cfg, st.inp["q"], st.cache(), idx, cnt, st.out, st.tau, st.supp,
                                    st.workspace(ekv.EKV_OP_DECODE_SPARSE))
        got += [x.clone() for x in (st.out, st.tau, st.supp)]
        idx = torch.arange(pages, device="cuda", dtype=torch.int32).expand(st.w.batch, heads[0], pages).contiguous()
        cnt = ((lens + page - 1) // page)[:, None].expand(st.w.batch, heads[0]).contiguous()
        ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), idx, cnt, st.out, st.tau, st.supp,
                              st.workspace(ekv.EKV_OP_DECODE_SPARSE))
        torch.cuda.synchronize()
        return got + [x.clone() for x in (st.out, st.tau, st.supp)]

    whole = decode(DeviceState(w, inp), inp["seq_lens"])
    for b in range(5):
        st = alone(w, inp, b)
        for x, part in zip(whole, decode(st, st.inp["seq_lens"])):
            assert same(x[b:b + 1], part)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("page", [12, 16, 32, 64])
def test_build_of_large_caches(page, dtype):
    # K of five sequences 143 MB (float32: 287), of one 29 MB (57)
    w = synth.Workload("streams", 5, 8, 8, 128, 14001, page, dtype)
    inp = synth.make_inputs(w, 7 + page, device="cuda")
    inp["seq_lens"] = torch.tensor([14001, 13990, 1, 4097, 14001], device="cuda", dtype=torch.int32)

    def build(st):
        got = [st.box_stats, st.gauss_stats] + ([st.enable_box8()] if dtype == "bf16" else [])
        ekv.ekv_stats_build(st.cfg, st.cache(), st.stats())
        torch.cuda.synchronize()
        return got

    whole = build(DeviceState(w, inp))
    for b in range(5):
        for x, part in zip(whole, build(alone(w, inp, b))):
            assert same(x[b:b + 1], part)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_short_sequences_in_a_large_capacity(dtype):
    """The kind of the loads follows the capacity (16 384 pages: 268 MB of statistics and more): short sequences in it give the
    bits that they give in a capacity of their own, and what lies past them is not written."""
    tight = synth.Workload("reserved", 2, 16, 8, 128, 1003, 16, dtype)
    inp = synth.make_inputs(tight, 12, device="cuda")
    inp["seq_lens"] = torch.tensor([1003, 17], device="cuda", dtype=torch.int32)
    wide = tight.scaled(context=262144)
    table = torch.zeros(2, wide.pages_per_seq, device="cuda", dtype=torch.int32)
    table[:, :tight.pages_per_seq] = inp["block_table"]
    got = []
    for w, own in ((tight, inp), (wide, dict(inp, block_table=table))):
        st = DeviceState(w, own)
        st.box_stats.fill_(7.0)
        st.gauss_stats.fill_(7.0)
        ekv.ekv_stats_build(st.cfg, st.cache(), st.stats())
        ekv.ekv_score_pages(st.cfg, own["q"], st.stats(), own["seq_lens"], ekv.EKV_SCORE_BOTH, st.box, st.mu, st.sigma)
        ekv.ekv_decode_full(st.cfg, own["q"], st.cache(), st.out, st.tau, st.supp, st.workspace(ekv.EKV_OP_DECODE_FULL))
        torch.cuda.synchronize()
        for x in (st.box_stats, st.gauss_stats):
            for b, pages in enumerate((63, 2)):
                assert bool((x[b, :, pages:] == 7.0).all())
        got.append([st.out, st.tau, st.supp] + [x[:, :, :63].clone() for x in (st.box_stats, st.gauss_stats, st.box, st.mu, st.sigma)])
    for a, b in zip(*got):
        assert same(a, b)
