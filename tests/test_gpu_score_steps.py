"""The decode's score pass over steps of four tokens (float32 caches and bf16 pages other than 16, 32 and 64): every page
size's remainder of steps, every number of heads, ragged ends, and more items than a wavefront resolves at once.

Results against the float64 oracle under the rules of tests/helpers.py; and bit for bit between the decode of all pages,
the same pages as a list per KV head and as lists per head, which differ in the heads a step serves."""
import math

import pytest
import torch

from oracle import entmaxkv_oracle as orc
from paper_2605_21649_amd import binding as ekv
from paper_2605_21649_amd import synth
from tests.helpers import DeviceState, unit_kv, check_decode_unit

pytestmark = pytest.mark.gpu


def decode_three_ways(w, inp):
    st = DeviceState(w, inp)
    lens = st.inp["seq_lens"]
    pages = torch.arange(st.cap, device="cuda", dtype=torch.int32).expand(w.batch, w.n_q_heads, st.cap).contiguous()
    counts = ((lens + w.page_size - 1) // w.page_size)[:, None].expand(w.batch, w.n_q_heads).contiguous()
    ws = st.workspace(ekv.EKV_OP_DECODE_SPARSE)
    got = []
    for way in ("all", "group", "head"):
        if way == "all":
            ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), st.out, st.tau, st.supp, st.workspace(ekv.EKV_OP_DECODE_FULL))
        elif way == "group":
            ekv.ekv_decode_sparse_group(st.cfg, st.inp["q"], st.cache(), pages[:, :w.n_kv_heads].contiguous(),
                                        counts[:, :w.n_kv_heads].contiguous(), st.out, st.tau, st.supp, ws)
        else:
            ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), pages, counts, st.out, st.tau, st.supp, ws)
        torch.cuda.synchronize()
        got.append([x.clone() for x in (st.out, st.tau, st.supp)])
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    return [x.cpu().numpy() for x in got[0]]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("page", [4, 8, 12, 20, 24, 28, 36, 40, 44, 48, 52, 56, 60, 64])
@pytest.mark.parametrize("heads", [(2, 2), (4, 2), (4, 1), (8, 1)])
def test_every_page_size_and_number_of_heads(dtype, page, heads):
    w = synth.Workload("steps", 3, heads[0], heads[1], 128, 5003, page, dtype, scale=0.5 / math.sqrt(128.0))
    inp = synth.make_inputs(w, 3 + page, device="cpu")
    inp["seq_lens"] = torch.tensor([5003, 1, 4200 - page], dtype=torch.int32)
    out, tau, supp = decode_three_ways(w, inp)
    for b, h in ((0, 0), (1, heads[0] - 1), (2, heads[0] - 1)):
        q, K, V = unit_kv(inp, w, b, h)
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        check_decode_unit(w, out[b, h], float(tau[b, h]), int(supp[b, h]), None, ref, boundary_expected=True)


def items_per_wavefront(w, units, all_pages):
    """Items (groups of pages of 33 to 64 tokens) that a wavefront of the score pass takes, by the launcher's rule."""
    items = units * -(-w.pages_per_seq // max(1, 64 // w.page_size))
    per_cu = (128 if units <= 1024 else 32) if all_pages else (16 if units <= 256 else 8)
    workgroups = min(-(-items // 4), per_cu * torch.cuda.get_device_properties(0).multi_processor_count)
    return items / (4 * workgroups)


@pytest.mark.parametrize("dtype,page", [("f32", 8), ("f32", 20), ("f32", 36), ("bf16", 12), ("bf16", 28), ("bf16", 48)])
@pytest.mark.parametrize("heads", [(8, 8), (16, 8), (32, 8), (64, 8)])
def test_wavefronts_that_take_several_batches(heads, dtype, page):
    """130 sequences on the same pages, 1040 units and more: in every mode a wavefront takes more items than the four that it
    resolves at once, and crosses from unit to unit; the lists of 64 heads are so many that their prefix is kept in memory."""
    w = synth.Workload("batches", 130, heads[0], heads[1], 128, 9603, page, dtype)
    for units, all_pages in ((130 * heads[1], True), (130 * heads[1], False), (130 * heads[0], False)):
        assert items_per_wavefront(w, units, all_pages) > 4.5
    inp = synth.make_inputs(w.scaled(batch=1), 13 + page, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(page)
    inp["q"] = torch.randn(130, heads[0], 128, generator=gen, device="cuda").to(inp["q"].dtype)
    inp["block_table"] = inp["block_table"].expand(130, -1).contiguous()
    inp["seq_lens"] = torch.tensor([9603 - 7 * (b % 5) for b in range(130)], device="cuda", dtype=torch.int32)
    out, tau, supp = decode_three_ways(w, inp)
    inp = {key: x.cpu() for key, x in inp.items()}
    for b, h in ((0, 0), (64, heads[0] // 2), (129, heads[0] - 1)):
        q, K, V = unit_kv(inp, w, b, h)
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        check_decode_unit(w, out[b, h], float(tau[b, h]), int(supp[b, h]), None, ref, boundary_expected=True)


@pytest.mark.parametrize("dtype,page", [("f32", 8), ("f32", 36), ("bf16", 12), ("bf16", 48)])
def test_more_items_than_a_wavefront_resolves_at_once(dtype, page):
    """128 lists of 40 000 tokens: by lists per head five and more items to a wavefront of the score pass in pages of 36 and 48,
    four and fewer in the others; one or two by the other ways (more of them: the test above)."""
    w = synth.Workload("steps", 4, 32, 8, 128, 40003, page, dtype)
    inp = synth.make_inputs(w, 11 + page, device="cuda")
    inp["seq_lens"] = torch.tensor([40003, 39000, 37, 40000], device="cuda", dtype=torch.int32)
    out, tau, supp = decode_three_ways(w, inp)
    inp = {key: x.cpu() for key, x in inp.items()}
    for b, h in ((1, 31), (2, 5)):
        q, K, V = unit_kv(inp, w, b, h)
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        check_decode_unit(w, out[b, h], float(tau[b, h]), int(supp[b, h]), None, ref, boundary_expected=True)
