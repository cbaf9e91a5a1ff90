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


@pytest.mark.parametrize("dtype,page", [("f32", 8), ("f32", 36), ("bf16", 12), ("bf16", 48)])
def test_more_items_than_a_wavefront_resolves_at_once(dtype, page):
    """128 lists of 40 000 tokens: five and more items to each of the score pass's wavefronts (four per batch of lookups)."""
    w = synth.Workload("steps", 4, 32, 8, 128, 40003, page, dtype)
    inp = synth.make_inputs(w, 11 + page, device="cuda")
    inp["seq_lens"] = torch.tensor([40003, 39000, 37, 40000], device="cuda", dtype=torch.int32)
    out, tau, supp = decode_three_ways(w, inp)
    inp = {key: x.cpu() for key, x in inp.items()}
    for b, h in ((1, 31), (2, 5)):
        q, K, V = unit_kv(inp, w, b, h)
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        check_decode_unit(w, out[b, h], float(tau[b, h]), int(supp[b, h]), None, ref, boundary_expected=True)
