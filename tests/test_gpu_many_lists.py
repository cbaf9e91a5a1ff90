"""The prefix of the lists' lengths and the search for a wavefront's list that every launch over lists begins with: one list to
thousands, empty ones at the front, in rows and at the end, so that a wavefront's range starts in any of them and spans many.

Bit for bit against every sequence decoded by a call of its own, whose search is over a handful of lists."""
import math

import pytest
import torch

from paper_2605_21649_amd import binding as ekv
from paper_2605_21649_amd import synth
from tests.helpers import DeviceState

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("page,dtype", [(16, "bf16"), (8, "f32")])
@pytest.mark.parametrize("batch,heads", [(1, 1), (1, 64), (13, 5), (33, 8), (513, 8), (1030, 8)])
def test_lists_decoded_together_equal_lists_decoded_alone(batch, heads, page, dtype):
    cap = 2048 // page + 2                           # too long for the decode in one launch
    w = synth.Workload("lists", batch, heads, 1 if heads == 8 else heads, 128, cap * page, page, dtype,
                       scale=0.5 / math.sqrt(128.0), n_planted=0)
    gen = torch.Generator().manual_seed(batch + page)
    n = torch.randint(-cap // 4, 9, (batch, heads), generator=gen).clamp_(0)
    n[torch.rand(batch, heads, generator=gen) < 0.02] = cap
    n[0, 0] = 0
    n[batch - 1] = 0
    n[batch // 2, heads - 1] = 3
    pages = torch.stack([torch.randperm(cap, generator=gen).sort().values for _ in range(heads)]).int().expand(batch, heads, cap)
    one = synth.make_inputs(w.scaled(batch=4 if batch > 4 else batch), 7, device="cuda")
    inp = dict(one, q=torch.randn(batch, heads, 128, generator=gen).to(synth.torch_dtype(dtype)).cuda(),
               block_table=one["block_table"].repeat(-(-batch // one["block_table"].shape[0]), 1)[:batch].contiguous(),
               seq_lens=torch.full((batch,), cap * page - 3, dtype=torch.int32, device="cuda"))
    st = DeviceState(w, inp, cap=cap)
    pages, n = pages.contiguous().cuda(), n.int().cuda()
    lse, soft = torch.zeros_like(st.tau), torch.zeros_like(st.out)
    ekv.ekv_decode_sparse(st.cfg, st.inp["q"], st.cache(), pages, n, st.out, st.tau, st.supp, st.workspace(ekv.EKV_OP_DECODE_SPARSE))
    ekv.ekv_decode_sparse_softmax(st.cfg, st.inp["q"], st.cache(), pages, n, soft, lse, st.workspace(ekv.EKV_OP_DECODE_SPARSE_SOFTMAX))
    whole = [st.out, st.tau, st.supp, soft, lse]
    alone = [torch.zeros_like(x) for x in whole]
    cfg = ekv.make_config(1, heads, w.n_kv_heads, 128, page, dtype, w.alpha, w.score_scale, cap, cap)
    ws = [torch.empty(max(256, ekv.ekv_workspace_bytes(cfg, op)), device="cuda", dtype=torch.uint8)
          for op in (ekv.EKV_OP_DECODE_SPARSE, ekv.EKV_OP_DECODE_SPARSE_SOFTMAX)]
    i = st.inp
    for b in sorted(set(range(0, batch, 1 + batch // 60)) | {batch // 2, batch - 1}):
        s = slice(b, b + 1)
        cache = ekv.cache_view(i["k_pool"], i["v_pool"], i["block_table"][s], i["seq_lens"][s])
        out, tau, supp, so, ls = [x[s] for x in alone]
        ekv.ekv_decode_sparse(cfg, i["q"][s], cache, pages[s], n[s], out, tau, supp, ws[0])
        ekv.ekv_decode_sparse_softmax(cfg, i["q"][s], cache, pages[s], n[s], so, ls, ws[1])
        for a, e in zip(whole, alone):
            assert torch.equal(a[b].view(torch.uint8), e[b].view(torch.uint8)), b
