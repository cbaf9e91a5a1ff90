"""The softmax over page lists in batches of four steps: every page size's remainder of steps, lists that end within a
wavefront's pair of pages, a partial last page; against the float64 oracle, with the bounds of the path's other test."""
import math

import numpy as np
import pytest
import torch

from oracle import entmaxkv_oracle as orc
from paper_2605_21649_amd import binding as ekv
from paper_2605_21649_amd import synth
from tests.helpers import DeviceState, rel_err, unit_kv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("page", [4, 8, 12, 16, 20, 28, 32, 36, 48, 60, 64])
def test_every_page_size(dtype, page):
    w = synth.Workload("softmax-steps", 2, 4, 2, 128, 2003, page, dtype, scale=0.5 / math.sqrt(128.0))
    inp = synth.make_inputs(w, 9 + page, device="cpu")
    inp["seq_lens"] = torch.tensor([2003, 1401], dtype=torch.int32)
    cap = 27
    st = DeviceState(w, inp, cap=cap)
    rng = np.random.default_rng(page)
    lists = {}
    for b, lens in enumerate((2003, 1401)):
        total = -(-lens // page)
        for h, count in enumerate((1, 2, 17, cap)):
            pages = np.sort(rng.choice(total - 1, min(count, total) - 1, replace=False))
            lists[b, h] = np.append(pages, total - 1)                          # the partial last page
            st.page_idx[b, h, :len(lists[b, h])] = torch.from_numpy(lists[b, h].astype(np.int32)).cuda()
            st.n_sel[b, h] = len(lists[b, h])
    lse = torch.zeros_like(st.tau)
    ekv.ekv_decode_sparse_softmax(st.cfg, st.inp["q"], st.cache(), st.page_idx, st.n_sel, st.out, lse,
                                  st.workspace(ekv.EKV_OP_DECODE_SPARSE_SOFTMAX))
    torch.cuda.synchronize()
    out, own = st.out.clone(), lse.clone()
    cache = st.cache()
    cache.n_phys_pages = 2 ** 31 - 1                    # a view may declare more pages than the table names
    ekv.ekv_decode_sparse_softmax(st.cfg, st.inp["q"], cache, st.page_idx, st.n_sel, st.out, lse,
                                  st.workspace(ekv.EKV_OP_DECODE_SPARSE_SOFTMAX))
    torch.cuda.synchronize()
    assert torch.equal(st.out, out) and torch.equal(lse, own)
    for (b, h), pages in lists.items():
        q, K, V = unit_kv(inp, w, b, h)
        ref = orc.softmax_attention(q, K, V, w.score_scale, orc.pages_to_tokens(pages, page, K.shape[0]))
        assert rel_err(st.out[b, h].cpu().numpy(), ref["o"]) <= 2e-5
        assert abs(float(lse[b, h]) - ref["lse"]) <= 2e-5 * max(1.0, abs(ref["lse"]))
