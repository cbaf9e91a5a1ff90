"""The dense decode's score pass of large calls (bf16 pages of 16, 32 and 64; 256 MiB of K and 8 MiB of scores and more), which
holds scores in LDS and stores them late: every number of heads and page size, sequences from none to all of the capacity, so
that a wavefront gets from no item to more than it holds.

Bit for bit against the same pages as a list per KV head, whose scores are stored at once; the oracle checks this path at full
size (test_gpu_full_size.py, test_gpu_full_size_c5.py)."""
import math

import pytest
import torch

from paper_2605_21649_amd import binding as ekv
from paper_2605_21649_amd import synth
from tests.helpers import DeviceState

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("page", [16, 32, 64])
@pytest.mark.parametrize("heads,context,lens", [
    ((4, 4), 131072, [131072 - 7, 0, 1, 4099]),
    ((8, 4), 65536, [3, 65536, 0, 65536 - 31]),
    ((16, 4), 65536, [65536, 65536 - 1, 65, 65536 - 64]),
    ((32, 4), 65536, [0, 65536 - 17, 63, 2048]),
    ((16, 4), 65536, [1, 64, 0, 129]),               # fewer items than wavefronts
    ((16, 4), 65536, [0, 0, 0, 0]),
    ((8, 1), 1048576 - 3, [1048576 - 3]),            # one long row, odd items per wavefront at its end
])
def test_windows_equal_the_scores_of_a_list(heads, context, lens, page):
    w = synth.Workload("windows", len(lens), heads[0], heads[1], 128, context, page, "bf16", scale=0.5 / math.sqrt(128.0))
    assert len(lens) * heads[1] * w.pages_per_seq * page * 256 >= 256 << 20
    assert len(lens) * heads[0] * w.pages_per_seq * page * 4 >= 8 << 20
    inp = synth.make_inputs(w, 17 + page, device="cuda")
    inp["seq_lens"] = torch.tensor(lens, dtype=torch.int32, device="cuda")
    st = DeviceState(w, inp)
    pages = torch.arange(st.cap, device="cuda", dtype=torch.int32).expand(w.batch, w.n_kv_heads, st.cap).contiguous()
    counts = ((st.inp["seq_lens"] + page - 1) // page)[:, None].expand(w.batch, w.n_kv_heads).contiguous()
    decode = ekv.ekv_decode_sparse_group if w.group > 1 else ekv.ekv_decode_sparse
    decode(st.cfg, st.inp["q"], st.cache(), pages, counts, st.out, st.tau, st.supp, st.workspace(ekv.EKV_OP_DECODE_SPARSE))
    want = [x.clone() for x in (st.out, st.tau, st.supp)]
    for _ in range(3):                               # over a scratch that holds the last call's scores
        for x in (st.out, st.tau, st.supp):
            x.zero_()
        ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), st.out, st.tau, st.supp, st.workspace(ekv.EKV_OP_DECODE_FULL))
        for a, b in zip((st.out, st.tau, st.supp), want):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
