"""The dense decode's score pass of large calls (bf16 pages of 16, 32 and 64; 256 MiB of K and 8 MiB of scores and more), which
holds scores in LDS and stores them late: every number of heads and page size, sequences from none to all of the capacity, a
wavefront's range from no item to more than one batch of lookups and more than it holds, and from one unit to thousands.

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
    inp = synth.make_inputs(w, 17 + page, device="cuda")
    inp["seq_lens"] = torch.tensor(lens, dtype=torch.int32, device="cuda")
    compare_with_lists(w, inp)


def compare_with_lists(w, inp):
    page, slots = w.page_size, w.pages_per_seq * w.page_size
    assert w.batch * w.n_kv_heads * slots * 256 >= 256 << 20 and w.batch * w.n_q_heads * slots * 4 >= 8 << 20
    assert w.batch * w.n_kv_heads <= 4096
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


def shared_pages(batch, heads, context, page, lens, pool_pages=4096):
    """Inputs whose sequences share the pages of a small pool: K of any size as far as the kernel sees."""
    w = synth.Workload("windows", batch, heads[0], heads[1], 128, context, page, "bf16", scale=0.5 / math.sqrt(128.0))
    inp = synth.make_inputs(w.scaled(batch=1, context=pool_pages * page), 23 + page, device="cuda")
    gen = torch.Generator().manual_seed(page + heads[0])
    inp["block_table"] = torch.randint(0, pool_pages, (batch, w.pages_per_seq), generator=gen).int().cuda()
    inp["q"] = torch.randn(batch, heads[0], 128, generator=gen).bfloat16().cuda()
    inp["seq_lens"] = torch.tensor(lens, dtype=torch.int32, device="cuda")
    return w, inp


@pytest.mark.parametrize("page", [16, 32, 64])
@pytest.mark.parametrize("group", [1, 2, 4, 8])
def test_ranges_longer_than_a_batch_and_than_the_lds(group, page):
    w, inp = shared_pages(3, (4 * group, 4), 786432, page, [786432 - 7, 660003, 786432])
    wavefronts = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    items = sum(-(-n // 64) for n in inp["seq_lens"].tolist()) * 4 // wavefronts
    assert items > page and items > 8192 // 64 // group      # a batch of lookups is 64 page slots, a wavefront holds 8192 scores
    compare_with_lists(w, inp)


@pytest.mark.parametrize("batch,heads,page", [(512, (8, 8), 16), (512, (32, 8), 32), (33, (8, 8), 64), (511, (64, 8), 16)])
def test_thousands_of_units(batch, heads, page):
    context = 512 if batch > 100 else 8192
    gen = torch.Generator().manual_seed(batch)
    lens = torch.randint(0, context + 1, (batch,), generator=gen)
    lens[torch.rand(batch, generator=gen) < 0.2] = 0
    lens[0], lens[batch - 1] = 1, context
    compare_with_lists(*shared_pages(batch, heads, context, page, lens.tolist()))
