"""float32 page scores have one order of summation, whatever loads the statistics come by: pages are selected by comparing
them, so that a last bit decides between two pages at a cut, and under a flat attention the page decides the output.

The order: the eight channels 8c..8c+7 in turn by fused multiply-adds, the sixteen such sums pairwise (neighbours first), the
rows of a record (bounds below and above) last.  Emulated here in extended precision, rounded to float32 after every step."""
import numpy as np
import pytest
import torch

from paper_2605_21649_amd import binding as ekv
from paper_2605_21649_amd import synth
from tests.helpers import DeviceState

pytestmark = pytest.mark.gpu


def row_sums(coef, rows):
    """coef [..., 128] times rows [..., 128] summed in the kernels' order."""
    coef, rows = (x.astype(np.longdouble).reshape(*x.shape[:-1], 16, 8) for x in (coef, rows))
    acc = np.zeros(np.broadcast_shapes(coef.shape, rows.shape)[:-1], np.float32)
    for i in range(8):                              # 48 bits of product, 64 of sum: one rounding, to float32
        acc = (coef[..., i] * rows[..., i] + acc.astype(np.longdouble)).astype(np.float32)
    while acc.shape[-1] > 1:
        acc = acc[..., 0::2] + acc[..., 1::2]
    return acc[..., 0]


@pytest.mark.parametrize("heads", [(2, 2), (4, 2), (8, 2), (16, 2)])
@pytest.mark.parametrize("tokens", [801, 16 * 20480])          # 0.1 MB of statistics, and 42 (a stream) of which some are checked
def test_float32_scores_keep_their_order(heads, tokens):
    w = synth.Workload("order", 1, heads[0], heads[1], 128, tokens, 16, "f32")
    inp = synth.make_inputs(w, 7, device="cuda")
    st = DeviceState(w, inp, cap=8)
    gen = torch.Generator(device="cuda").manual_seed(8)
    st.box_stats.normal_(generator=gen)
    st.gauss_stats.normal_(generator=gen)
    st.gauss_stats[..., 1, :].abs_()
    ekv.ekv_score_pages(st.cfg, st.inp["q"], st.stats(), st.inp["seq_lens"], ekv.EKV_SCORE_BOTH, st.box, st.mu, st.sigma)
    torch.cuda.synchronize()
    pages = np.unique(np.append(np.arange(0, w.pages_per_seq, 1 if tokens < 4096 else 37), w.pages_per_seq - 1))
    scale, group = np.float32(w.score_scale), heads[0] // heads[1]
    for h in range(heads[0]):
        q = st.inp["q"][0, h].cpu().numpy()
        box, gauss = (x[0, h // group].cpu().numpy()[pages] for x in (st.box_stats, st.gauss_stats))
        want = scale * (row_sums(np.minimum(q, 0), box[:, 0]) + row_sums(np.maximum(q, 0), box[:, 1]))
        assert np.array_equal(st.box[0, h].cpu().numpy()[pages], want)
        assert np.array_equal(st.mu[0, h].cpu().numpy()[pages], scale * row_sums(q, gauss[:, 0]))
        assert np.array_equal(st.sigma[0, h].cpu().numpy()[pages], scale * np.sqrt(row_sums(q * q, gauss[:, 1])))


@pytest.mark.parametrize("heads", [(2, 2), (4, 2), (8, 2), (16, 2)])
@pytest.mark.parametrize("reserved", [32, 4096])                # capacity in tokens: 2 MB of K, and 268 (a stream)
def test_float32_decode_scores_keep_their_order(heads, reserved):
    """Over one token tau is its score less one, an exact difference for scores in [0.5, 2], and the softmax's lse the score.
    A threshold on page bounds compares them with tau, so its last bit decides as well."""
    w = synth.Workload("order", 64, heads[0], heads[1], 128, 16, 16, "f32")
    gen = torch.Generator(device="cuda").manual_seed(9)
    dev = dict(device="cuda", dtype=torch.float32)
    q = torch.rand(64, heads[0], 128, generator=gen, **dev)
    k, v = torch.rand(64, heads[1], 16, 128, generator=gen, **dev), torch.randn(64, heads[1], 16, 128, generator=gen, **dev)
    lens = torch.ones(64, device="cuda", dtype=torch.int32)
    pages = reserved // 16
    table = torch.arange(64, device="cuda", dtype=torch.int32)[:, None].expand(64, pages).contiguous()
    cfg = ekv.make_config(64, heads[0], heads[1], 128, 16, "f32", 1.5, 1.0 / 16.0, pages, pages)
    cache = ekv.cache_view(k, v, table, lens)
    # 1 / 32 a channel, an exact factor: (alpha - 1) * score around 1
    kq = k[:, :, 0].cpu().numpy().repeat(heads[0] // heads[1], 1)
    score = np.float32(1.0 / 16.0) * row_sums(q.cpu().numpy(), kq)
    want = np.float32(0.5) * score
    sure = (want >= 0.5) & (want <= 2.0)
    assert sure.mean() > 0.9

    def room(op):
        return torch.empty(max(256, ekv.ekv_workspace_bytes(cfg, op)), device="cuda", dtype=torch.uint8)

    for way in ("all", "group", "head"):
        lists = heads[1] if way == "group" else heads[0]
        idx, cnt = (torch.zeros(64, lists, pages, device="cuda", dtype=torch.int32), torch.ones(64, lists, device="cuda", dtype=torch.int32))
        out, tau = torch.zeros(64, heads[0], 128, **dev), torch.zeros(64, heads[0], **dev)
        supp = torch.zeros(64, heads[0], device="cuda", dtype=torch.int32)
        if way == "all":
            ekv.ekv_decode_full(cfg, q, cache, out, tau, supp, room(ekv.EKV_OP_DECODE_FULL))
        elif way == "group":
            ekv.ekv_decode_sparse_group(cfg, q, cache, idx, cnt, out, tau, supp, room(ekv.EKV_OP_DECODE_SPARSE))
        else:
            ekv.ekv_decode_sparse(cfg, q, cache, idx, cnt, out, tau, supp, room(ekv.EKV_OP_DECODE_SPARSE))
        torch.cuda.synchronize()
        assert np.array_equal(tau.cpu().numpy()[sure], (want - np.float32(1.0))[sure]), way

    ekv.ekv_decode_sparse_softmax(cfg, q, cache, idx, cnt, out, tau, room(ekv.EKV_OP_DECODE_SPARSE_SOFTMAX))
    torch.cuda.synchronize()
    assert np.array_equal(tau.cpu().numpy(), score)
