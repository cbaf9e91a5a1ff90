"""Box-threshold selection at the edges of its forms: one launch for rows of up to 4096, 8192 and 16384 pages, two beyond; lists cut
at their capacity; the given list as the output.  Scores times a = 1/2 are exact in float32, so the sets are the oracle's."""
import numpy as np
import pytest
import torch

from oracle import entmaxkv_oracle as orc
from paper_2605_21649_amd import binding as ekv
from paper_2605_21649_amd import synth
from tests.helpers import DeviceState

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("M,cap", [(1, 1), (63, 20), (64, 64), (1024, 1000), (4095, 4095), (4096, 300), (4096, 4096), (4097, 4097), (8191, 500), (8192, 8192), (8193, 8193), (12288, 12288), (12289, 400),
                                   (16383, 16383), (16384, 700), (16385, 16385)])
def test_rows_at_the_edges(M, cap, in_place):
    w = synth.Workload("box-rows", 2, 4, 4, 128, 4 * M, 4, "bf16")
    inp = synth.make_inputs(w, 3, device="cpu")
    lens = [4 * M, max(1, 4 * (M - M // 3) - 2)]
    inp["seq_lens"] = torch.tensor(lens, dtype=torch.int32)
    st = DeviceState(w, inp, cap=cap)
    rng = np.random.default_rng(M)
    scores = rng.normal(size=(2, 4, M)).astype(np.float32)
    tau = np.array([[np.quantile(scores[b, 0], 0.9) / 2, np.inf, -np.inf, scores[b, 3].max() / 2] for b in range(2)], np.float32)
    given = [[rng.choice(M, min(M, cap, n), replace=False).astype(np.int32) for n in (0, 40, 3, 500)] for _ in range(2)]
    for b in range(2):
        for h in range(4):
            st.page_idx[b, h, :len(given[b][h])] = torch.from_numpy(given[b][h]).cuda()
            st.n_sel[b, h] = len(given[b][h])
    st.box.copy_(torch.from_numpy(scores))
    out, n_out = (st.page_idx, st.n_sel) if in_place else (torch.full_like(st.page_idx, -7), torch.zeros_like(st.n_sel))
    added, over = torch.zeros_like(st.n_sel), torch.zeros_like(st.n_sel)
    ekv.ekv_select_box_threshold(st.cfg, st.box, st.inp["seq_lens"], torch.from_numpy(tau).cuda(), st.page_idx, st.n_sel, out,
                                 n_out, added, over, st.workspace(ekv.EKV_OP_SELECT_BOX_THRESHOLD))
    torch.cuda.synchronize()
    for b in range(2):
        pages = -(-lens[b] // 4)
        for h in range(4):
            old = np.array(sorted(p for p in given[b][h] if p < pages), dtype=np.int64)
            union, new = orc.refine_selection(scores[b, h, :pages].astype(np.float64), 1.5, float(tau[b, h]), old)
            assert int(n_out[b, h]) == min(len(union), cap) and int(added[b, h]) == len(new)
            assert int(over[b, h]) == (len(union) > cap)
            np.testing.assert_array_equal(out[b, h, :int(n_out[b, h])].cpu().numpy(), union[:cap])
