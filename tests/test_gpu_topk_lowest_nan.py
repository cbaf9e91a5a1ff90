"""Top-k by one workgroup with scores whose key is the lowest there is (a NaN of all ones): they are pages like the others, the
last to be taken, also where the budget takes them and the other scores lie on both sides of zero."""
import numpy as np
import pytest
import torch

from paper_2605_21649_amd import binding as ekv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [513, 1024, 2626, 16384])
@pytest.mark.parametrize("at", ["first", "last", "both", "all"])
@pytest.mark.parametrize("offset", [0.0, 15.0])
def test_lowest_nan_is_taken_last(M, at, offset):
    rng = np.random.default_rng(M)
    Hq, P = 2, 16
    x = (rng.standard_normal((1, Hq, M)) + offset).astype(np.float32)
    bad = {"first": [0], "last": [M - 1], "both": [0, M - 1], "all": list(range(M))}[at]
    x.view(np.uint32)[..., bad] = 0xffffffff
    order = np.where(np.isnan(x), -np.inf, x)
    box, lens = torch.from_numpy(x).cuda(), torch.tensor([M * P], dtype=torch.int32, device="cuda")
    for k in sorted({1, M // 2, M - 1, M}):
        cfg = ekv.make_config(1, Hq, Hq, 128, P, "bf16", 1.5, 1.0, M, k)
        idx = torch.full((1, Hq, k), -7, device="cuda", dtype=torch.int32)
        n_sel = torch.full((1, Hq), -1, device="cuda", dtype=torch.int32)
        ws = torch.empty(max(256, ekv.ekv_workspace_bytes(cfg, ekv.EKV_OP_SELECT_TOPK)), device="cuda", dtype=torch.uint8)
        ekv.ekv_select_topk(cfg, box, lens, k, idx, n_sel, ws)
        torch.cuda.synchronize()
        assert (n_sel.cpu().numpy() == k).all()
        for h in range(Hq):
            assert np.array_equal(idx[0, h].cpu().numpy(), np.sort(np.argsort(-order[0, h], kind="stable")[:k])), (k, h)
