"""Top-k by one workgroup over scores on both sides of zero, whose keys span most of their 32 bits: the histogram over equal
steps of the scores, and its ways out -- a range that is not finite, a step with hundreds of scores.

Exact against a stable sort: larger score first, lower page first among equals (-0 and +0 are equal), ascending order."""
import numpy as np
import pytest
import torch

from paper_2605_21649_amd import binding as ekv

pytestmark = pytest.mark.gpu


def scores(kind, rng, M):
    x = (rng.standard_normal(M) * 1.5 + 15).astype(np.float32)
    if kind == "one_negative":
        x[M - 1] = -2.5
    elif kind == "normal":
        x -= 15
    elif kind == "crowded":                                  # one step holds nearly all of them
        x[:] = 15 + rng.random(M).astype(np.float32) * 1e-3
        x[0], x[1] = -4e4, 5e4
    elif kind == "levels":
        x[:] = rng.integers(-3, 4, M)
    elif kind == "zeros":
        x[:] = np.where(rng.random(M) < 0.5, np.float32(0.0), np.float32(-0.0))
        x[3] = -1.0
    elif kind == "infinite":
        x[5], x[M // 2], x[7] = np.inf, -np.inf, -1.0
    elif kind == "huge":
        x[2], x[4] = -3e38, 3e38
    elif kind == "tiny":
        x[:] = (rng.integers(-9, 9, M) * 1e-45).astype(np.float32)
    return x


@pytest.mark.parametrize("kind", ["one_negative", "normal", "crowded", "levels", "zeros", "infinite", "huge", "tiny"])
@pytest.mark.parametrize("M", [513, 1024, 1025, 2049, 2626, 4097, 8192, 8193, 16384])
def test_topk_of_scores_around_zero(kind, M):
    rng = np.random.default_rng(M)
    ks = sorted({1, 53, M // 3, M - 1, M})
    Hq, P = 3, 16
    x = np.stack([scores(kind, rng, M) for _ in range(Hq)])[None]
    lens = torch.tensor([M * P - 5], dtype=torch.int32, device="cuda")
    box = torch.from_numpy(x).cuda()
    for k in ks:
        cfg = ekv.make_config(1, Hq, Hq, 128, P, "bf16", 1.5, 1.0, M, k)
        idx = torch.full((1, Hq, k), -7, device="cuda", dtype=torch.int32)
        n_sel = torch.full((1, Hq), -1, device="cuda", dtype=torch.int32)
        ws = torch.empty(max(256, ekv.ekv_workspace_bytes(cfg, ekv.EKV_OP_SELECT_TOPK)), device="cuda", dtype=torch.uint8)
        ekv.ekv_select_topk(cfg, box, lens, k, idx, n_sel, ws)
        torch.cuda.synchronize()
        assert (n_sel.cpu().numpy() == k).all()
        for h in range(Hq):
            want = np.sort(np.argsort(-x[0, h], kind="stable")[:k])
            assert np.array_equal(idx[0, h].cpu().numpy(), want), (k, h)
