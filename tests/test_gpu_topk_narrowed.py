"""Top-k by one workgroup over scores on both sides of zero whose equal steps do not separate them: the step of the k-th score
holds hundreds, and the radix passes go on inside it, whatever lies above and below; outliers that make the steps useless.

Exact against a stable sort: larger score first, lower page first among equals (-0 and +0 are equal), ascending order."""
import numpy as np
import pytest
import torch

from paper_2605_21649_amd import binding as ekv

pytestmark = pytest.mark.gpu


def scores(kind, rng, M):
    x = rng.standard_normal(M).astype(np.float32)
    pick = rng.random(M)
    if kind == "two_clusters":                               # both ends of the range: hundreds or thousands in the k-th's step
        x = (np.where(pick < 0.5, -1, 1) * (1 + rng.random(M) * 2e-4)).astype(np.float32)
    elif kind == "three_values":                             # the step holds one value
        x = rng.integers(-1, 2, M).astype(np.float32) * np.float32(0.3)
    elif kind == "one_ulp":                                  # two neighbouring values in one step
        x = np.where(pick < 0.4, np.float32(1), np.where(pick < 0.8, np.nextafter(np.float32(1), np.float32(2)), np.float32(-1)))
    elif kind == "around_zero":                              # the step itself lies on both sides of zero
        x = np.where(pick < 0.9, x * 1e-4, x * 3).astype(np.float32)
        x[pick < 0.1] = -0.0
    elif kind == "spread_exponents":                         # a step of zero's many octaves
        x = (np.sign(x) * np.exp2(rng.uniform(-40, 3, M))).astype(np.float32)
    elif kind == "outliers":
        x[0], x[M - 1] = -7e4, 6e4
    elif kind == "outliers_in_half":                         # in half of the wavefronts
        at = np.arange(0, M, 128)
        x[at] = np.where(np.arange(len(at)) % 2, 9e3, -9e3)
        x[M // 2:] = rng.standard_normal(M - M // 2).astype(np.float32)
    return x.astype(np.float32)


@pytest.mark.parametrize("kind", ["two_clusters", "three_values", "one_ulp", "around_zero", "spread_exponents", "outliers",
                                  "outliers_in_half"])
@pytest.mark.parametrize("M", [513, 1023, 1024, 2049, 4096, 5000, 8193, 16384])
def test_topk_inside_one_step(kind, M):
    rng = np.random.default_rng(M)
    Hq, P = 4, 16
    x = np.stack([scores(kind, rng, M) for _ in range(Hq)])[None]
    if kind == "outliers_in_half":
        x[0, 1] = x[0, 1, ::-1]
    lens = torch.tensor([M * P - 5], dtype=torch.int32, device="cuda")
    box = torch.from_numpy(x).cuda()
    for k in sorted({1, M // 50, M // 3, M // 2, 3 * M // 4, M - 1, M}):
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
