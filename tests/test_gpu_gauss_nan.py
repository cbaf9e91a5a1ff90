"""A page whose estimated mean is NaN (a key that is not finite) must not vanish from the mass of the Gaussian selector: no point
satisfies the threshold equation then, and tau_hat falls back to the left end of its bracket, max (alpha - 1) mu - 1, where
every page that could hold a support token is kept.  In the selector of one launch and in the sliced one, for every exponent."""
import pytest
import torch

from paper_2605_21649_amd import binding as ekv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alpha", [2.0, 1.5, 4.0 / 3.0, 1.25])
@pytest.mark.parametrize("M", [65, 2048, 8192, 8193, 20000])
def test_a_nan_mean_leaves_the_left_end(M, alpha):
    H, P = 3, 16
    gen = torch.Generator().manual_seed(M)
    mu = 0.5 * torch.randn(1, H, M, generator=gen)
    sigma = 0.5 + torch.rand(1, H, M, generator=gen)
    bad = [0, M // 2, M - 1]
    for h in range(H):
        mu[0, h, bad[h]] = float("nan")
    left = ((alpha - 1.0) * mu.nan_to_num(-9e9)).amax(-1) - 1.0
    cfg = ekv.make_config(1, H, H, 128, P, "bf16", alpha, 1.0, M, M)
    lens = torch.tensor([M * P - 5], dtype=torch.int32, device="cuda")
    tau = torch.zeros(1, H, device="cuda")
    idx = torch.full((1, H, M), -1, device="cuda", dtype=torch.int32)
    n_sel, overflow = (torch.full((1, H), -1, device="cuda", dtype=torch.int32) for _ in range(2))
    ws = torch.empty(max(256, ekv.ekv_workspace_bytes(cfg, ekv.EKV_OP_SELECT_GAUSS)), device="cuda", dtype=torch.uint8)
    ekv.ekv_select_gauss(cfg, mu.cuda(), sigma.cuda(), lens, 0.99, 0.0, tau, idx, n_sel, overflow, ws)
    torch.cuda.synchronize()
    # bisection ends at a step of 3e-7 of the threshold; the left end itself is two float32 roundings from the one above
    assert ((tau.cpu() - left).abs() <= 1e-6 * left.abs().clamp(min=1.0)).all(), (tau.cpu(), left)
    for h in range(H):
        # a page whose mean alone reaches the threshold is kept whatever its estimate adds
        sure = torch.nonzero((alpha - 1.0) * mu[0, h] > left[0, h] + 1e-4).flatten().tolist()
        assert set(sure) - {bad[h]} <= set(idx[0, h, :n_sel[0, h]].tolist())
