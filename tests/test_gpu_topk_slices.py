"""Top-k over rows of many slices (more than 16384 pages): budgets on both sides of a slice's list, the selection crowded into
a few slices or spread, single values that fill slices, ragged rows beside empty ones, every number of slices' edge, and both
sides of the line between two launches and three (for few rows 509 pages at 52 slices, 336 at 64).

Exact against a stable sort: larger score first, lower page first among equals, written in ascending order."""
import numpy as np
import pytest
import torch

from paper_2605_21649_amd import binding as ekv

pytestmark = pytest.mark.gpu

SLICE = 4096


def scores(kind, rng, rows, M):
    x = rng.standard_normal((rows, M)).astype(np.float32)
    if kind == "trend":
        x += np.linspace(0, 6, M, dtype=np.float32)          # the best pages are the last slices' own
    elif kind == "levels":
        x = rng.integers(0, 5, (rows, M)).astype(np.float32)
    elif kind == "one_slice":
        x[:, SLICE:2 * SLICE] += 50
    elif kind == "equal":
        x[:] = 1.25
    elif kind == "equal_but_few":
        x[:] = -0.0
        x[:, rng.choice(M, 40, replace=False)] = 1.0
        x[:, 5] = 0.0
    return x


@pytest.mark.parametrize("kind", ["normal", "trend", "levels", "one_slice", "equal", "equal_but_few"])
@pytest.mark.parametrize("M,k,Hq", [(16385, 1, 2), (4 * SLICE + 1, 600, 2), (5 * SLICE, 2560, 2), (5 * SLICE - 1, 2561, 2), (20000, 10000, 2),
                                    (65536, 1311, 2), (65537, 511, 2), (64 * SLICE, 5243, 2), (64 * SLICE - 31, 140000, 2), (17000, 17000, 2),
                                    (52 * SLICE, 508, 2), (52 * SLICE, 510, 2), (64 * SLICE, 336, 2), (64 * SLICE - 31, 337, 2),
                                    (64 * SLICE, 5243, 22)])
def test_topk_over_slices(kind, M, k, Hq):
    B, P = 3, 16
    rng = np.random.default_rng(M + k)
    x = scores(kind, rng, B * Hq, M).reshape(B, Hq, M)
    lens = np.array([M * P - 7, 0, (M // 2) * P + 1], dtype=np.int32)
    cfg = ekv.make_config(B, Hq, Hq, 128, P, "bf16", 1.5, 1.0, M, k)
    box = torch.from_numpy(x).cuda()
    flat = torch.full((B * Hq * k + 4096,), -7, device="cuda", dtype=torch.int32)
    idx = flat[:B * Hq * k].view(B, Hq, k)
    n_sel = torch.full((B, Hq), -1, device="cuda", dtype=torch.int32)
    ws = torch.empty(max(256, ekv.ekv_workspace_bytes(cfg, ekv.EKV_OP_SELECT_TOPK)), device="cuda", dtype=torch.uint8)
    for _ in range(2):
        ekv.ekv_select_topk(cfg, box, torch.from_numpy(lens).cuda(), k, idx, n_sel, ws)
    torch.cuda.synchronize()
    for b in range(B):
        m = -(-int(lens[b]) // P)
        want_n = min(k, m)
        assert (n_sel[b].cpu().numpy() == want_n).all()
        assert (idx[b, :, want_n:] == -7).all()              # nothing behind a row's count
        for h in range(Hq):
            want = np.sort(np.argsort(-x[b, h, :m], kind="stable")[:want_n])
            assert np.array_equal(idx[b, h, :want_n].cpu().numpy(), want), (b, h)
    assert (flat[B * Hq * k:] == -7).all()
