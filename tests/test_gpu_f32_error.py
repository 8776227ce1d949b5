"""The fp32 router's rounding: its logits are no further from float64 than a sum
over 64 lanes (lane l adds the products of the features l, l + 64, ... with
fused multiply-adds, the lanes are added in pairs), which is emulated here
in numpy.  The bound is 1.05 of that sum's 2-norm distance: four standard
deviations of the estimate over 64 x 64 logits."""
import numpy as np
import pytest
import torch

from paper_2605_30876_amd import lib

pytestmark = pytest.mark.gpu


def _lane_sums(x, w):
    """fp32 x . w^T as 64 lanes and a tree sum it."""
    T, H = x.shape
    n = (H + 63) // 64
    xp, wp = np.zeros((T, n * 64)), np.zeros((w.shape[0], n * 64))
    xp[:, :H], wp[:, :H] = x, w
    acc = np.zeros((T, w.shape[0], 64), dtype=np.float32)
    for i in range(n):
        s = slice(64 * i, 64 * i + 64)
        acc = (acc.astype(np.float64) + xp[:, None, s] * wp[None, :, s]).astype(np.float32)  # one rounding, as fma
    while acc.shape[-1] > 1:
        acc = acc[..., 0::2] + acc[..., 1::2]
    return acc[..., 0]


@pytest.mark.parametrize("H", [96, 256, 1000, 1022, 1024, 2048])
def test_router_rounding(gpu_lib, H):
    T, E = 64, 64
    g = torch.Generator().manual_seed(H)
    x, w = torch.randn((T, H), generator=g), torch.randn((E, H), generator=g) * 0.02
    logits, probs = torch.empty((T, E), device="cuda"), torch.empty((T, E), device="cuda")
    print("case", H, flush=True)
    lib.dmoe_router_logits(x.cuda(), w.cuda(), None, T, H, E, logits, probs)
    want = x.double().numpy() @ w.double().numpy().T
    err = np.linalg.norm(logits.cpu().double().numpy() - want)
    ref = np.linalg.norm(_lane_sums(x.numpy(), w.numpy()).astype(np.float64) - want)
    assert err <= 1.05 * ref, (err / np.linalg.norm(want), ref / np.linalg.norm(want))
