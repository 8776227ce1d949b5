"""The fp32 shared expert at sizes where a lane's weight offset passes 32 bits
(an index of reduction step 12 and up times two matrices of 200 million
units), and where the units take more than one launch.  The weights are zero
except at a few units, the first and the last among them; the expected output
is the float64 formula over those.  Tolerance: fp32 products and sums of at
most 16 + 4 terms, expf within a few ulp: 1e-5."""
import pytest
import torch

from paper_2605_30876_amd import lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,I", [(16, 200_000_000), (4, 280_000_001)])
def test_wide_shared_expert(gpu_lib, H, I):
    print("case", H, I, flush=True)
    g = torch.Generator().manual_seed(I)
    units = [0, 1, 134_217_728, 134_217_727, I // 3, I - 2, I - 1]
    x = torch.randn((1, H), generator=g)
    wg, wu, wd = (torch.randn((len(units), H), generator=g) for _ in range(3))
    w13 = torch.zeros((H, 2 * I), device="cuda")
    w2 = torch.zeros((I, H), device="cuda")
    for n, u in enumerate(units):
        w13[:, u] = wg[n].cuda()
        w13[:, I + u] = wu[n].cuda()
        w2[u] = wd[n].cuda()
    y = torch.full((1, H), float("nan"), device="cuda")
    ws = torch.empty((lib.dmoe_shared_ffn_workspace_size(1, I, lib.DMOE_F32),), dtype=torch.uint8, device="cuda")
    lib.dmoe_shared_expert_ffn(x.cuda().reshape(-1), w13, w2, 1, H, I, y, ws)
    torch.cuda.synchronize()
    a, b = wg.double() @ x[0].double(), wu.double() @ x[0].double()
    want = (a / (1 + torch.exp(-a)) * b) @ wd.double()
    err = float((y.cpu().double()[0] - want).abs().max() / want.square().mean().sqrt())
    del w13, w2, ws
    torch.cuda.empty_cache()
    assert err <= 1e-5, err
