"""The tile kernels' launch shapes that larger forwards take: wide gate/up
workgroups (256 weight rows) over items of every even token-tile count, and
wide down workgroups over a hidden size that leaves the last one half empty
(H % 256 == 128).  Against the CPU oracle, bf16 tolerance (2e-2 of the
output's RMS), scaled-half and float32 slot outputs."""
import pytest
import torch

from dmoe_synth import get_config, make_inputs
from paper_2605_30876_amd.layer import MoELayer
from parity import run_and_check

pytestmark = pytest.mark.gpu

SHAPES = {
    # 172 grid items x 8 wide row blocks; blocks of 24: items of 8 to 128 rows
    "wide_gateup": dict(H=384, E=64, I=1024, I_s=1024, k=8, NB=64, bs=24),
    # 472 grid items x 9 wide row blocks of the down projection (the last half empty)
    "wide_down": dict(H=2176, E=256, I=128, I_s=128, k=8, NB=96, bs=32),
}


@pytest.mark.parametrize("slots", ["f16s", "f32"])
@pytest.mark.parametrize("routing", ["block", "token"])
@pytest.mark.parametrize("name", list(SHAPES))
def test_wide_tile_workgroups(gpu_lib, name, routing, slots):
    cfg = get_config("small_bf16").with_(name=name, **SHAPES[name])
    print("case", name, routing, slots, flush=True)
    d = {k: (None if v is None else v.cuda()) for k, v in make_inputs(cfg, seed=4).items()}
    m = MoELayer(cfg.H, cfg.E, cfg.I, cfg.I_s, cfg.k, cfg.NB, cfg.bs, device="cuda", slot_format=slots)
    run_and_check(cfg, d, routing, m)


@pytest.mark.parametrize("n", [128, 256, 384, 512, 640])
@pytest.mark.parametrize("nb", [16, 64])
def test_ring_ends(gpu_lib, n, nb):
    """Both products of 2 to 10 two-step stages (4 to 20 one-step ones where
    the grid takes wide workgroups): every remainder of the three-stage trips."""
    cfg = get_config("small_bf16").with_(name="ring", H=n, E=64, I=n, I_s=n, k=8, NB=nb, bs=48)
    print("case", n, nb, flush=True)
    d = {k: (None if v is None else v.cuda()) for k, v in make_inputs(cfg, seed=8).items()}
    m = MoELayer(cfg.H, cfg.E, cfg.I, cfg.I_s, cfg.k, cfg.NB, cfg.bs, device="cuda")
    run_and_check(cfg, d, "block", m, sample_tokens=list(range(0, cfg.T, 7)))
