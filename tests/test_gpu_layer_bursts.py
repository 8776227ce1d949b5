"""The one-block layer at hidden sizes that take each of its gate/up bursts
(one or several of 2, 4, 6, 7, 8, 10 and 16 K-steps per wave, and the bursts
of up to 16 with a shorter last one that 12, 22, 26, 28 and 30 steps take),
one and two token tiles, with and without a router bias and a shared expert.
Against the CPU oracle, bf16 tolerance (2e-2 of the output's RMS)."""
import pytest
import torch

from dmoe_synth import get_config, make_inputs
from paper_2605_30876_amd.layer import MoELayer, pack_weights
from parity import run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bs,bias,I_s", [(32, "none", 128), (7, "zipf", 0), (16, "zipf", 256)])
@pytest.mark.parametrize("H", [256, 512, 768, 1024, 1280, 1536, 1792, 2048, 2304, 2560, 2816, 3072, 3328, 3584, 3840,
                               4096])
def test_one_block_layer_bursts(gpu_lib, H, bs, bias, I_s):
    cfg = get_config("small_bf16").with_(name="bursts", H=H, E=20, I=128, I_s=I_s, k=3, NB=1, bs=bs, bias=bias)
    print("case", H, bs, bias, I_s, flush=True)
    d = {k: (None if v is None else v.cuda()) for k, v in make_inputs(cfg, seed=6).items()}
    m = MoELayer(cfg.H, cfg.E, cfg.I, cfg.I_s, cfg.k, cfg.NB, cfg.bs, device="cuda")
    assert m.fused("block")
    run_and_check(cfg, d, "block", m)
    # the one-call layer against the chain: same selection, y within the
    # rounding of the activations (2^-9 of each) and of the slots
    w = pack_weights(d)
    y = m.forward(d["x"], w, "block").clone()
    experts = m.block_experts.clone()
    yc = m.forward(d["x"], w, "block", chained=True).clone()
    torch.cuda.synchronize()
    assert torch.equal(experts, m.block_experts)
    assert float((y - yc).abs().max()) <= 2e-2 * float(yc.square().mean().sqrt())
