"""The decode kernels over items of several passes (popular experts under a
Zipf bias, the shared expert's rows): the one-tile kernels, whose workgroups
run all 16-row passes of an item over a down slice of five to eight K-steps,
of four, and of both (routed and shared experts of different widths); the two-
and four-tile kernels, one pass per workgroup, at hidden sizes that leave the
down projection's last eight tiles half empty.  Against the CPU oracle, bf16
tolerance (2e-2 of the output's RMS)."""
import pytest
import torch

from dmoe_synth import get_config, make_inputs
from paper_2605_30876_amd.layer import MoELayer
from parity import run_and_check, run_and_check_topp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("routing", ["token", "topp"])
@pytest.mark.parametrize("I,I_s", [(1024, 1024), (640, 0), (768, 512), (512, 1024), (512, 512)])
@pytest.mark.parametrize("nb,bs", [(2, 32), (4, 27)])
def test_one_tile_passes(gpu_lib, routing, I, I_s, nb, bs):
    cfg = get_config("small_bf16").with_(name="passes", H=256, E=64, I=I, I_s=I_s, k=4, NB=nb, bs=bs, bias="zipf")
    print("case", routing, I, I_s, nb, bs, flush=True)
    d = {k: (None if v is None else v.cuda()) for k, v in make_inputs(cfg, seed=9).items()}
    m = MoELayer(cfg.H, cfg.E, cfg.I, cfg.I_s, cfg.k, cfg.NB, cfg.bs, device="cuda")
    if routing == "topp":
        run_and_check_topp(cfg, d, m)
    else:
        run_and_check(cfg, d, routing, m)
    assert int(m.sched.work[:int(m.sched.n_work[0]), 2].max()) > 16  # an item of several passes


# rows per item decide the tile count: blocks of 24 and 32 take two tiles, of
# 64 four (few enough weight tiles that the tile kernels stay out)
@pytest.mark.parametrize("H,I,I_s", [(384, 128, 128), (2176, 128, 0), (1152, 256, 384)])
@pytest.mark.parametrize("nb,bs", [(3, 32), (6, 24), (5, 27), (3, 64)])
def test_split_passes(gpu_lib, H, I, I_s, nb, bs):
    cfg = get_config("small_bf16").with_(name="split", H=H, E=24, I=I, I_s=I_s, k=4, NB=nb, bs=bs, bias="zipf")
    print("case", H, I, I_s, nb, bs, flush=True)
    d = {k: (None if v is None else v.cuda()) for k, v in make_inputs(cfg, seed=10).items()}
    m = MoELayer(cfg.H, cfg.E, cfg.I, cfg.I_s, cfg.k, cfg.NB, cfg.bs, device="cuda")
    run_and_check(cfg, d, "block", m)
    assert int(m.sched.work[:int(m.sched.n_work[0]), 2].max()) > 32
