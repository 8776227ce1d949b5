"""The one-tile decode kernels over items of several 16-row passes: a wave's
down slice of five to eight K-steps (held in registers from pass to pass), of
four, and of both (routed and shared experts of different widths).  Popular
experts (Zipf bias) collect many rows, the shared expert all tokens.  Against
the CPU oracle, bf16 tolerance (2e-2 of the output's RMS)."""
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
