"""fp32 layers at the edges of their matrix-core tiles: reductions that 16
does not divide, units that 4 or 16 do not divide, items of more than one pass
(32 rows), wide (64-unit) and narrow (16-unit) workgroups, and a router whose
rows are not 16-byte aligned.  Against the CPU oracle (float64 FFN); tolerance
of every fp32 layer, 1e-4 of the output's RMS."""
import numpy as np
import pytest
import torch

import oracle as O
from dmoe_synth import get_config, make_inputs
from paper_2605_30876_amd import lib
from paper_2605_30876_amd.layer import MoELayer
from parity import run_and_check

pytestmark = pytest.mark.gpu

SHAPES = {
    "one_chunk": dict(H=4, E=3, I=1, I_s=1, k=2, NB=2, bs=3),
    "odd_units": dict(H=100, E=7, I=37, I_s=0, k=3, NB=1, bs=17),
    "odd_shared": dict(H=36, E=5, I=20, I_s=21, k=2, NB=3, bs=11),
    "wide_ragged": dict(H=260, E=24, I=604, I_s=596, k=4, NB=2, bs=33),
    "many_rows": dict(H=68, E=4, I=64, I_s=40, k=2, NB=5, bs=64),
    "wide_pieces": dict(H=512, E=40, I=448, I_s=448, k=2, NB=9, bs=40),
    # wide down workgroups over activation rows that are not 16-byte aligned
    "wide_down_odd": dict(H=2048, E=8, I=37, I_s=0, k=2, NB=4, bs=8),
}

# Token routing over more than 128 MiB of weights (non-temporal loads): narrow
# and wide workgroups of both kernels, aligned and unaligned activation rows,
# items of one pass and (popular experts, the shared expert) of several.
STREAM = {
    "odd_units": dict(H=2048, E=48, I=201, I_s=201, k=4, NB=4, bs=20),
    "narrow": dict(H=128, E=64, I=1400, I_s=1400, k=4, NB=1, bs=16),
    "narrow_odd": dict(H=128, E=64, I=1401, I_s=1401, k=4, NB=1, bs=16),
    "passes": dict(H=512, E=48, I=604, I_s=604, k=4, NB=4, bs=20),
}


@pytest.mark.parametrize("routing", ["block", "token"])
@pytest.mark.parametrize("name", list(SHAPES))
def test_f32_layer_edges(gpu_lib, name, routing):
    cfg = get_config("small_f32").with_(name="f32_" + name, bias="none", **SHAPES[name])
    print("case", name, routing, flush=True)
    d = {k: (None if v is None else v.cuda()) for k, v in make_inputs(cfg, seed=5).items()}
    m = MoELayer(cfg.H, cfg.E, cfg.I, cfg.I_s, cfg.k, cfg.NB, cfg.bs, dtype=torch.float32, device="cuda")
    run_and_check(cfg, d, routing, m)


@pytest.mark.parametrize("name", list(STREAM))
def test_f32_layer_streaming(gpu_lib, name):
    cfg = get_config("small_f32").with_(name="f32_stream_" + name, bias="zipf", **STREAM[name])
    print("case", name, flush=True)
    d = {k: (None if v is None else v.cuda()) for k, v in make_inputs(cfg, seed=11).items()}
    m = MoELayer(cfg.H, cfg.E, cfg.I, cfg.I_s, cfg.k, cfg.NB, cfg.bs, dtype=torch.float32, device="cuda")
    assert (m.max_work("token") + 1) * 3 * cfg.H * max(cfg.I, cfg.I_s) * 4 > 128 << 20
    run_and_check(cfg, d, "token", m)
    if cfg.T > 32:
        assert int(m.sched.work[:int(m.sched.n_work[0]), 2].max()) > 32  # an item of several passes


@pytest.mark.parametrize("T,H,E", [(1, 1, 1), (16, 16, 16), (17, 33, 19), (5, 130, 300), (40, 1024, 33)])
def test_f32_router_edges(gpu_lib, T, H, E):
    g = torch.Generator().manual_seed(T * 7 + H + E)
    x, w = torch.randn((T, H), generator=g), torch.randn((E, H), generator=g) * 0.1
    logits, probs = torch.empty((T, E), device="cuda"), torch.empty((T, E), device="cuda")
    print("case", T, H, E, flush=True)
    lib.dmoe_router_logits(x.cuda(), w.cuda(), None, T, H, E, logits, probs)
    want = x.double().numpy() @ w.double().numpy().T
    # H products summed in fp32 in any order: at most (H + 1) roundings of the absolute sum
    bound = (H + 1) * 2.0 ** -23 * (np.abs(x.numpy()) @ np.abs(w.numpy()).T) + 1e-12
    assert (np.abs(logits.cpu().numpy() - want) <= bound).all()
    np.testing.assert_allclose(probs.cpu().numpy(), O.softmax_rows(want.astype(np.float32)), atol=1e-6)
