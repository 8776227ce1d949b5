"""One-call routing at the sizes where its launches change, bit for bit against
the separate entry points: schedules of one round of entries and more
(512), blocks below and above the LDS limit of a routing workgroup, ragged
last workgroups, odd expert counts.  Three eager calls on one set of buffers
and three replays of a captured graph, with other work between them, each on
other hidden states; the work items are compared too."""
import pytest
import torch

from dmoe_synth import get_config, make_inputs
from paper_2605_30876_amd.layer import MoELayer

pytestmark = pytest.mark.gpu

TOKEN = [dict(E=256, k=8, NB=1, bs=32), dict(E=256, k=8, NB=2, bs=32), dict(E=256, k=8, NB=5, bs=13), dict(E=257, k=8, NB=1, bs=32), dict(E=48, k=4, NB=1, bs=64),
         dict(E=48, k=5, NB=4, bs=13), dict(E=16, k=1, NB=7, bs=3), dict(E=9, k=9, NB=3, bs=9)]
BLOCK = [dict(E=64, k=8, NB=2, bs=5), dict(E=64, k=8, NB=64, bs=4), dict(E=64, k=8, NB=65, bs=4),
         dict(E=256, k=8, NB=3, bs=64), dict(E=256, k=8, NB=2, bs=72), dict(E=256, k=8, NB=2, bs=80),
         dict(E=300, k=17, NB=5, bs=24), dict(E=512, k=3, NB=6, bs=9),
         # both sides of the lines between one workgroup per block and separate launches
         dict(E=219, k=8, NB=3, bs=16), dict(E=219, k=8, NB=3, bs=17), dict(E=219, k=8, NB=6, bs=64),
         dict(E=301, k=5, NB=2, bs=8), dict(E=301, k=5, NB=2, bs=9), dict(E=301, k=5, NB=1, bs=16),
         dict(E=301, k=5, NB=1, bs=17), dict(E=101, k=4, NB=1, bs=32), dict(E=101, k=4, NB=1, bs=33),
         dict(E=128, k=6, NB=4, bs=32), dict(E=128, k=6, NB=4, bs=33), dict(E=128, k=6, NB=1, bs=64),
         dict(E=128, k=6, NB=1, bs=65), dict(E=192, k=8, NB=2, bs=64), dict(E=192, k=8, NB=2, bs=65),
         dict(E=188, k=8, NB=2, bs=33)]


def _snapshot(m, routing, rows):
    s = m.sched
    n, nw = int(s.n_unique[0]), int(s.n_work[0])
    return [m.probs, m.combine_w, m.experts(routing), m.gaps(routing), s.n_unique[:1], s.n_work[:1], s.unique[:n],
            s.offsets[:n + 1], s.row_token[:rows], s.row_slot[:rows], s.work[:nw]]


@pytest.mark.parametrize("routing,over", [(r, o) for r in ("token", "topp") for o in TOKEN] +
                         [("block", o) for o in BLOCK])
def test_routing_launch_sizes(gpu_lib, routing, over):
    cfg = get_config("small_bf16").with_(name="rs", H=256, I=128, I_s=0, **over)
    print("case", routing, over, flush=True)
    mk = lambda: MoELayer(cfg.H, cfg.E, cfg.I, cfg.I_s, cfg.k, cfg.NB, cfg.bs, device="cuda")  # noqa: E731
    fused, chain = mk(), mk()
    rows = cfg.T * cfg.k
    ds = [make_inputs(cfg, seed=s, device="cuda") for s in range(4)]
    wr = ds[0]["w_router"]
    x = ds[0]["x"].clone()

    def check():
        torch.cuda.synchronize()
        chain.route(x, wr, None, routing, fused=False)
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(zip(_snapshot(fused, routing, rows), _snapshot(chain, routing, rows))):
            assert torch.equal(a, b), i

    for t in (fused.sched.n_work, fused.sched.work, fused.sched.row_token):
        t.fill_(-7)
    for d in ds[:3]:
        x.copy_(d["x"])
        fused.route(x, wr, None, routing, fused=True)
        check()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        fused.route(x, wr, None, routing, fused=True)
    for d in (ds[3], ds[1], ds[2]):
        x.copy_(d["x"])
        fused.sched.n_work.fill_(3)
        g.replay()
        check()


@pytest.mark.parametrize("E,NB,bs", [(161, 2, 40), (161, 2, 41), (161, 1, 64), (161, 1, 65), (128, 3, 64), (128, 3, 65)])
def test_block_routing_launch_sizes_f32(gpu_lib, E, NB, bs):
    """The fp32 lines between one workgroup per block and separate launches."""
    cfg = get_config("small_f32").with_(name="rs32", H=96, E=E, I=16, I_s=0, k=5, NB=NB, bs=bs)
    print("case", E, NB, bs, flush=True)
    mk = lambda: MoELayer(cfg.H, cfg.E, cfg.I, cfg.I_s, cfg.k, cfg.NB, cfg.bs, dtype=torch.float32, device="cuda")  # noqa: E731
    fused, chain = mk(), mk()
    for seed in (0, 1):
        d = make_inputs(cfg, seed=seed, device="cuda")
        fused.route(d["x"], d["w_router"], None, "block", fused=True)
        chain.route(d["x"], d["w_router"], None, "block", fused=False)
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(zip(_snapshot(fused, "block", cfg.T * cfg.k), _snapshot(chain, "block", cfg.T * cfg.k))):
            assert torch.equal(a, b), i
