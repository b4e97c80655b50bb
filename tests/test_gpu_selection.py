"""The selection of the kernels with 16 elements per lane where a lane holds more of a block's smallest values than the
shortened columns keep, around the ranks at which its forms change, against the kernels with 8 per lane
(compared with the oracle elsewhere): the same inputs leave the same bytes.  And the selection in blocks of 2048 from the bound
that the old state gives, against the oracle."""
import numpy as np
import pytest

from parity_common import compare_step, flip_budget, make_cfgs
from test_gpu_both_forms import PIECE
from test_gpu_parity import GpuSide, dev, gpu  # noqa: F401
from test_gpu_table_forms import bits

pytestmark = pytest.mark.gpu


def crowded(n, B, gen):
    """Magnitudes of a gradient: rising along a block, falling, rising with ties, the smallest ones in one run of 16 (a lane's)
    or of 7, 8 and 9 of it, among larger scattered ones."""
    import torch
    at = torch.arange(n, device="cuda")
    i, kind, run = at % B, at // B % 8, (at // (8 * B)) % (B // 16)
    x = 1.0 + torch.rand(n, device="cuda", generator=gen)
    inside = i - 16 * run
    g = torch.where(kind == 0, 1.0 + i, torch.where(kind == 1, float(B) - i, torch.where(kind == 2, 1.0 + i // 5, 100 * x)))
    for k, many in ((3, 16), (4, 7), (5, 8), (6, 9)):
        g = torch.where((kind == k) & (inside >= 0) & (inside < many), x, g)
    return g * 1e-3


@pytest.mark.parametrize("B,rank", [(128, r) for r in (1, 2, 8, 9, 10, 11, 12, 13, 15, 16, 17, 18, 24)]
                         + [(64, r) for r in (1, 5, 6, 7, 8, 9, 10, 11, 12, 16)])
def test_crowded_lanes(gpu, B, rank):  # noqa: F811
    import torch
    n = (3 << 20) + 2048
    gen = torch.Generator(device="cuda").manual_seed(rank)
    p0 = torch.randn(n, device="cuda", generator=gen)
    cfg = gpu.make_config(2, 3, B, 1, quantile_p=(rank - 0.5) / B)
    sides = [(p0.clone(), gpu.SoloState(n, cfg).buffers()) for _ in range(2)]
    for step in (1, 2):
        g = (crowded(n, B, gen) * torch.sign(torch.randn(n, device="cuda", generator=gen))).to(torch.bfloat16)
        gpu.solo_adamw_step(sides[0][0], g, *sides[0][1], n, step, cfg)
        q, st = sides[1]
        for a in range(0, n, PIECE):
            part = (st[0][a // 16:], st[1][a // B:], st[2][a // 10:], st[3][a // B:], st[4][a // B:])
            gpu.solo_adamw_step(q[a:], g[a:], *part, min(PIECE, n - a), step, gpu.make_config(2, 3, B, 1, quantile_p=(rank - 0.5) / B, index_offset=a))
    torch.cuda.synchronize()
    for x, y in zip((sides[0][0], *sides[0][1]), (sides[1][0], *sides[1][1])):
        assert torch.equal(bits(x), bits(y))


@pytest.mark.parametrize("p", (0.05, 0.1, 0.3, 0.97))
@pytest.mark.parametrize("blocks,opt", [(5, "adamw"), (5, "adabelief"), (1027, "adamw")])
def test_bound_of_the_old_state(so, gpu, blocks, opt, p):  # noqa: F811
    """Late step numbers on a state (the bound is used then): quantiles right above the bound, beyond the first pass's
    quarter octave (gradients that jump), on it (idle blocks), and blocks that have no state yet."""
    from paper_2505_00347_amd import synth
    n = blocks * 2048 + 77
    oc, gc = make_cfgs(so, gpu, 2, 3, 2048, False, p=p, optimizer=opt, eps=1e-12 if opt == "adabelief" else 1e-8)
    rng = np.random.default_rng(blocks)
    kind = np.arange(n) // 2048 % 5
    prm, st = synth.make_params(n), so.State(n, oc)
    side = GpuSide(gpu, n, gc)
    flips = 0
    for k, step in enumerate((1, 8, 60, 1000, 1001)):
        x = rng.standard_normal(n).astype(np.float32) * np.float32(1e-3)
        g = np.where(kind == 1, x * (k == 0), np.where(kind == 2, x * 1000.0 ** (k % 2), np.where(kind == 3, x * (k >= 3), x))).astype(np.float32)
        side.load(prm, st)
        side.step(dev(g), step)
        before = prm.astype(np.float64)
        margin = so.step_packed(prm, g, st, step, oc, want_margin=True, threads=8)
        flips += compare_step(so, oc, n, prm, st, margin, side.fetch(), 1e-6, 2e-6 * oc.lr, p_before=before)
    assert flips <= flip_budget(5 * n)
