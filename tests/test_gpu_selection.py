"""The selection of the kernels with 16 elements per lane where a lane holds more of a block's smallest values than the
shortened columns keep, around the ranks at which its forms change, against the kernels with 8 per lane
(compared with the oracle elsewhere): the same inputs leave the same bytes."""
import pytest

from test_gpu_both_forms import PIECE
from test_gpu_parity import gpu  # noqa: F401
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
