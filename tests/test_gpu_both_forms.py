"""Every instantiation of the kernels with 16 elements per lane against those with 8, which the other GPU tests
compare with the oracle: the same inputs leave the same bytes.  A flat buffer in one call runs the first, in
pieces of 2,560,000 elements the second; a table of five million elements the first, its tensors one by one the second."""
import math

import pytest

from test_dispatch_lines import PIECES8, last8
from test_gpu_parity import gpu  # noqa: F401
from test_gpu_table_forms import bits, table_against_flat

pytestmark = pytest.mark.gpu

FORMATS = [(bm, bv, B) for B in (64, 128) for bm in (2, 3, 4) for bv in (2, 3, 4)]
PIECE = 2560000                     # whole blocks and code words, below every size that runs 16 per lane
ENDS = [0, 1, 511, 512, 513, 1023, 80, 8, 700]


def gradients(n, B, gen, dtype):
    """One kind per block: scattered, outliers, mostly zero, few values, equal, single, all zero, a wide range."""
    import torch
    x = torch.randn(n, device="cuda", generator=gen)
    u = torch.rand(n, device="cuda", generator=gen)
    at = torch.arange(n, device="cuda")
    kind = at // B % 8
    g = x.clone()
    for k, y in ((1, torch.where(u < 0.01, 100 * x, x)), (2, torch.where(u < 0.9, 0.0, x)), (3, x.round()),
                 (4, torch.ones_like(x)), (5, (at % B == 5).float()), (6, torch.zeros_like(x)), (7, x * 10.0 ** (15 * u - 12))):
        g = torch.where(kind == k, y, g)
    return (g * 1e-3).to(dtype)


@pytest.mark.parametrize("ext", (False, True))
@pytest.mark.parametrize("de", (False, True))
@pytest.mark.parametrize("bf16", (False, True))
@pytest.mark.parametrize("k,bm,bv,B", [(k, *f) for k, f in enumerate(FORMATS)])
def test_flat(gpu, k, bm, bv, B, bf16, de, ext):  # noqa: F811
    import torch
    dtype = torch.bfloat16 if bf16 else torch.float32
    for j, p in enumerate((0.1, 0.45)):
        n = last8(bf16, ext, math.ceil(p * B)) + 2048 + ENDS[(2 * k + j) % len(ENDS)]
        flags = 1 | (2 if de else 0) | ((4, 8)[j] if ext else 0)          # AdaBelief, coupled decay
        off = 8 * ((1 << 32) - 700)

        def config(offset):
            return gpu.make_config(bm, bv, B, 1 if bf16 else 0, flags=flags, quantile_p=p, index_offset=offset)

        gen = torch.Generator(device="cuda").manual_seed(k)
        p0 = torch.randn(n, device="cuda", generator=gen)
        scale = torch.tensor([0.5], device="cuda") if ext else None
        sides = [(p0.clone(), torch.zeros(n, dtype=torch.bfloat16, device="cuda") if ext else None,
                  gpu.SoloState(n, config(off)).buffers()) for _ in range(2)]
        for step in (1, 2, 3):
            g = gradients(n, B, gen, dtype)
            q, h, st = sides[0]
            gpu.solo_adamw_step_mp(q, h, g, scale, *st, n, step, config(off))
            q, h, st = sides[1]
            for a in range(0, n, PIECE):
                part = (st[0][a // (32 // bm):], st[1][a // B:], st[2][a // (32 // bv):], st[3][a // B:], st[4][a // B:])
                gpu.solo_adamw_step_mp(q[a:], None if h is None else h[a:], g[a:], scale, *part, min(PIECE, n - a), step,
                                       config(off + a))
        torch.cuda.synchronize()
        for x, y in zip((sides[0][0], sides[0][1], *sides[0][2]), (sides[1][0], sides[1][1], *sides[1][2])):
            assert x is None or torch.equal(bits(x), bits(y)), (p, n)


@pytest.mark.parametrize("ext", (False, True))
@pytest.mark.parametrize("de", (False, True))
@pytest.mark.parametrize("bf16", (False, True))
@pytest.mark.parametrize("k,bm,bv,B", [(k, *f) for k, f in enumerate(FORMATS)])
def test_table(gpu, k, bm, bv, B, bf16, de, ext):  # noqa: F811
    ends = ENDS[k % len(ENDS):] + ENDS[:k % len(ENDS)]
    sizes = [1800 * 1024 + ends[0], 1, 5120 + ends[1], 2560, 2400 * 1024 + ends[2], 7680 + ends[3], 1200 * 1024 + ends[4], 77]
    assert all(n <= PIECE for n in sizes) and sum(n // 1024 for n in sizes) > PIECES8
    table_against_flat(gpu, sizes, bm, bv, B, bf16, de, flags=4 if ext else 0, mp=ext, p=(0.1, 0.3)[k % 2], steps=3)
