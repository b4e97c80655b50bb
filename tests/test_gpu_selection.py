"""The selection of the kernels with 8 elements per lane at the ranks where its form changes, against the oracle.  That of the kernels with 16 elements per lane where a lane holds more of a block's smallest values than the
shortened columns keep, around the ranks at which its forms change, against the kernels with 8 per lane
(compared with the oracle elsewhere): the same inputs leave the same bytes.  And the selection in blocks of 2048 from the bound
that the old state gives, against the oracle."""
import numpy as np
import pytest

from parity_common import compare_step, flip_budget, make_cfgs
from test_dispatch_lines import QUAD_BLOCKS, last8
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
    n = last8(True, rank=rank) + 2048
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


def ordered(n, B, rng):
    """Magnitudes by block: scattered, rising, falling, ties, equal, the smallest ones in one run of 8 (a lane's), or spread
    one to a run, mostly zero, a wide range."""
    i, block = np.arange(n) % B, np.arange(n) // B
    x = 1.0 + rng.random(n)
    kinds = (x, 1.0 + i, float(B) - i, 1.0 + i // 5, np.ones(n), np.where(i // 8 == block % (B // 8), x, 100 * x),
             np.where(i % 8 == block % 8, x, 100 * x), np.where(rng.random(n) < 0.9, 0.0, x), x * 10.0 ** rng.integers(-9, 3, n))
    return np.choose(block % len(kinds), kinds) * np.where(rng.random(n) < 0.5, -1e-3, 1e-3)


@pytest.mark.parametrize("bf16", (False, True))
@pytest.mark.parametrize("B,rank", [(128, r) for r in (1, 2, 7, 8, 9, 13, 15, 16, 17, 32, 39, 63, 64, 65, 100, 127, 128)]
                         + [(64, r) for r in (1, 2, 7, 8, 9, 15, 16, 17, 33, 63, 64)])
def test_merged_lists(so, gpu, B, rank, bf16):  # noqa: F811
    """8 per lane: the ranks at which the length of the merged lists changes, full blocks and a shorter last one."""
    rng = np.random.default_rng(rank)
    flips = total = 0
    for n in (48 * 128 + 77, 48 * 128 + B // 2, 5):
        oc, gc = make_cfgs(so, gpu, 2, 3, B, bf16, p=(rank - 0.5) / B)
        prm, st = rng.standard_normal(n).astype(np.float32), so.State(n, oc)
        side = GpuSide(gpu, n, gc)
        for step in (1, 2, 3):
            g = ordered(n, B, rng).astype(np.float32)
            if bf16:
                g = (g.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
            side.load(prm, st)
            side.step(dev((g.view(np.uint32) >> 16).astype(np.uint16)) if bf16 else dev(g), step)
            before = prm.astype(np.float64)
            margin = so.step_packed(prm, g, st, step, oc, want_margin=True)
            flips += compare_step(so, oc, n, prm, st, margin, side.fetch(), 1e-6, 2e-6 * oc.lr, p_before=before)
            total += n
    assert flips <= flip_budget(total)


# Forms of a launch over blocks of 2048: four wavefronts per block or two, flat or a table, plain or with the variants
# (a table of the buffer alone has few blocks; "large table": with a second tensor of many)
FORMS = [(5, 2, 3, "flat", {}), (5, 2, 3, "flat", dict(optimizer="adabelief")), (QUAD_BLOCKS + 3, 2, 3, "flat", {}),
         (QUAD_BLOCKS + 3, 3, 3, "flat", dict(de=True, bf16=True)), (QUAD_BLOCKS + 3, 4, 2, "flat", dict(optimizer="adabelief", mp=True)),
         (QUAD_BLOCKS + 3, 2, 4, "flat", dict(optimizer="adam_l2", de=True)), (5, 4, 3, "flat", dict(de=True, bf16=True, mp=True)),
         (6, 2, 3, "table", dict(bf16=True)), (6, 4, 4, "table", dict(de=True, optimizer="adabelief", mp=True)),
         (6, 3, 2, "large table", dict(bf16=True)), (6, 4, 3, "large table", dict(de=True, mp=True, optimizer="adabelief"))]


def sides(so, gpu, n, bm, bv, launch, p, optimizer="adamw", de=False, bf16=False, mp=False):  # noqa: F811
    """The oracle's config and state, and the GPU's side with a step(gradients, step)."""
    from paper_2505_00347_amd import synth
    scale = 0.5 if mp else None
    oc, gc = make_cfgs(so, gpu, bm, bv, 2048, bf16, p=p, optimizer=optimizer, de=de, grad_scale=scale,
                       eps=1e-12 if optimizer == "adabelief" else 1e-8)
    side = GpuSide(gpu, n, gc, scale, mp, launch == "large table")

    def step(g, k):
        x = dev((g.view(np.uint32) >> 16).astype(np.uint16)) if bf16 else dev(g)
        if launch == "table":
            gpu.SoloMultiTable([(side.p, x, side.state, side.p_bf16)], gc).step(k, grad_scale=side.grad_scale)
        else:
            side.step(x, k)

    def gradients(x):
        x = x.astype(np.float32)
        return (x.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32) if bf16 else x

    return oc, synth.make_params(n), so.State(n, oc), side, step, gradients


@pytest.mark.parametrize("p", (0.05, 0.1, 0.3, 0.97))
@pytest.mark.parametrize("blocks,bm,bv,launch,more", FORMS)
def test_bound_of_the_old_state(so, gpu, blocks, bm, bv, launch, more, p):  # noqa: F811
    """Late step numbers on a state (the bound is used then): quantiles right above the bound, beyond the first pass's
    quarter octave (gradients that jump), on it (idle blocks), and blocks that have no state yet."""
    n = blocks * 2048 + 77
    oc, prm, st, side, step, gradients = sides(so, gpu, n, bm, bv, launch, p, **more)
    rng = np.random.default_rng(blocks)
    kind = np.arange(n) // 2048 % 5
    flips = 0
    for k, late in enumerate((1, 8, 60, 1000, 1001)):
        x = rng.standard_normal(n).astype(np.float32) * np.float32(1e-3)
        g = gradients(np.where(kind == 1, x * (k == 0), np.where(kind == 2, x * 1000.0 ** (k % 2), np.where(kind == 3, x * (k >= 3), x))))
        side.load(prm, st)
        step(g, late)
        before = prm.astype(np.float64)
        margin = so.step_packed(prm, g, st, late, oc, want_margin=True, threads=8)
        flips += compare_step(so, oc, n, prm, st, margin, side.fetch(), 1e-6, 2e-6 * oc.lr, p_before=before)
        side.check_bf16_copy(so)
    assert flips <= flip_budget(5 * n)


@pytest.mark.parametrize("blocks,bm,bv,launch,more", [f for f in FORMS if f[4].get("optimizer") != "adam_l2"])
def test_late_non_finite_gradients_stay_inside_their_blocks(so, gpu, blocks, bm, bv, launch, more):  # noqa: F811
    """A NaN or an infinity in the gradient of a late step, and the step after it, whose bound comes from what that left of
    the block's scale and base: every other block equals the oracle's, which has neither."""
    n = blocks * 2048 + 77
    oc, prm, st, side, step, gradients = sides(so, gpu, n, bm, bv, launch, 0.1, **more)
    rng = np.random.default_rng(bm)
    for late in (1, 2, 999):
        so.step_packed(prm, gradients(rng.standard_normal(n) * 1e-3), st, late, oc, threads=8)
    side.load(prm, st)
    spoiled = np.zeros(-(-n // 2048), bool)
    for k, late in enumerate((1000, 1001)):
        g = gradients(rng.standard_normal(n) * 1e-3)
        dirty = g.copy()
        if k == 0:
            bad = rng.choice(4 * 2048, 12, replace=False)        # of the first four blocks
            bad = np.concatenate([bad, bad[:1] + (blocks - 4) // 2 * 2048 + 2048])
            dirty[bad[:4]], dirty[bad[4:8]], dirty[bad[8:]] = np.nan, np.inf, -np.inf
            spoiled[bad // 2048] = True
        step(dirty, late)
        before = prm.astype(np.float64)
        margin = so.step_packed(prm, g, st, late, oc, want_margin=True, threads=8)
        tainted = spoiled.copy()
        flips = compare_step(so, oc, n, prm, st, margin, side.fetch(), 1e-5, 1e-5 * oc.lr, tainted, p_before=before)
        assert flips <= flip_budget(n) and (tainted & ~spoiled).sum() <= flips
        spoiled = tainted
    assert not spoiled.all()
