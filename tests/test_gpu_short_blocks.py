"""GPU parity of blocks of 2048, full and short: up to QUAD_BLOCKS blocks of a launch run on four wavefronts with 8
elements per lane, more on two with 16.  The first form against the oracle (same bar as
test_gpu_parity.py), the second against the first, byte for byte, and against the oracle on a few buffers."""
import numpy as np
import pytest

from parity_common import compare_step, flip_budget, make_cfgs
from test_dispatch_lines import QUAD_BLOCKS
from test_gpu_parity import GpuSide, dev, gpu, run_teacher_forced  # noqa: F401
from test_gpu_table_forms import table_against_flat

pytestmark = pytest.mark.gpu

B = 2048
# ends inside a 16-byte vector, a lane's share of 8 and of 16, a code word of 8, 10 and 16, a wavefront's share
# of 512 and of 1024; as many keys as are compared at once, one less and one more
ENDS = [1, 3, 7, 8, 15, 17, 31, 32, 33, 80, 100, 511, 512, 513, 700, 1000, 1023, 1024, 1025, 1030, 1536, 2033, 2046, 2047]
FORMATS = [(bm, bv) for bm in (2, 3, 4) for bv in (2, 3, 4)]


@pytest.mark.parametrize("de", (False, True))
@pytest.mark.parametrize("k,bm,bv", [(k, *f) for k, f in enumerate(FORMATS)])
def test_every_end(so, gpu, k, bm, bv, de):  # noqa: F811
    for j, end in enumerate(ENDS):
        for n in (end, 2 * B + end):
            ext = dict(grad_scale=0.5, bf16_copy=True) if (j + k) % 3 == 0 else {}
            opt = ("adamw", "adamw", "adam_l2", "adabelief")[(j + k) % 4]
            run_teacher_forced(so, gpu, n, bm, bv, B, bf16=(j + k) % 2 == 0, steps=2, seed0=100 * k + j, de=de, optimizer=opt,
                               eps=1e-12 if opt == "adabelief" else 1e-8, **ext)


@pytest.mark.parametrize("p", (0.0, 0.1, 0.5, 0.97))
@pytest.mark.parametrize("bm,bv,n", [(2, 3, 1000), (4, 4, 2047), (3, 2, 33), (2, 2, 513)])
def test_selection_of_a_short_block(so, gpu, bm, bv, n, p):  # noqa: F811
    """The quantile by four wavefronts over scattered values, clusters, equal values, zeros and magnitudes far
    below the maximum."""
    from paper_2505_00347_amd import synth
    rng = np.random.default_rng(n)
    flips = total = 0
    for kind in range(7):
        oc, gc = make_cfgs(so, gpu, bm, bv, B, False, p=p, off=8 * 77)
        prm, st = synth.make_params(n), so.State(n, oc)
        side = GpuSide(gpu, n, gc)
        for step in (1, 2, 3):
            x = rng.standard_normal(n)
            g = (x, np.ones(n), np.where(rng.random(n) < 0.9, 0.0, x), np.rint(x), x * 10.0 ** rng.integers(-12, 3, n),
                 np.where(rng.random(n) < 0.01, 100 * x, x), np.zeros(n))[kind].astype(np.float32) * np.float32(1e-3)
            side.load(prm, st)
            side.step(dev(g), step)
            before = prm.astype(np.float64)
            margin = so.step_packed(prm, g, st, step, oc, want_margin=True)
            flips += compare_step(so, oc, n, prm, st, margin, side.fetch(), 1e-6, 2e-6 * oc.lr, p_before=before)
            total += n
    assert flips <= flip_budget(total)


def block_kinds(n, rng):
    """Gradients of one kind per block: scattered, outliers, mostly zero, few values, equal, single, all zero, a
    wide range of magnitudes."""
    x = rng.standard_normal(n)
    at = np.arange(n)
    kind = at // B % 8
    g = np.select([kind == k for k in range(8)], [
        x, np.where(rng.random(n) < 0.01, 100 * x, x), np.where(rng.random(n) < 0.9, 0.0, x), np.rint(x), np.ones(n),
        np.where(at % B == 5, 1.0, 0.0), np.zeros(n), x * 10.0 ** rng.integers(-12, 3, n)])
    return (g * 1e-3).astype(np.float32)


@pytest.mark.parametrize("mp,optimizer", [(False, 0), (True, 0), (False, 4)])
@pytest.mark.parametrize("de", (False, True))
@pytest.mark.parametrize("k,bm,bv", [(k, *f) for k, f in enumerate(FORMATS)])
def test_both_forms_leave_the_same_bytes(gpu, k, bm, bv, de, mp, optimizer):  # noqa: F811
    """A buffer of more than QUAD_BLOCKS blocks in one call and in two, which take the other form."""
    import torch
    cut, off = (QUAD_BLOCKS * 3 // 5 // 5 * 5) * B, 8 * 99                      # (cut: whole blocks and whole code words)
    for bf16 in (False, True):
        for p, end in ((0.1, ENDS[(3 * k) % len(ENDS)]), (0.3, 0), (0.97, ENDS[(3 * k + 1) % len(ENDS)])):
            n = (QUAD_BLOCKS + 6) * B + end
            flags = 1 | (2 if de else 0) | optimizer

            def config(offset):
                return gpu.make_config(bm, bv, B, 1 if bf16 else 0, flags=flags, quantile_p=p, index_offset=offset)

            cfg = config(off)
            rng = np.random.default_rng(k)
            gen = torch.Generator(device="cuda").manual_seed(k)
            p0 = torch.randn(n, device="cuda", generator=gen)
            scale = torch.tensor([0.5], device="cuda") if mp else None
            sides = [(p0.clone(), torch.zeros(n, dtype=torch.bfloat16, device="cuda") if mp else None, gpu.SoloState(n, cfg).buffers())
                     for _ in range(2)]
            for step in (1, 2, 3):
                g = torch.from_numpy(block_kinds(n, rng)).cuda().to(torch.bfloat16 if bf16 else torch.float32)
                q, h, st = sides[0]
                gpu.solo_adamw_step_mp(q, h, g, scale, *st, n, step, cfg)
                q, h, st = sides[1]
                for a, b in ((0, cut), (cut, n)):
                    part = (st[0][a // (32 // bm):], st[1][a // B:], st[2][a // (32 // bv):], st[3][a // B:], st[4][a // B:])
                    gpu.solo_adamw_step_mp(q[a:], None if h is None else h[a:], g[a:], scale, *part, b - a, step, config(off + a))
            torch.cuda.synchronize()
            for x, y in zip((sides[0][0], sides[0][1], *sides[0][2]), (sides[1][0], sides[1][1], *sides[1][2])):
                assert x is None or torch.equal(x.view(torch.int16 if x.element_size() == 2 else torch.int32),
                                                y.view(torch.int16 if x.element_size() == 2 else torch.int32)), (bf16, p, end)


@pytest.mark.parametrize("bm,bv,bf16,de", [(2, 3, True, False), (4, 4, False, True), (3, 2, False, False)])
def test_many_blocks(so, gpu, bm, bv, bf16, de):  # noqa: F811
    for end in (0, 1, 1030):
        run_teacher_forced(so, gpu, (QUAD_BLOCKS + 1) * B + end, bm, bv, B, bf16=bf16, steps=2, seed0=end, de=de)


@pytest.mark.parametrize("bm,bv,bf16,de,mp", [(2, 3, True, False, False), (4, 2, False, True, True), (3, 3, True, False, True),
                                               (4, 4, False, False, False), (3, 4, True, True, False)])
def test_tables(gpu, bm, bv, bf16, de, mp):  # noqa: F811
    """Tables of short blocks only, of few blocks of both kinds, of many blocks (two wavefronts each) and of
    many tensors of mostly one block each (four)."""
    for sizes in (ENDS, ENDS + [2048, 0, 2048] + ENDS[::-1], [2049, 4096, 6000] + ENDS[:5] + [9 * B + 1000, 2048],
                  [n + 45 * B for n in ENDS], [ENDS[k % len(ENDS)] + B * (k % 5 == 0) for k in range(1000)]):
        table_against_flat(gpu, sizes, bm, bv, B, bf16, de, mp=mp)


@pytest.mark.parametrize("n", (1000, 2047, 3 * B + 1000, (QUAD_BLOCKS + 6) * B + 700))
def test_nothing_behind_the_end_is_written(gpu, n):  # noqa: F811
    """Buffers that go on behind the last element, its code word and its block keep what is there."""
    import torch
    for bm, bv, bf16 in ((2, 3, True), (3, 4, False), (4, 2, True)):
        cfg = gpu.make_config(bm, bv, B, 1 if bf16 else 0)
        gen = torch.Generator(device="cuda").manual_seed(n)
        real = gpu.SoloState(n, cfg)
        grown = [torch.cat([t, torch.full((64,), 7 if t.dtype == torch.int32 else 7.0, dtype=t.dtype, device="cuda")])
                 for t in real.buffers()]
        p, h = (torch.full((n + 64,), 7.0, dtype=t, device="cuda") for t in (torch.float32, torch.bfloat16))
        g = torch.full((n + 64,), float("nan"), dtype=torch.bfloat16 if bf16 else torch.float32, device="cuda")
        g[:n] = (torch.randn(n, device="cuda", generator=gen) * 1e-3).to(g.dtype)
        for step in (1, 2):
            gpu.solo_adamw_step_mp(p, h, g, None, *grown, n, step, cfg)
        torch.cuda.synchronize()
        for t in (p[n:], h[n:], *(t[-64:] for t in grown)):
            assert bool((t == 7).all())
        assert bool(torch.isfinite(p).all()) and all(bool(torch.isfinite(t).all()) for t in (grown[1], grown[3], grown[4]))
