"""GPU parity of the kernels that give a lane 16 elements: flat buffers behind the lines of
test_dispatch_lines.py, and the largest ones in front of them, which run 8; tables of many pieces.  Same bar as
test_gpu_parity.py.  (Every instantiation of them is compared with the 8-per-lane kernels in
test_gpu_both_forms.py; blocks of 2048 have a test file of their own,
test_gpu_short_blocks.py.)"""
import numpy as np
import pytest

from parity_common import compare_step, flip_budget, make_cfgs
from test_dispatch_lines import LAST8_FP32, PIECES8, last8
from test_gpu_parity import GpuSide, dev, gpu, run_teacher_forced  # noqa: F401

pytestmark = pytest.mark.gpu

FORMATS = [(bm, bv, B) for B in (64, 128) for bm in (2, 3, 4) for bv in (2, 3, 4)]
# elements behind the line (the first: the largest buffer with 8 per lane): whole chunks of 1024 only; a chunk short of one
# element, of all but one; ends in either half of a chunk, on and next to a code word's and a block's end
BEHIND = [0, 1, 1023, 1024, 1025, 512, 511, 1024 + 513, 2048 + 8, 1024 + 80]


@pytest.mark.parametrize("k,bm,bv,B", [(k, *f) for k, f in enumerate(FORMATS)])
def test_formats_and_ragged_ends(so, gpu, k, bm, bv, B):  # noqa: F811
    for j in range(3):
        # (the last one: 8 per lane)
        bf16, copy = (k + j) % 2 == 0, (k + 2 * j) % 4 == 0
        n = last8(bf16, copy) + BEHIND[(2 * k + j) % len(BEHIND)] if j < 2 else (5 << 18) + 1 + (k * 401) % 1100
        opt = ("adamw", "adam_l2", "adabelief")[(k + j) % 3]
        ext = dict(grad_scale=0.5, bf16_copy=True) if copy else {}
        run_teacher_forced(so, gpu, n, bm, bv, B, bf16=bf16, steps=2 if j < 2 else 3, seed0=10 * k, de=(k // 2 + j) % 2 == 1,
                           optimizer=opt, eps=1e-12 if opt == "adabelief" else 1e-8, **ext)


@pytest.mark.parametrize("p", (0.0, 0.1, 0.3, 0.97))
@pytest.mark.parametrize("bm,bv,B", [(2, 3, 128), (4, 2, 64)])
def test_ties_zeros_and_quantiles(so, gpu, bm, bv, B, p):  # noqa: F811
    """Blocks in which most or all lanes tie, blocks of zeros, single entries, a wide range of
    magnitudes, from a state two steps old, over the ranks of small and large quantiles."""
    from paper_2505_00347_amd import synth
    n = LAST8_FP32 + 3 * 1024 + 77
    oc, gc = make_cfgs(so, gpu, bm, bv, B, False, p=p, off=8 * ((1 << 32) - 700))
    rng = np.random.default_rng(5)
    block = np.arange(n) // B
    kinds = block % 7
    prm, st = synth.make_params(n), so.State(n, oc)
    side = GpuSide(gpu, n, gc)
    flips = 0
    for step in (1, 2, 3):
        x = rng.standard_normal(n).astype(np.float32)
        g = np.where(kinds == 0, x, np.where(kinds == 1, 0.0, np.where(kinds == 2, 1.0, np.where(
            kinds == 3, np.rint(x), np.where(kinds == 4, np.where(np.arange(n) % B == 5, 1.0, 0.0), np.where(
                kinds == 5, x * 10.0 ** rng.integers(-12, 6, n), np.sign(x))))))).astype(np.float32) * np.float32(1e-3)
        side.load(prm, st)
        side.step(dev(g), step)
        before = prm.astype(np.float64)
        margin = so.step_packed(prm, g, st, step, oc, want_margin=True, threads=8)
        flips += compare_step(so, oc, n, prm, st, margin, side.fetch(), 1e-6, 2e-6 * oc.lr, p_before=before)
    assert flips <= flip_budget(3 * n)


@pytest.mark.parametrize("bm,bv,B,bf16,de,ext", [(2, 3, 128, True, False, False), (3, 3, 128, True, True, True),
                                                  (4, 4, 128, True, False, False), (2, 4, 64, False, True, True),
                                                  (2, 2, 64, False, False, False), (3, 4, 128, False, False, True)])
def test_tables(gpu, bm, bv, B, bf16, de, ext):  # noqa: F811
    """A table of tensors whose ends fall everywhere in a unit and in a chunk (units of 5120 and of
    2560 elements, with entries for a ragged end and without): every tensor as the flat step
    leaves it that starts at the tensor's own place in the xi stream, byte for byte."""
    import torch
    sizes = [400001, 2559, 2560, 2561, 0, 5119, 5120, 5121, 1023, 1024, 1025, 511, 7, 2049, 3071, 3072, 3073, 7680, 1,
             400000, PIECES8 * 1024]
    gen = torch.Generator(device="cuda").manual_seed(7)
    flags = 1 | (2 if de else 0)
    cfg = gpu.make_config(bm, bv, B, 1 if bf16 else 0, flags=flags, index_offset=8 * 321)
    scale = torch.tensor([0.5], device="cuda") if ext else None
    ps = [torch.randn(n, device="cuda", generator=gen) for n in sizes]
    sts = [gpu.SoloState(n, cfg) if n else None for n in sizes]
    hs = [torch.zeros(n, dtype=torch.bfloat16, device="cuda") if ext else None for n in sizes]
    flat = [(p.clone(), gpu.SoloState(len(p), cfg) if len(p) else None, None if h is None else h.clone())
            for p, h in zip(ps, hs)]
    for step in (1, 2, 3):
        gs = [(torch.randn(n, device="cuda", generator=gen) * 1e-3).to(torch.bfloat16 if bf16 else torch.float32)
              for n in sizes]
        keep = [k for k, n in enumerate(sizes) if n]
        gpu.SoloMultiTable([(ps[k], gs[k], sts[k], hs[k]) for k in keep], cfg).step(step, grad_scale=scale)
        off = 8 * 321
        for k in keep:
            c = gpu.make_config(bm, bv, B, 1 if bf16 else 0, flags=flags, index_offset=off)
            p, st, h = flat[k]
            gpu.solo_adamw_step_mp(p, h, gs[k], scale, *st.buffers(), sizes[k], step, c)
            off += -(-sizes[k] // 2560) * 2560
    torch.cuda.synchronize()
    for k in keep:
        p, st, h = flat[k]
        assert torch.equal(ps[k].view(torch.int32), p.view(torch.int32)), sizes[k]
        assert h is None or torch.equal(hs[k].view(torch.int16), h.view(torch.int16)), sizes[k]
        for a, b in zip(sts[k].buffers(), st.buffers()):
            assert torch.equal(a.view(torch.int32), b.view(torch.int32)), sizes[k]


@pytest.mark.parametrize("p", (0.0, 0.1, 0.5, 0.97))
@pytest.mark.parametrize("bm,bv,tail", [(2, 3, 1), (4, 4, 1030), (3, 2, 2047), (2, 2, 0)])
def test_selection_in_blocks_of_2048(so, gpu, bm, bv, tail, p):  # noqa: F811
    """The quantile of a large block over everything its passes tell apart: scattered values, clusters,
    many equal values, zeros, magnitudes far below the maximum (below the first pass's range), and
    a shorter last block of each kind."""
    from paper_2505_00347_amd import synth
    n = 14 * 2048 + tail
    rng = np.random.default_rng(bm * 100 + bv)
    kind = (np.arange(n) // 2048 + tail) % 7
    for de in (False, True):
        oc, gc = make_cfgs(so, gpu, bm, bv, 2048, False, p=p, de=de)
        prm, st = synth.make_params(n), so.State(n, oc)
        side = GpuSide(gpu, n, gc)
        flips = 0
        for step in range(1, 7):
            x = rng.standard_normal(n).astype(np.float32)
            far = x * 10.0 ** rng.uniform(-11, 3, n)
            g = np.select([kind == 0, kind == 1, kind == 2, kind == 3, kind == 4, kind == 5],
                          [x, far, np.where(rng.random(n) < 0.5, 0.0, far), np.where(rng.random(n) < 0.9, 0.0, x),
                           np.rint(x), np.full(n, 1.0)], np.zeros(n)).astype(np.float32) * np.float32(1e-3)
            side.load(prm, st)
            side.step(dev(g), step)
            before = prm.astype(np.float64)
            margin = so.step_packed(prm, g, st, step, oc, want_margin=True, threads=8)
            flips += compare_step(so, oc, n, prm, st, margin, side.fetch(), 1e-6, 2e-6 * oc.lr, p_before=before)
        assert flips <= flip_budget(6 * n)
