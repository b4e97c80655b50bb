"""GPU tests of the forms a multi-tensor launch takes: every tensor is left as the flat step leaves it that
starts at the tensor's own place in the xi stream, byte for byte."""
import pytest

from test_dispatch_lines import PIECES8, QUAD_BLOCKS, pieces
from test_gpu_parity import gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def bits(t):
    import torch
    return t.view(torch.int16 if t.element_size() == 2 else torch.int32)


def table_against_flat(gpu, sizes, bm, bv, B, bf16=True, de=False, flags=0, mp=False, p=0.1, steps=2, spoil=None):  # noqa: F811
    """Steps the tensors in one launch and one by one; returns the (param, state, copy) of the table's side.
    spoil(params): changes the parameters first."""
    import torch
    off0 = 8 * 321
    flags |= 1 | (2 if de else 0)

    def config(off):
        return gpu.make_config(bm, bv, B, 1 if bf16 else 0, flags=flags, quantile_p=p, index_offset=off)

    cfg = config(off0)
    gen = torch.Generator(device="cuda").manual_seed(7)
    scale = torch.tensor([0.5], device="cuda") if mp else None
    ps = [torch.randn(n, device="cuda", generator=gen) for n in sizes]
    if spoil:
        spoil(ps)
    sides = [[(q.clone(), gpu.SoloState(n, cfg), torch.zeros(n, dtype=torch.bfloat16, device="cuda") if mp else None)
              for q, n in zip(ps, sizes)] for _ in range(2)]
    dtype = torch.bfloat16 if bf16 else torch.float32
    gs = [torch.zeros(n, dtype=dtype, device="cuda") for n in sizes]
    table = gpu.SoloMultiTable([(q, g, st, h) for (q, st, h), g in zip(sides[0], gs)], cfg)
    for step in range(1, steps + 1):
        for g in gs:
            g.copy_((torch.randn(len(g), device="cuda", generator=gen) * 1e-3).to(dtype))
        table.step(step, grad_scale=scale)
        off = off0
        for (q, st, h), g, n in zip(sides[1], gs, sizes):
            gpu.solo_adamw_step_mp(q, h, g, scale, *st.buffers(), n, step, config(off))
            off += -(-n // 2560) * 2560
    torch.cuda.synchronize()
    for n, (q, st, h), (q1, st1, h1) in zip(sizes, *sides):
        assert torch.equal(bits(q), bits(q1)), n
        assert h is None or torch.equal(bits(h), bits(h1)), n
        for a, b in zip(st.buffers(), st1.buffers()):
            assert torch.equal(bits(a), bits(b)), n
    return sides[0]


@pytest.mark.parametrize("bf16,B", [(True, 128), (False, 64), (True, 2048)])
def test_a_parameter_that_is_not_finite_leaves_the_state_alone(gpu, bf16, B):  # noqa: F811
    """Plain AdamW does not feed parameters back into the moments, however short the table."""
    import torch

    def spoil(ps):
        ps[0][17], ps[0][5119], ps[1][0] = float("inf"), float("nan"), float("-inf")

    for n in (10240, max((QUAD_BLOCKS + 1) * 2048, (PIECES8 + 1) * 1024)):      # 8 and 16 elements per lane (blocks of 2048: four wavefronts and two)
        sizes, many = [n, 5120 + 77], n > 10240
        assert (pieces(sizes) > PIECES8) == many and (n // 2048 > QUAD_BLOCKS) == many
        for q, st, _ in table_against_flat(gpu, sizes, 2, 3, B, bf16, spoil=spoil):
            assert all(bool(torch.isfinite(x).all()) for x in (st.m_scale, st.v_scale, st.v_base))


# ends of every kind: less than a word, a block, a 512-element piece, a chunk; one and two pieces behind
# whole chunks; empty tensors between and behind
ENDS = [600, 1, 0, 79, 512, 513, 1023, 1024, 1025, 1535, 1537, 2047, 2048, 2560, 5119, 5120, 5121, 7, 3000, 0, 0]


# (the last one: behind them a tensor that makes the table one of many pieces, stepped with 16 elements per lane)
@pytest.mark.parametrize("count,bm,bv,B,bf16,de,mp,long", [(1, 2, 3, 128, True, False, False, False), (2, 4, 2, 64, True, True, True, False),
                                                            (63, 3, 3, 128, False, False, True, False), (64, 2, 2, 64, False, True, False, False),
                                                            (65, 3, 4, 128, False, False, False, False), (400, 4, 4, 128, True, False, True, False),
                                                            (4097, 2, 3, 64, True, False, False, False),
                                                            (2, 4, 2, 64, True, True, True, True), (63, 3, 3, 128, False, False, True, True),
                                                            (65, 3, 4, 128, False, False, False, True), (400, 4, 4, 128, True, False, True, True)])
def test_many_short_tensors(gpu, count, bm, bv, B, bf16, de, mp, long):  # noqa: F811
    """The search for the tensor of a wavefront (64 tensors at a step) and the pieces of tensors that are
    mostly ends, in tables of few pieces and of many."""
    sizes = [ENDS[k % len(ENDS)] for k in range(count)] + [PIECES8 * 1024] * long
    assert pieces(sizes) > PIECES8 or not long
    table_against_flat(gpu, sizes, bm, bv, B, bf16, de, mp=mp)


@pytest.mark.parametrize("bf16", (True, False))
def test_a_launch_sized_by_the_units(gpu, bf16):  # noqa: F811
    """A caller that hands back only the documented bits of the flags gets the same step."""
    import torch
    cfg = gpu.make_config(3, 2, 128, 1 if bf16 else 0)
    sizes = [n for n in ENDS if n] * 40
    dtype = torch.bfloat16 if bf16 else torch.float32
    sides = []
    for bits_kept in (~0, 3):
        gen = torch.Generator(device="cuda").manual_seed(1)
        items = [(torch.randn(n, device="cuda", generator=gen), torch.randn(n, device="cuda", generator=gen).to(dtype),
                  gpu.SoloState(n, cfg)) for n in sizes]
        table = gpu.SoloMultiTable(items, cfg)
        assert table.flags >> 2 == pieces(sizes)
        table.flags &= bits_kept
        table.step(1)
        table.step(2)
        sides.append([x for p, _, st in items for x in (p, *st.buffers())])
    assert all(torch.equal(bits(a), bits(b)) for a, b in zip(*sides))
