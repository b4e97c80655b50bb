"""The pieces that a table's tensors are cut into, as the host counts them (no GPU: made-up addresses)."""
import numpy as np
import pytest

from paper_2505_00347_amd import solo


def cut(n):
    """Pieces of n elements: whole chunks of 1024 and 512 elements each up to the end of the last code word;
    512 elements each."""
    whole = n // 1024
    rest = -(-(-(-n // 80) * 80 - 1024 * whole) // 512) if n % 1024 else 0
    return whole + rest, -(-(-(-n // 80) * 80) // 512) if n % 512 else n // 512


def build(sizes, cfg):
    arr = (solo.solo_tensor * len(sizes))()
    for k, n in enumerate(sizes):
        arr[k] = solo.solo_tensor(16, None, *[16] * 6, n)
    units = solo.solo_multi_units(arr, len(sizes), cfg)
    buf = np.zeros(solo.solo_multi_table_bytes(len(sizes), units), np.uint8)
    rc, flags = solo.solo_multi_table_build(arr, len(sizes), cfg, buf.ctypes.data, buf.size)
    assert rc == solo.SOLO_OK
    return units, flags, buf[:96 * len(sizes)].view(np.uint32).reshape(len(sizes), 24)[:, 22:]


@pytest.mark.parametrize("bm,bv,B,bf16,de", [(2, 3, 128, 1, False), (4, 4, 64, 0, False), (4, 3, 128, 1, True),
                                              (2, 2, 64, 0, True)])
def test_counts_in_front_of_every_tensor(bm, bv, B, bf16, de):
    cfg = solo.make_config(bm, bv, B, bf16, flags=3 if de else 1)
    rng = np.random.default_rng(1)
    sizes = [0, 1, 79, 80, 81, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2559, 2560, 5119, 5120, 5121, 0, 0] + \
        [int(x) for x in rng.integers(0, 40000, 300)] + [0]
    units, flags, first = build(sizes, cfg)
    want = np.cumsum([(0, 0)] + [cut(n) for n in sizes], axis=0)
    assert np.array_equal(first, want[:-1])
    pieces = want[-1][0]
    assert flags >> 2 == pieces and flags & 3 == 0
    assert pieces <= 5 * units and want[-1][1] <= 2 * pieces       # what a launch is sized by


def test_a_launch_over_many_short_tensors_fits():
    """1.5 million tensors of 4600 elements: the work-items of the launch stay below 2^32 (sized by the
    units, of which a ragged end has one per 512 elements, they would not)."""
    cfg = solo.make_config(2, 3, 128, 1)
    units, flags, _ = build([4600] * 1500000, cfg)
    assert 5 * 64 * units > 1 << 32
    assert flags >> 2 == 1500000 * cut(4600)[0] and 64 * (flags >> 2) < 1 << 32
