"""The natively marshalled step calls of the binding accept and refuse what the ctypes signatures of the
same entry points do (no GPU: every call returns before a launch)."""
import ctypes as C

import pytest

from paper_2505_00347_amd import solo


def ctypes_step(args, stream):
    ptr = [a if a is None or isinstance(a, int) else a.data_ptr() for a in args[:9]]
    return solo.lib().solo_adamw_step_mp(*ptr, args[9], args[10], C.byref(args[11]), stream)


class Address:
    def __init__(self, value):
        self.value = value

    def data_ptr(self):
        return self.value


@pytest.mark.parametrize("n,step,pointers,bits", [(0, 1, 16, 2), (100, 0, 16, 2), (100, 1, 0, 2), (100, 1, 20, 2),
                                                    (100, 1, None, 2), (-1, 1, 16, 2), (1 << 41, 1, 16, 2),
                                                    (100, 1, 16, 7), (0, 1, None, 7)])
def test_same_return_codes(n, step, pointers, bits):
    cfg = solo.make_config(bits_m=bits, bits_v=3, beta1=0.5)
    for wrap in (lambda p: p, lambda p: p if p is None else Address(p)):
        a = [wrap(pointers), None, wrap(pointers), None, *[wrap(pointers)] * 5, n, step, cfg]
        want = ctypes_step(a, 0)
        assert solo.solo_adamw_step_mp(*a, stream=0, check=False) == want
        assert solo.solo_adamw_step(a[0], a[2], *a[4:], stream=0, check=False) == want
    if want != solo.SOLO_OK:
        with pytest.raises(solo.SoloError):
            solo.solo_adamw_step_mp(*a, stream=0)


def test_refused_types():
    cfg = solo.make_config()
    good = [16, None, 16, None, 16, 16, 16, 16, 16, 0, 1, cfg]
    assert solo.solo_adamw_step_mp(*good) == solo.SOLO_OK          # n == 0: the stream is not asked for
    for k, bad in ((9, 1.5), (9, None), (10, "1"), (11, None), (11, solo.solo_tensor())):
        with pytest.raises(C.ArgumentError):
            solo.solo_adamw_step_mp(*good[:k], bad, *good[k + 1:])
    for k in (0, 2, 4):
        with pytest.raises(AttributeError):
            solo.solo_adamw_step_mp(*good[:k], 1.5, *good[k + 1:])
    with pytest.raises(C.ArgumentError):
        solo.solo_adamw_step_multi(16, 1, 1.0, 0, None, 1, cfg, stream=0)
    assert solo.solo_adamw_step_multi(16, 1, 0, 0, None, 1, cfg) == solo.SOLO_OK
    assert solo.solo_adamw_step_multi(8, 1, 1, 0, None, 1, cfg, stream=0, check=False) == solo.SOLO_E_INVALID
