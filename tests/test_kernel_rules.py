"""Rules that choose between two kernels, asked on the host (no GPU): each takes the kernel that was measured to be the faster
one, at points on both sides of its lines."""
import ctypes

import pytest

import paper_2006_16668_amd as moe

UNITS = 256                                     # of the device that was measured


def _rule(mangled, *types):
    f = getattr(ctypes.CDLL(moe.library_path()), mangled)
    f.argtypes, f.restype = types, ctypes.c_bool
    return f


# d, L, sequence-heads, us of the short kernel and of the other
@pytest.mark.parametrize("d,L,n,short,other", [
    (128, 48, 64, 7.8, 9.9), (128, 100, 400, 21.5, 21.9), (128, 191, 96, 15.6, 16.0), (128, 200, 200, 29.5, 29.0),
    (128, 200, 152, 28.2, 27.1), (128, 300, 20, 20.9, 20.0), (128, 300, 132, 34.4, 32.4), (128, 700, 128, 95.2, 90.4),
    (64, 48, 64, 6.0, 6.7), (64, 193, 32, 11.6, 12.7), (64, 300, 132, 20.3, 19.9), (64, 700, 12, 24.3, 23.1), (64, 700, 88, 46.8, 52.1),
    (64, 700, 248, 88.8, 91.6), (64, 900, 80, 58.3, 62.3), (64, 1000, 80, 64.3, 68.6), (64, 1000, 112, 88.9, 86.9)])
def test_dq_of_ragged_sequences(d, L, n, short, other):
    rule = _rule("_ZN3moe18attention_dq_shortEiixi", ctypes.c_int, ctypes.c_int, ctypes.c_longlong, ctypes.c_int)
    assert rule(d, L, n * ((L + 127) // 128), UNITS) == (short < other)
