"""Rules that choose between two kernels, asked on the host (no GPU): each takes the kernel that was measured to be the faster
one, at points on both sides of its lines."""
import ctypes

import pytest

import paper_2006_16668_amd as moe
from paper_2006_16668_amd.binding import _Config
from test_gpu_attention_blocks import OTHERS, WIDE
from test_gpu_gradient_pairs import CASES as PAIR_CASES

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


def test_attention_gradients_of_few_and_many_sequences():
    """The bit-for-bit test's few and many take different kernels where it says so."""
    wide = _rule("_ZN3moe18attention_dkv_wideExii", ctypes.c_longlong, ctypes.c_int, ctypes.c_int)
    short = _rule("_ZN3moe18attention_dq_shortEiixi", ctypes.c_int, ctypes.c_int, ctypes.c_longlong, ctypes.c_int)
    for cases, many in ((WIDE, True), ([c for c in OTHERS if c[0] == 128 and c[2] % 128 == 0], False)):
        for _, heads, L, B in cases:
            assert wide(B * heads, L, UNITS) is many and not wide(2 * heads, L, UNITS)
    assert any(L % 256 == 128 for _, _, L, _ in WIDE)
    took = [(short(d, L, 2 * heads * ((L + 127) // 128), UNITS), short(d, L, B * heads * ((L + 127) // 128), UNITS))
            for d, heads, L, B in OTHERS if L % 128]
    assert (True, False) in took and (False, True) in took


# tokens, M, E, us of a layer of H 64 that packs wg first and of one whose gate splits it
@pytest.mark.parametrize("tokens,M,E,packed,split", [
    (64, 4096, 32, 67.7, 59.9), (64, 1024, 33, 33.0, 32.0), (700, 1536, 64, 48.3, 47.1), (4096, 2048, 64, 65.7, 64.7),
    (700, 2560, 33, 63.1, 65.3), (64, 3072, 64, 65.2, 69.3), (64, 4096, 33, 78.3, 84.2), (700, 4096, 64, 88.9, 93.2)])
def test_gate_weights_of_one_call(tokens, M, E, packed, split):
    assert _rule("_ZN3moe14gate_splits_wgEii", ctypes.c_int, ctypes.c_int)(E, M) == (split < packed)


@pytest.mark.parametrize("d", [64, 128])
def test_widest_attention_takes_the_matrix_cores(d):
    """The plain kernels, for other widths, refuse sequences of about 4000 tokens (2000 backward)."""
    ok = _rule("_ZN3moe17attention_mfma_okEiiii", *[ctypes.c_int] * 4)
    bf16, f32 = 1, 0
    for heads in (1, 43690 * 128 // d, 43691 * 128 // d, 0x7fffff // d):       # up to the limit of heads . d
        assert ok(bf16, 5000, heads, d) and not ok(f32, 5000, heads, d)


# the tiles of the data and the weight gradient that share a launch, for dh with dwo and dbuf with dwi; None: two launches
SMALL, FLAT, LARGE = "64x64", "64x128", "128x128"
PAIRS = [((SMALL, SMALL), (SMALL, SMALL)), ((SMALL, SMALL), (SMALL, SMALL)), ((SMALL, SMALL), (SMALL, SMALL)),
         ((SMALL, FLAT), (SMALL, FLAT)), ((SMALL, LARGE), (SMALL, LARGE)), ((SMALL, LARGE), (FLAT, LARGE)),
         ((FLAT, SMALL), (SMALL, SMALL)), ((SMALL, SMALL), (FLAT, SMALL)), ((LARGE, LARGE), None), ((FLAT, FLAT), (SMALL, FLAT)),
         ((LARGE, LARGE), (LARGE, LARGE)), ((FLAT, LARGE), (LARGE, LARGE)), ((LARGE, SMALL), (SMALL, FLAT)),
         ((LARGE, FLAT), (FLAT, FLAT))]
FORMS = {2: LARGE, 3: LARGE, 4: FLAT, 5: FLAT, 6: SMALL, 7: SMALL}


def _pair(cfg, masked):
    rule = _rule("_ZN3moe19gradient_pair_formsERK10moe_configbiPiS3_", ctypes.c_void_p, ctypes.c_bool, ctypes.c_int,
                 ctypes.c_void_p, ctypes.c_void_p)
    c, data, weight = _Config(cfg.G, cfg.S, cfg.M, cfg.H, cfg.E, cfg.C, 1), ctypes.c_int(), ctypes.c_int()
    if not rule(ctypes.byref(c), masked, UNITS, ctypes.byref(data), ctypes.byref(weight)):
        return None
    return FORMS[data.value], FORMS[weight.value]


@pytest.mark.parametrize("cfg,want", list(zip(PAIR_CASES, PAIRS)), ids=lambda v: getattr(v, "name", ""))
def test_pairs_of_gradients(cfg, want):
    assert (_pair(cfg, True), _pair(cfg, False)) == want


def test_every_pair_kernel_is_launched_by_a_case():
    assert len(PAIRS) == len(PAIR_CASES)
    assert len({p for case in PAIRS for p in case if p is not None}) == 9
