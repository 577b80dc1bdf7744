"""CPU: which sweep kernel a launch takes after the autotuner has measured a size.  The
built-in rule changes inside a size class (floor(log2(tiles))); a measured choice holds
on the measured size's side of such a change only, a choice set by a caller in the
whole class."""
import ctypes

import pytest

import paper_1711_02146_amd as pam

PM, GAUSS16, GAUSS = pam.PA_MODEL_PM, pam.PA_MODEL_GAUSS16, pam.PA_MODEL_GAUSS
BIT = pam.PA_LAYOUT_BITPACK64
PACKED, SEVERAL, ONE = 1, 2, 3  # kernels with several tiles per workgroup, and with one


@pytest.fixture
def tune():
    lib = ctypes.CDLL(pam.LIB_PATH)
    u32, u64 = ctypes.c_uint32, ctypes.c_uint64
    form = lib._ZN2pa15sweep_split_forEjjjm  # pa::sweep_split_for
    form.restype, form.argtypes = u32, [u32, u32, u32, u64]
    record = lib._ZN2pa18sweep_split_recordEjjjmj  # pa::sweep_split_record
    record.restype, record.argtypes = None, [u32, u32, u32, u64, u32]
    pam.pa_autotune_reset()
    yield form, record
    pam.pa_autotune_reset()


def test_measured_choice_is_between_the_kernels_that_were_timed(tune):
    """+-J on four waves: one tile per workgroup below 1500 tiles at L = 6 and 3200 at
    L = 8, several from there up."""
    form, record = tune
    for L, line in ((6, 1500), (8, 3200)):
        low, high = line - 100, line + 100
        assert form(PM, BIT, L, low) == 4 and form(PM, BIT, L, high) == PACKED
        record(PM, BIT, L, low, 8)  # eight waves against four on one tile
        assert form(PM, BIT, L, low) == 8 and form(PM, BIT, L, line - 1) == 8
        assert form(PM, BIT, L, line) == PACKED and form(PM, BIT, L, high) == PACKED
        record(PM, BIT, L, high, 8)  # eight waves against the packed form
        assert form(PM, BIT, L, line) == 8 and form(PM, BIT, L, high) == 8
        assert form(PM, BIT, L, low) == 4


@pytest.mark.parametrize("model", [GAUSS16, GAUSS])
def test_measured_choice_follows_the_rounds_of_workgroups(tune, model):
    """L = 10: two tiles per workgroup are faster at 512 tiles (one round against
    two), one at 768 (three rounds against two of twice the length)."""
    form, record = tune
    assert form(model, BIT, 10, 512) == SEVERAL and form(model, BIT, 10, 768) == ONE
    record(model, BIT, 10, 512, 4)
    assert form(model, BIT, 10, 512) == SEVERAL and form(model, BIT, 10, 768) == ONE
    record(model, BIT, 10, 768, 8)
    assert form(model, BIT, 10, 768) == ONE and form(model, BIT, 10, 700) == ONE
    assert form(model, BIT, 10, 512) == SEVERAL
    record(model, BIT, 10, 512, 8)  # measured otherwise: taken where the rule says the same
    assert form(model, BIT, 10, 512) == ONE and form(model, BIT, 10, 768) == ONE


def test_set_choice_holds_in_the_whole_class(tune):
    form, _ = tune
    pam.pa_autotune_set(10, 64 * 512, 4, model="gauss")
    assert form(GAUSS, BIT, 10, 512) == SEVERAL and form(GAUSS, BIT, 10, 768) == SEVERAL
    pam.pa_autotune_set(6, 64 * 1100, 4)
    assert form(PM, BIT, 6, 1100) == 4 and form(PM, BIT, 6, 1600) == PACKED


def test_built_in_rule_at_l6(tune):
    """+-J, L = 6: eight waves on a tile where a launch leaves most compute units one
    tile each, four below and above."""
    form, _ = tune
    assert [form(PM, BIT, 6, t) for t in (1, 47, 48, 256, 257, 1499, 1500)] == [4, 4, 8, 8, 4, 4,
                                                                                PACKED]
