"""The form in which a launch evaluates its tiles' slots (fstat_slot_form, a
host function of the library): one that keeps coefficients from slot to slot
where most tiles gain from it, and never one that cannot evaluate some unit of
the launch, however few tiles that unit has."""
import pytest

import paper_0904_1826_amd as P

T = 1800.0
SHARED, WORDS = 1, 2
TAU = 1.0e7


def _unit(f0=700.0, n_bins=5000, step=1.0, shift=0.5, tiles=100):
    return (step / T, shift / (TAU * T), T, int(f0 * T) - n_bins // 2, n_bins, TAU, tiles)


def test_units_that_gain_share_and_the_majority_decides():
    assert P.fstat_slot_form([_unit()]) != 0
    assert P.fstat_slot_form([_unit(shift=1.5)]) == 0
    assert P.fstat_slot_form([_unit(step=0.37)]) == 0
    assert P.fstat_slot_form([_unit(), _unit(step=0.37, tiles=90)]) != 0
    assert P.fstat_slot_form([_unit(), _unit(step=0.37, tiles=110)]) == 0


@pytest.mark.parametrize("n_bins", [1 << 20, (1 << 20) + 1, 1 << 21, 1 << 25])
def test_a_wide_band_is_never_read_by_words(n_bins):
    """A word of the position holds a bin within [2^20, 2^21); a unit with
    bins beyond in the launch, even with one tile of ten thousand, must not
    be evaluated so."""
    wide = _unit(f0=18000.0, n_bins=n_bins, tiles=1)
    assert P.fstat_slot_form([wide]) != WORDS
    for units in ([_unit()] * 100 + [wide], [wide] + [_unit()] * 100):
        assert P.fstat_slot_form(units) != WORDS


@pytest.mark.parametrize("k_first,n_bins,form", [
    (1 << 20, 1 << 20, WORDS), ((1 << 20) - 1, 5000, SHARED), ((1 << 21) - 5000, 5000, WORDS),
    ((1 << 21) - 5000, 5001, SHARED), (90000, 5000, SHARED), (0, 1 << 25, SHARED)])
def test_words_where_the_band_lies_in_their_binade(k_first, n_bins, form):
    u = (1.0 / T, 0.0, T, k_first, n_bins, TAU, 10)
    assert P.fstat_slot_form([u]) == form
    assert P.fstat_slot_form([u] + [_unit()] * 9) == form


def test_bad_arguments():
    lib = P.load_library()
    assert lib.fstat_slot_form(0, None, None, None) == P.FSTAT_E_ARG
    assert lib.fstat_slot_form(1, None, None, None) == P.FSTAT_E_ARG
