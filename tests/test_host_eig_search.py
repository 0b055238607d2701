"""Where the eigenvalue search looks next: around the zero of the secant through the values at both ends of the interval, and at
thirds of it where there is no such line.  Needs no GPU."""
import ctypes

import pytest

from testing_lib import load


def _points(flo, elo, fhi, ehi, wanted, q):
    out = (ctypes.c_double * 2)()
    return load().lq_test_search_points(flo, elo, fhi, ehi, wanted, q, ctypes.addressof(out)), out[0], out[1]


@pytest.mark.parametrize("flo,elo,fhi,ehi,zero", [(-0.5, 0, 0.5, 0, 0.5), (0.75, 3, -0.75, 4, 1 / 3), (-0.6, -40, 0.6, -42, 0.8)])
def test_secant(flo, elo, fhi, ehi, zero):
    for q in (0.125, 1e-9):
        secant, a, b = _points(flo, elo, fhi, ehi, 1, q)
        assert secant == 1
        assert a == pytest.approx(max(zero - q, zero / 2), abs=1e-15) and b == pytest.approx(min(zero + q, (1 + zero) / 2), abs=1e-15)


@pytest.mark.parametrize("flo,fhi,wanted", [(0.0, 0.7, 1), (-0.7, 0.0, 1), (0.0, 0.0, 1), (0.5, 0.7, 1), (-0.5, 0.7, 0),
                                             (float("nan"), 0.7, 1), (-0.7, float("inf"), 0)])
def test_thirds(flo, fhi, wanted):
    """An end whose value is not known (0), ends of one sign, several eigenvalues in the interval, a value that is not finite."""
    assert _points(flo, 0, fhi, 0, wanted, 0.125) == (0, 1 / 3, 2 / 3)
