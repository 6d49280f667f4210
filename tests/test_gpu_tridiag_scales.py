"""The tridiagonal solver on matrices in any units, and where a division of its
interval meets a pivot exactly: entries of 1e10 and of 1e200, zero pivots, and
powers of two, which have to come out as the same bits scaled."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")
torch = pytest.importorskip("torch")

CELLS = 257  # of one division of the interval


def _lowest(a, b):
    """Lowest eigenvalue by the library of the matrix with diagonal a, off-diagonal b."""
    n = len(a)
    da = torch.tensor(np.asarray(a, dtype=np.float64), device="cuda")
    db = torch.tensor(np.append(np.asarray(b, dtype=np.float64), 0.0), device="cuda")
    ln = torch.tensor([n], dtype=torch.int32, device="cuda")
    return float(mbr.tridiag_lowest(da, db, ln, n).cpu()[0])


def _exact(a, b):
    return np.linalg.eigvalsh(np.diag(a) + np.diag(b, 1) + np.diag(b, -1))[0]


def _division(a, b, t):
    """Point t of the first division of the Gershgorin interval."""
    r = np.abs(np.append(b, 0)) + np.abs(np.append(0, b))
    lo, hi = (a - r).min(), (a + r).max()
    pad = 1e-12 * max(abs(lo), abs(hi))
    lo, hi = lo - pad, hi + pad
    return lo + (hi - lo) / CELLS * (t + 1)


# tolerance: the interval ends 4.5e-16 of its bounds wide and the counts are those of a matrix off by a few
# roundings of its norm, so 4e-15 of the norm covers both for these small matrices
@pytest.mark.parametrize("unit", [1.0, 1e10, 1e-10, 1e200, 1e-200])
def test_zero_pivot_coupled_to_the_lowest_state(unit):
    c = 64 * unit
    b = np.array([c / 64, c, c])
    a = np.array([_division(np.zeros(4), b, 20), 0.0, 0.0, 0.0])  # a pivot of exactly 0, the lowest eigenvalue just below
    assert _division(a, b, 20) == a[0]
    s = 1 / unit
    assert abs(_lowest(a, b) * s - _exact(a * s, b * s)) <= 4e-15 * 128


@pytest.mark.parametrize("unit", [1.0, 1e10, 1e-10, 1e200, 1e-200])
def test_zero_pivot_before_the_lowest_state(unit):
    # the lowest state stands by itself behind a block whose first pivot is exactly 0 at the first division
    S = 257 * unit
    b = np.array([unit, 0.0, 0.0])
    a = np.array([_division(np.array([0.0, 0.0, -S, S]), 0 * b, 0), 0.0, -S, S])
    assert _division(a, b, 0) == a[0]
    assert abs(_lowest(a, b) + S) <= 4e-15 * S


@pytest.mark.parametrize("n", [1, 2, 7, 40, 2049])
def test_powers_of_two_scale_the_result_exactly(n):
    r = np.random.RandomState(n)
    a, b = r.uniform(-3, 3, n), r.uniform(0.1, 2, n - 1)
    e = _lowest(a, b)
    if n < 100:
        assert abs(e - _exact(a, b)) <= 4e-15 * 8
    for k in (-900, -60, 60, 900):
        assert _lowest(np.ldexp(a, k), np.ldexp(b, k)) == np.ldexp(e, k)


def test_zero_and_constant_matrices():
    assert _lowest(np.zeros(5), np.zeros(4)) == 0.0
    assert _lowest(np.full(5, -2.5), np.zeros(4)) == pytest.approx(-2.5, rel=1e-15)
