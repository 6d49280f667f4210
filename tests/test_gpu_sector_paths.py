"""Sectors of 26 to 32 orbitals listed run by run or high part by high part: the
lists on both sides of the rule that decides, with few and many windows, windows
that overlap, modular weights (negative ones too) and both widths, against the
oracle; and few particles among many orbitals do not take long."""
import time

import numpy as np
import pytest

from oracle import combinatorics as OC
from tests._util import host_u32, host_u64, say

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")
torch = pytest.importorskip("torch")


def _states(sec):
    s = sec.states()
    return host_u32(s).astype(np.uint64) if sec.width_bits == 32 else host_u64(s)


def _full(M):
    return (1 << M) - 1


def _spin(L, n_up, n_dn):
    return [(_full(L), n_dn, n_dn), (_full(L) << L, n_up, n_up)]


def _oracle(M, cons):
    """The oracle's list; the particle number that the windows imply is said, so that it walks C(M, N) patterns."""
    exact = [c for c in cons if c[1] == c[2]]
    covered = sum(c[0] for c in exact) == _full(M)  # of windows that share no bits
    return OC.sector_enumerate(M, ([(_full(M), *[sum(c[1] for c in exact)] * 2)] if covered else []) + cons)


SECTORS = [
    (32, [(_full(32), 1, 1)]), (32, [(_full(32), 3, 3)]), (32, [(_full(32), 4, 4)]), (32, [(_full(32), 30, 30)]), (31, [(_full(31), 26, 26)]),
    (28, [(_full(28), 5, 5)]), (28, [(_full(28), 6, 6)]), (26, [(_full(26), 7, 7)]),
    (32, _spin(16, 1, 2)), (32, _spin(16, 3, 3)), (30, _spin(15, 2, 5)), (30, _spin(15, 13, 15)), (30, _spin(15, 0, 0)),
    # a window in the low bits, one in the high bits, and both overlapping the particle number's
    (28, [(_full(28), 6, 6), (0xFF, 2, 8)]), (28, [(_full(28), 6, 6), (0xFF << 20, 4, 8)]), (32, [(_full(32), 5, 5), (0xFFF << 10, 1, 3)]),
    # many windows, and ones that nothing passes
    (30, [(_full(30), 4, 4)] + [(0x3F << i, 0, 3) for i in range(8)]), (24, [(_full(24), 5, 5)] + [(0x3F << i, 0, 3) for i in range(8)]),
    (32, [(_full(32), 4, 4), (0xF, 0, 0), (0xF0, 4, 4), (0xF00, 1, 1)]),
    # the particle number implied by three windows
    (30, [(0x3FF, 2, 2), (0x3FF << 10, 1, 1), (0x3FF << 20, 2, 2)]),
]


@pytest.mark.parametrize("case", range(len(SECTORS)))
@pytest.mark.parametrize("width", [32, 64])
def test_lists_on_both_sides_of_the_rule(case, width):
    M, cons = SECTORS[case]
    say("sector: M", M, "width", width, cons)
    assert np.array_equal(_states(mbr.sector_build(M, cons, width)), _oracle(M, cons))


@pytest.mark.parametrize("L,n_up,n_dn,modulus", [(16, 2, 2, 16), (16, 2, 5, 16), (14, 1, 2, 14), (15, 2, 3, 2 ** 31 - 1), (16, 0, 4, 5)])
@pytest.mark.parametrize("width", [32, 64])
def test_modular_lists_on_both_sides_of_the_rule(L, n_up, n_dn, modulus, width):
    w = [(7 * i) % 31 - 15 for i in range(2 * L)]  # some negative
    cons = _spin(L, n_up, n_dn)
    st = _oracle(2 * L, cons)
    total = np.zeros(st.size, dtype=np.int64)
    for b in range(2 * L):
        total += (st >> np.uint64(b) & np.uint64(1)).astype(np.int64) * w[b]
    for residue in {0, 3 % modulus, int(total[0]) % modulus}:
        got = _states(mbr.sector_build_mod(2 * L, cons, w, modulus, residue, width_bits=width))
        assert np.array_equal(got, st[total % modulus == residue])


def _best(M, cons):
    t = []
    for _ in range(5):
        torch.cuda.synchronize()
        a = time.perf_counter()
        sec = mbr.sector_build(M, cons)
        t.append(time.perf_counter() - a)
        del sec
    return min(t)


@pytest.mark.parametrize("M,cons", [(32, [(_full(32), 2, 2)]), (32, [(_full(32), 4, 4)]), (30, [(_full(30), 5, 5)]), (32, _spin(16, 2, 3))])
def test_few_particles_among_many_orbitals_are_listed_soon(M, cons):
    # a few thousand patterns and more, as few among 20 orbitals: about twice the time, and 6 to 30 times where the
    # high parts were dealt out at a stride
    small = _best(20, [(_full(20), 2, 2)])
    big = _best(M, cons)
    say("us: 20 orbitals", small * 1e6, "M", M, cons, big * 1e6)
    assert big <= 4 * small
