"""GPU parity of the general operator's product over the paths its kernels
choose between, against the oracle's tuple apply: row counts around the sixteen
rows of a wave and the 64 of a tile, one wave and several on a row group, sum
tables from LDS and from memory, sectors that have none (walked by the trie),
tuples that leave the sector, 64-bit patterns, and rows that no tuple acts on
beside entries that are not finite."""
import numpy as np
import pytest

from oracle import combinatorics as OC
from oracle import hamiltonian as OH
import synth
from tests._util import dev_u32, say
from tests.test_gpu_terms import EPS64, _check, _oracle_terms, _random_nconserving, _ring_momentum, _momentum_sector

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")
torch = pytest.importorskip("torch")


# (M, N): 1, 15, 16, 17, 120 and 4,960 rows; M = 32 has a table of high parts too large for LDS
@pytest.mark.parametrize("M,N", [(6, 0), (15, 1), (16, 1), (17, 1), (16, 2), (31, 3), (32, 3)])
@pytest.mark.parametrize("kind", ["stag", "trie"])
def test_particle_number_sectors(M, N, kind):
    say("operator: M", M, "N", N, kind)
    cons = OC.constraints(M, N)
    sec = mbr.sector_build(M, cons)
    r = mbr.build_staggered_tables(M, N, 8) if kind == "stag" else mbr.build_trie(sec, 8)
    t, cl = _random_nconserving(M, 7 * M + N, 4 * M)
    _check(sec, r, OC.sector_enumerate(M, cons), M, t, cl, seed=M + N)


def _check_inside(sec, ranker, st, M, N, t, cl, seed):
    """Against the oracle's apply on all of C^M_N, the vector zero outside the sector: what leaves it adds nothing."""
    full = OC.sector_enumerate(M, OC.constraints(M, N))
    at = np.searchsorted(full, st)
    x = 2 * synth.uniform01(seed, st.size) - 1
    xf = np.zeros(full.size)
    xf[at] = x
    want, ab = OH.apply(full, _oracle_terms(M, t, cl), xf, with_abssum=True)
    op = mbr.operator_create(sec, ranker, mbr.terms_from_hamiltonian(M, t, cl))
    y = torch.empty(st.size, dtype=torch.float64, device="cuda")
    mbr.operator_apply(op, torch.from_numpy(x).cuda(), y)
    assert (np.abs(y.cpu().numpy() - want[at]) <= 64 * EPS64 * ab[at] + 1e-300).all()


@pytest.mark.parametrize("lo", [1, 3])
def test_window_sector_without_sum_tables(lo):
    # at least `lo` particles among the low orbitals: high parts with nested, unequal sets of low parts,
    # and tuples that move the particles out of the window
    M, N = 12, 6
    cons = [((1 << M) - 1, N, N), (0x3F, lo, 6)]
    sec = mbr.sector_build(M, cons)
    st = OC.sector_enumerate(M, cons)
    t, cl = _random_nconserving(M, 40 + lo, 6 * M)
    _check_inside(sec, mbr.build_trie(sec, 5), st, M, N, t, cl, seed=lo)


def test_list_sector_with_leaving_tuples():
    # every third member of a particle-number sector, adopted from a list
    M, N = 14, 6
    st = OC.sector_enumerate(M, OC.constraints(M, N))[::3]
    sec = mbr.sector_from_list(M, dev_u32(st))
    t, cl = _random_nconserving(M, 77, 5 * M)
    _check_inside(sec, mbr.build_trie(sec, 7), st, M, N, t, cl, seed=9)


@pytest.mark.parametrize("kind,k", [("stag", 6), ("stag", 14), ("trie", 10)])
def test_64_bit_patterns(kind, k):
    M, N = 40, 3
    cons = OC.constraints(M, N)
    sec = mbr.sector_build(M, cons, width_bits=64)
    r = mbr.build_staggered_tables(M, N, k, width_bits=64) if kind == "stag" else mbr.build_trie(sec, k)
    t, cl = _random_nconserving(M, 13, 60)
    _check(sec, r, OC.sector_enumerate(M, cons), M, t, cl, seed=k)


@pytest.mark.parametrize("L,n,K", [(11, 5, 0), (11, 6, 4), (12, 6, 1)])
def test_rows_of_one_high_part(L, n, K):
    # 19,404 to 71,148 rows: the kernel over rows that share their high part, with and without shared tiles
    say("operator: ring", L, n, K)
    M, t, cl = _ring_momentum(L, 4.0)
    cons, w, st = _momentum_sector(L, n, n, K)
    sec = mbr.sector_build_mod(M, cons, w, L, K)
    _check(sec, mbr.build_trie(sec, 7), st, M, t, cl, seed=L + K)


def test_many_rows_few_tuples():
    # real-space hopping on 10 sites with unequal spins, 52,920 rows, long-range bonds: more tuples per row than lanes
    L = 10
    M = 2 * L
    u = synth.uniform01(21, L * L)
    t = np.zeros((M, M))
    for i in range(L):
        for j in range(i):
            for o in (0, L):
                t[o + i, o + j] = t[o + j, o + i] = 2 * u[i * L + j] - 1
    cl = [(L + i, i, L + i, i, 4.0 + i) for i in range(L)]
    cons = OC.spin_constraints(L, 4, 5)
    sec = mbr.sector_build(M, cons)
    _check(sec, mbr.build_trie(sec, 10), OC.sector_enumerate(M, cons), M, t, cl, seed=5)


@pytest.mark.parametrize("M,N", [(10, 4), (18, 7)])  # 210 rows, split over waves; 31,824 rows of one high part each
def test_rows_read_only_what_their_tuples_reach(M, N):
    """Entries that are not finite reach exactly the rows whose tuples lead to
    them: a tuple that does not act adds nothing, not zero times its target."""
    cons = OC.constraints(M, N)
    st = OC.sector_enumerate(M, cons)
    sec = mbr.sector_build(M, cons)
    t = np.zeros((M, M))
    t[0, 1] = t[1, 0] = 1.0
    for i in range(2, M):
        t[i, i] = 0.25 * i
    t[M - 1, 2] = t[2, M - 1] = -0.5
    cl = [] if M < 18 else _random_nconserving(M, 2, 900)[1]
    terms = mbr.terms_from_hamiltonian(M, t, cl)
    op = mbr.operator_create(sec, mbr.build_staggered_tables(M, N, 6), terms)
    x = 2 * synth.uniform01(3, st.size) - 1
    x[5], x[17], x[st.size - 1] = np.inf, np.nan, -np.inf
    y = torch.empty(st.size, dtype=torch.float64, device="cuda")
    mbr.operator_apply(op, torch.from_numpy(x).cuda(), y)
    got = y.cpu().numpy()
    # reached rows: the tuples with prefactor 1 on a vector of 0 and 1
    reach = np.zeros(st.size)
    reach[[5, 17, st.size - 1]] = 1.0
    ot = _oracle_terms(M, t, cl)
    _, hit = OH.apply(st, ot, reach, with_abssum=True)
    want, ab = OH.apply(st, ot, np.where(np.isfinite(x), x, 0.0), with_abssum=True)
    assert np.array_equal(~np.isfinite(got), hit != 0)
    fine = hit == 0
    assert (np.abs(got - want)[fine] <= 64 * EPS64 * ab[fine] + 1e-300).all()
