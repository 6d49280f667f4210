"""Lanczos steps however they are launched: several per graph, one per graph or
kernel by kernel, on sectors of few and many tiles and with sectors that stop on
the way, give the same bits; the Gram-Schmidt coefficients summed inside the
subtraction or by their own kernel agree to rounding; and the tridiagonal solver
around the size it stages in LDS."""
import numpy as np
import pytest

from oracle import hamiltonian as OH
import synth
from tests._util import say

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")
torch = pytest.importorskip("torch")


def _steps(h, parts, m, **kw):
    lz = mbr.lanczos_create(h, m, **kw)
    mbr.lanczos_start(lz, torch.from_numpy(2 * synth.uniform01(3, h.dim) - 1).cuda())
    for n in parts:
        mbr.lanczos_step(lz, n)
    e0, done = mbr.lanczos_result(lz)
    a, b = mbr.lanczos_coeffs(lz)
    return e0, done, a, b


# one sector (18, 400 and 63,504 rows) and several, of which some stop at their dimension within a graph
@pytest.mark.parametrize("L,sectors", [(4, [(1, 3)]), (6, [(3, 3)]), (10, [(5, 5)]), (6, [(0, 1), (1, 1), (3, 3), (6, 6), (2, 4)])])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("reorth", [False, True])
def test_steps_do_not_depend_on_how_they_are_launched(L, sectors, prec, reorth):
    say("lanczos steps: L", L, sectors, "precision", prec, "reorth", reorth)
    h = mbr.hubbard_create(L, OH.chain_bonds(L), sectors, U=[3.0] * L, precision=prec)
    want = _steps(h, [1] * 27, 27, reorth=reorth, use_graph=False)
    for parts in ([27], [8, 8, 8, 3], [3, 17, 7], [1, 16, 8, 2]):
        for graph in (True, False):
            for g, w in zip(_steps(h, parts, 27, reorth=reorth, use_graph=graph), want):
                assert np.array_equal(g, w), (parts, graph)


def test_gram_schmidt_coefficients_summed_either_way():
    # 853,776 rows in one sector: more groups than the subtraction sums itself; batched groups against the tiles
    # of per-sector launches, to rounding of the fp64 sums over twelve steps
    h = mbr.hubbard_create(12, OH.chain_bonds(12), [(6, 6)], U=[3.0] * 12)
    e1 = _steps(h, [12], 12, reorth=True)
    e2 = _steps(h, [12], 12, reorth=True, batched=False)
    plain = _steps(h, [12], 12)
    for other in (e2, plain):
        assert np.allclose(e1[2], other[2], rtol=0, atol=1e-10) and np.allclose(e1[3], other[3], rtol=0, atol=1e-10)


@pytest.mark.parametrize("n", [1, 2, 3, 257, 2047, 2048, 2049, 4096])
def test_tridiagonal_lowest_around_its_staging(n):
    # diagonal 0, off-diagonal 1: -2 cos(pi / (n + 1)).  The counts belong to a matrix whose entries are off by a few
    # roundings (norm 2), and the interval ends 4.5e-16 of its bounds wide: 2e-14 covers both
    a = torch.zeros(2, n, dtype=torch.float64, device="cuda")
    b = torch.ones(2, n, dtype=torch.float64, device="cuda")
    a[1] = 0.75  # the same spectrum, shifted
    ln = torch.full((2,), n, dtype=torch.int32, device="cuda")
    e = mbr.tridiag_lowest(a, b, ln, n).cpu().numpy()
    want = -2 * np.cos(np.pi / (n + 1))
    assert abs(e[0] - want) <= 2e-14 and abs(e[1] - (want + 0.75)) <= 2e-14
