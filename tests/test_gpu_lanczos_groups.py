"""Gram-Schmidt Lanczos on sectors around the rules for its groups: coefficients
summed inside the subtraction (up to 64 groups a sector) or by their own kernel,
one alpha_up block a group or as many as leave two groups a CU, blocks that do
not divide evenly, alone and beside other sectors, batched and per sector."""
import numpy as np
import pytest

from oracle import hamiltonian as OH
import synth
from tests._util import say

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")
torch = pytest.importorskip("torch")


def _coeffs(L, sectors, m, prec=0, **kw):
    """Energy and coefficients of the first sector; its start vector does not depend on the others."""
    h = mbr.hubbard_create(L, OH.chain_bonds(L), sectors, U=[3.0] * L, precision=prec)
    lz = mbr.lanczos_create(h, m, **kw)
    mbr.lanczos_start(lz, torch.from_numpy(2 * synth.uniform01(3, h.dim) - 1).cuda())
    mbr.lanczos_step(lz, m)
    e0, done = mbr.lanczos_result(lz)
    a, b = mbr.lanczos_coeffs(lz)
    return e0[0], done[0], a[0], b[0]


def _same(x, y, atol):
    assert x[1] == y[1] and abs(x[0] - y[0]) <= atol
    assert np.allclose(x[2], y[2], rtol=0, atol=atol) and np.allclose(x[3], y[3], rtol=0, atol=atol)


@pytest.mark.parametrize("prec,atol", [(0, 1e-10), (1, 2e-4)])
def test_coefficients_summed_either_way(prec, atol):
    # 55 blocks of 462 rows, two a group: 28 groups, whose coefficients the subtraction sums itself when the sector
    # is alone.  Beside one of 231 groups the handle sums all sectors' coefficients separately; the groups stay the
    # same.  Rounding of the sums over twelve steps (norms below 30): 1e-10 in fp64, 2e-4 with fp32 vectors
    alone = _coeffs(11, [(2, 5)], 12, prec, reorth=True)
    for kw in (dict(reorth=True), dict(reorth=True, batched=False), dict()):
        _same(alone, _coeffs(11, [(2, 5), (5, 5)], 12, prec, **kw), atol)


# C(12,6) = 924, C(13,5) = 1287 and C(13,6) = 1716 blocks: two, three and four a group, or more where they are short;
# C(13,3) = 286 blocks of 1,716 rows: two a group in fp64, the last one of an odd number short where there are 495
@pytest.mark.parametrize("L,sector", [(12, (6, 2)), (12, (6, 6)), (13, (5, 3)), (13, (6, 2)), (13, (3, 6)), (12, (4, 6))])
def test_a_sector_alone_and_beside_another(L, sector):
    say("Gram-Schmidt groups: L", L, sector)
    alone = _coeffs(L, [sector], 10, reorth=True)
    _same(alone, _coeffs(L, [sector], 10, reorth=True, batched=False), 1e-10)
    _same(alone, _coeffs(L, [sector, (1, 1)], 10, reorth=True), 1e-10)
    _same(alone, _coeffs(L, [sector], 10), 1e-10)  # no reorthogonalisation: other kernels, the same recurrence this early
