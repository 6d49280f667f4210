"""The panel kernel of H·x (C_dn <= 1024 in fp32, <= 512 in fp64, <= 1024
there with bond-dependent hopping) where its
split can go wrong: groups of one to eight waves, blocks that do not fill the
last wave, fewer alpha_up blocks than groups, a last run of fewer blocks, up to
fifteen hops a half, uniform and bond-dependent hopping, uniform and
site-dependent U.  Each row sums the same terms in the same order with the
same fused operations as in the flat kernel, so the products are bitwise equal
to it; the rows are held to the oracle as the other kernels' are (64 eps of
the sum of absolute terms)."""
import numpy as np
import pytest

import synth
from oracle import hamiltonian as OH

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")
torch = pytest.importorskip("torch")

EPS64, EPS32 = 2.0 ** -52, 2.0 ** -23


def _dev(a, prec):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=torch.float64 if prec == mbr.F64 else torch.float32)


CASES = [
    # L, bonds, sectors
    (16, "star", [(1, 1), (1, 3), (3, 1), (2, 2), (1, 15), (15, 2), (0, 0), (2, 16)]),
    (12, "ring", [(6, 4), (5, 3), (2, 6), (0, 4), (12, 5), (4, 12), (1, 2)]),
    (11, "star", [(5, 5), (4, 4), (2, 8), (11, 3)]),
    (13, "ring", [(3, 2), (2, 3), (1, 11)]),
    (12, "star", [(2, 6), (3, 5), (0, 7), (1, 4)]),
    (4, "ring", [(2, 2), (1, 2), (2, 1), (4, 0)]),
    (1, "none", [(0, 0), (1, 0), (0, 1), (1, 1)]),
]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("L,kind,sectors", CASES)
def test_panel_products(L, kind, sectors, prec):
    if kind == "star":
        eps_b, V = synth.anderson_parameters(6, L - 1)
        bonds, eps = OH.star_bonds(V), [-3.0] + list(eps_b)
        U = [6.0] + [0.0] * (L - 2) + [0.5]
    else:
        bonds = OH.chain_bonds(L, periodic=True) if kind == "ring" else []
        U, eps = [3.0] * L, None
    h = mbr.hubbard_create(L, bonds, sectors, U=U, eps=eps, precision=prec)
    k = mbr.hubbard_get_config(h)["k"]
    x = 2 * synth.uniform01(71, h.dim) - 1
    if prec == mbr.F32:
        x = x.astype(np.float32).astype(np.float64)
    xd = _dev(x, prec)
    ys = []
    for G in (-1, 0, -2):
        mbr.hubbard_set_config(h, k, G, 512)
        y = torch.full_like(xd, float("nan"))
        mbr.hubbard_apply(h, xd, y)
        ys.append(y)
    assert torch.equal(ys[0], ys[1]) and torch.equal(ys[0], ys[2])
    y = ys[1].cpu().numpy().astype(np.float64)
    tl = OH.terms(L, bonds, U, eps)
    e = EPS64 if prec == mbr.F64 else EPS32
    for si, (nu, nd) in enumerate(sectors):
        o0, o1 = h.offsets[si], h.offsets[si + 1]
        st = OH.sector(L, nu, nd)
        rows = np.unique(np.concatenate([[0, st.size - 1], synth.uniform_indices(80 + si, min(st.size, 2000), st.size)]))
        want, ab = OH.apply(st, tl, x[o0:o1], rows=rows, with_abssum=True)
        bad = np.abs(y[o0:o1][rows] - want) > 64 * e * ab + 1e-300
        assert not bad.any(), (nu, nd, rows[np.nonzero(bad)[0][:5]])
