"""A cached launch shape is used for the Hamiltonian it was tuned for: not for
other amplitudes on the same bonds, which other kernels may serve, not for
another kind of U, and not when the line's key lacks the version of the shapes."""
import pytest

from oracle import hamiltonian as OH

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")
torch = pytest.importorskip("torch")

L = 6


def _create(t_uniform=True, u_uniform=True):
    bonds = OH.chain_bonds(L)
    if not t_uniform:
        bonds = [(b[0], b[1], 0.5 + 0.25 * i) for i, b in enumerate(bonds)]
    return mbr.hubbard_create(L, bonds, [(3, 3)], U=[2.0] * L if u_uniform else [2.0 + i for i in range(L)])


def test_cached_shape_is_for_its_own_hamiltonian(tmp_path, monkeypatch):
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("MBR_AUTOTUNE_CACHE", str(cache))
    mbr.hubbard_autotune(_create(), reps=1)
    (line,) = cache.read_text().splitlines()
    key = line.split()[0]
    planted = f"{key} 3 4 256 123.0\n"  # a shape and a time that tuning would not give
    cache.write_text(planted)
    got = mbr.hubbard_autotune(_create(), reps=1)
    assert (got["k"], got["G"], got["block"], got["tuned_ms"]) == (3, 4, 256, 123.0)
    for n, kw in enumerate((dict(t_uniform=False), dict(u_uniform=False), dict(t_uniform=False, u_uniform=False))):
        assert mbr.hubbard_autotune(_create(**kw), reps=1)["tuned_ms"] != 123.0
        assert len(cache.read_text().splitlines()) == n + 2  # tuned and appended under a key of its own


def test_line_of_an_older_version_is_not_taken(tmp_path, monkeypatch):
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("MBR_AUTOTUNE_CACHE", str(cache))
    mbr.hubbard_autotune(_create(), reps=1)
    key = cache.read_text().split()[0]
    cache.write_text(f"{key.split(';t')[0]} 3 4 256 123.0\n")  # bonds and sectors alone
    assert mbr.hubbard_autotune(_create(), reps=1)["tuned_ms"] != 123.0
    assert len(cache.read_text().splitlines()) == 2
