"""Sector lists and packed tries built on the device, at the sizes where their
kernels' tiles end: against the oracle's enumeration, and every member and
non-members ranked against bisection."""
import numpy as np
import pytest

from oracle import combinatorics as OC
import synth
from tests._util import dev_u32, dev_u64, host_rank, host_u32, host_u64, say

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")
torch = pytest.importorskip("torch")


def _states(sec):
    s = sec.states()
    return host_u32(s).astype(np.uint64) if sec.width_bits == 32 else host_u64(s)


def _brute(M, cons, weights=None, modulus=0, residue=0):
    a = np.arange(1 << M, dtype=np.uint64)
    keep = np.ones(a.size, dtype=bool)
    for mask, lo, hi in cons:
        c = np.zeros(a.size, dtype=np.int64)
        for b in range(M):
            if mask >> b & 1:
                c += (a >> np.uint64(b) & np.uint64(1)).astype(np.int64)
        keep &= (c >= lo) & (c <= hi)
    if modulus:
        w = np.zeros(a.size, dtype=np.int64)
        for b in range(M):
            w += (a >> np.uint64(b) & np.uint64(1)).astype(np.int64) * weights[b]
        keep &= w % modulus == residue
    return a[keep]


# below, at and above the 64 patterns of a step, the 2^10 of a wave and the first second high part
@pytest.mark.parametrize("M", [1, 5, 6, 7, 10, 11, 16])
@pytest.mark.parametrize("width", [32, 64])
def test_lists_of_windows(M, width):
    full = (1 << M) - 1
    for cons in ([], [(full, M // 2, M // 2)], [(full, min(1, M - 1), M - 1), (0x15 & full, 0, 1)],
                 [(1 << b, 0, 1) for b in range(min(M, 5))] + [(full, 0, max(1, M - 2))], [(full, M, M)], [(0x2A & full, 2, 2)]):
        say("sector: M", M, "width", width, cons)
        assert np.array_equal(_states(mbr.sector_build(M, cons, width)), _brute(M, cons))


@pytest.mark.parametrize("M,modulus", [(5, 3), (12, 7), (17, 2 ** 31 - 1), (18, 1)])
def test_lists_of_modular_weights(M, modulus):
    # negative weights and weights beyond the modulus
    w = [int(v) for v in (synth.splitmix64(M, M) % np.uint64(41)).astype(np.int64) - 20]
    cons = [((1 << M) - 1, 2, M - 1)]
    for residue in {0, modulus // 2, modulus - 1, 5 % modulus}:
        got = _states(mbr.sector_build_mod(M, cons, w, modulus, residue))
        assert np.array_equal(got, _brute(M, cons, w, modulus, residue))


@pytest.mark.parametrize("M,N", [(32, 4), (33, 4), (26, 20)])
def test_lists_around_32_orbitals(M, N):
    cons = OC.constraints(M, N)
    width = 32 if M <= 32 else 64
    assert np.array_equal(_states(mbr.sector_build(M, cons, width)), OC.sector_enumerate(M, cons))


# 1 to 184,756 members (tiles of 2,048 and 4,096), chunks of one digit, two digits and a short last one
@pytest.mark.parametrize("M,N", [(9, 9), (12, 6), (15, 7), (20, 10), (24, 3)])
@pytest.mark.parametrize("k", [3, 8, 9, 11, 16])
def test_tries_rank_every_member(M, N, k):
    say("trie: M", M, "N", N, "k", k)
    cons = OC.constraints(M, N)
    st = OC.sector_enumerate(M, cons)
    r = mbr.build_trie(mbr.sector_build(M, cons), k)
    q = np.concatenate([st, synth.splitmix64(5, 5000) & np.uint64(2 ** 32 - 1), synth.splitmix64(6, 5000) & np.uint64((1 << M) - 1)])
    assert np.array_equal(host_rank(mbr.rank_batch(r, dev_u32(q))), OC.bisect_rank(st, q))


@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 4096, 4097, 30000])
@pytest.mark.parametrize("k", [5, 13])
def test_tries_of_lists(n, k):
    # irregular 64-bit patterns
    st = np.unique(synth.splitmix64(8, n + 40) >> np.uint64(4))[:n]
    r = mbr.build_trie(mbr.sector_from_list(60, dev_u64(st), 64), k)
    q = np.concatenate([st, synth.splitmix64(9, 3000) >> np.uint64(4), st ^ np.uint64(1)])
    assert np.array_equal(host_rank(mbr.rank_batch(r, dev_u64(q))), OC.bisect_rank(st, q))
