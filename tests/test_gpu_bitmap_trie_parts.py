"""Bitmap tries where their records' 16-byte parts and the number of staged levels
change: every chunk value of a record in and out of the sector, and batches below
and above the size from which a workgroup per CU stages more levels."""
import numpy as np
import pytest

from oracle import combinatorics as OC
import synth
from tests._util import dev_u32, dev_u64, host_rank, say

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")


@pytest.mark.parametrize("k", [5, 6, 7, 8])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_every_chunk_value(k, seed):
    # irregular lists over two levels: all 2^(2k) patterns asked for, a third of them members, and a dense and a sparse node
    u = synth.splitmix64(seed, 1 << (2 * k))
    st = np.nonzero((u % np.uint64(3) == 0) | (np.arange(u.size) >> k == 1) | (np.arange(u.size) == 5 << k))[0].astype(np.uint64)
    r = mbr.build_bitmap_trie(mbr.sector_from_list(2 * k, dev_u32(st)), k)
    q = np.arange(1 << (2 * k + 1), dtype=np.uint64)  # and as many beyond the width
    assert np.array_equal(host_rank(mbr.rank_batch(r, dev_u32(q))), OC.bisect_rank(st, q))


# sectors whose third or fourth level fits a whole CU's LDS but not a small workgroup's share
@pytest.mark.parametrize("M,N,k,width", [(24, 8, 5, 32), (36, 5, 8, 64), (27, 5, 7, 32), (30, 5, 6, 32)])
@pytest.mark.parametrize("n", [(1 << 19) - 1, (1 << 19) + 3])
def test_staged_levels_by_batch(M, N, k, width, n):
    say("bitmap trie: M", M, "N", N, "k", k, "batch", n)
    cons = OC.constraints(M, N)
    st = OC.sector_enumerate(M, cons)
    r = mbr.build_bitmap_trie(mbr.sector_build(M, cons, width), k)
    q = st[synth.uniform_indices(7, n, st.size)]
    q[::7] ^= np.uint64(1) << (synth.splitmix64(8, q[::7].size) % np.uint64(width))
    dev = dev_u32 if width == 32 else dev_u64
    assert np.array_equal(host_rank(mbr.rank_batch(r, dev(q))), OC.bisect_rank(st, q))
