"""Every chunk value of the bitmap trie's steps: a third and two thirds of all
18-bit patterns as sectors, looked up with all 2^18 patterns and some beyond them.
The last level's records (64 to 128 KB) are read from memory by a small batch and
staged by a large one, and every part of a record, every word of a part and every
bit of a word is asked for, set and clear."""
import numpy as np
import pytest

from tests._util import dev_u32, dev_u64, say

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")
torch = pytest.importorskip("torch")

M = 18


@pytest.mark.parametrize("width", [32, 64])
@pytest.mark.parametrize("k", [3, 4, 5, 6, 7, 8])
def test_all_chunk_values(k, width):
    say("bitmap trie steps", k, width)
    every = np.arange(1 << M, dtype=np.uint64)
    far = np.array([1 << M, (1 << M) + 5, (1 << width) - 1, 1 << (width - 1)], dtype=np.uint64)
    for members in (every[every % 3 == 1], every[every % 3 != 1]):
        as_dev = dev_u32 if width == 32 else dev_u64
        s = mbr.sector_from_list(M, as_dev(members), width_bits=width)
        r = mbr.build_bitmap_trie(s, k)
        small = np.concatenate([every[::-1], far])            # 262,148 queries
        large = np.concatenate([every, far, small])[: -3]     # 524,293: an odd count past 2^19
        for q in (small, large):
            at = np.searchsorted(members, q)
            hit = members[np.minimum(at, members.size - 1)] == q
            want = np.where(hit, at, 0xFFFFFFFF).astype(np.uint32)
            got = mbr.rank_batch(r, as_dev(q)).cpu().numpy().view(np.uint32)
            assert np.array_equal(got, want), (k, width, members.size, q.size)
