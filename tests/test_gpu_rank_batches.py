"""Staggered and spin ranks around the batch sizes where a lane goes from one
vector of queries to two, with tables in LDS and in memory, aligned and not."""
import pytest

import synth
from tests._util import say

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")
torch = pytest.importorskip("torch")


# 256 CUs: eight workgroups of 1024 lanes each hold 2^21 vectors, of four 32-bit or two 64-bit patterns
@pytest.mark.parametrize("width,edge", [(32, 1 << 23), (64, 1 << 22)])
@pytest.mark.parametrize("k", [8, 14])
@pytest.mark.parametrize("kind", ["staggered", "spin"])
def test_ranks_around_one_vector_per_lane(width, edge, k, kind):
    if kind == "spin":
        L, nu, nd = (14, 6, 8) if width == 32 else (17, 3, 4)
        r, size = mbr.build_spin_ranker(L, nu, nd, k), None
        cons = [((1 << L) - 1, nd, nd), (((1 << L) - 1) << L, nu, nu)]
        M = 2 * L
    else:
        M, N = (22, 9) if width == 32 else (34, 5)
        r = mbr.build_staggered_tables(M, N, k, width)
        cons = [((1 << M) - 1, N, N)]
    sec = mbr.sector_build(M, cons, width)
    idx = torch.from_numpy(synth.uniform_indices(3, edge + 5, sec.size)).to(torch.int32).cuda()
    q = mbr.unrank_batch(sec, idx)
    q[::1001] |= 1 << (M - 1)  # some leave the sector
    want = idx.clone()
    member = mbr.rank_batch(mbr.build_bitmap_trie(sec, 8), q)
    for n in (edge - 3, edge, edge + 5):
        say("rank batch", kind, width, "k", k, "n", n)
        for off in (0, 1):
            got = mbr.rank_batch(r, q[off:n])
            assert torch.equal(got, member[off:n])
    keep = member >= 0
    assert torch.equal(member[keep & (q == mbr.unrank_batch(sec, idx))], want[keep & (q == mbr.unrank_batch(sec, idx))])


def test_calls_go_to_the_current_stream():
    side = torch.cuda.Stream()
    assert mbr.binding._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert mbr.binding._stream(None) == side.cuda_stream
    assert mbr.binding._stream(side) == side.cuda_stream
    assert mbr.binding._stream(None) == torch.cuda.current_stream().cuda_stream
