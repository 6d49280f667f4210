"""A Lanczos handle is ready for any stream when it is created: start and steps on a
stream that does not wait for the null stream, while another thread keeps the
null stream busy, give the bits of a quiet run; and a second start on the
same handle begins afresh, whatever the first run left behind."""
import threading

import numpy as np
import pytest

from oracle import hamiltonian as OH
import synth
from tests._util import say

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")
torch = pytest.importorskip("torch")


def _run(h, v0, reorth, stream, starts=1):
    lz = mbr.lanczos_create(h, 20, reorth=reorth)
    for _ in range(starts):
        mbr.lanczos_start(lz, v0, stream=stream)
        mbr.lanczos_step(lz, 11, stream=stream)
    e0, done = mbr.lanczos_result(lz, stream=stream)
    a, b = mbr.lanczos_coeffs(lz, stream=stream)
    return e0, done, a[:, :11], b[:, :11]


@pytest.mark.parametrize("reorth", [False, True])
def test_created_while_the_null_stream_is_busy(reorth):
    say("lanczos handles made beside a busy null stream, reorth", reorth)
    h = mbr.hubbard_create(8, OH.chain_bonds(8), [(4, 4), (3, 5)], U=[4.0] * 8)
    v0 = torch.from_numpy(2 * synth.uniform01(5, h.dim) - 1).cuda()
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    want = _run(h, v0, reorth, None)
    big = torch.zeros(1 << 26, device="cuda")
    stop = threading.Event()

    def busy():
        while not stop.is_set():
            for _ in range(4):
                big.add_(1.0)
            torch.cuda.default_stream().synchronize()

    t = threading.Thread(target=busy)
    t.start()
    try:
        got = [_run(h, v0, reorth, side) for _ in range(20)]
    finally:
        stop.set()
        t.join()
    for g in got:
        for a, b in zip(g, want):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("reorth", [False, True])
def test_a_second_start_begins_afresh(reorth):
    h = mbr.hubbard_create(8, OH.chain_bonds(8), [(4, 4)], U=[4.0] * 8)
    v0 = torch.from_numpy(2 * synth.uniform01(6, h.dim) - 1).cuda()
    for a, b in zip(_run(h, v0, reorth, None, starts=3), _run(h, v0, reorth, None)):
        assert np.array_equal(a, b)
