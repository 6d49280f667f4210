"""The learned index's gradient over batch sizes around its tiles (32 samples a
step, 256 workgroups) against the fp64 oracle, and from several threads at once
(one of them holds the entry point's own scratch, the others allocate)."""
import threading

import numpy as np
import pytest

from oracle import mlp as OM
import synth
from tests._util import dev_u32, say
from tests.test_zz_no_alloc import _bf16, _params, _split

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")
torch = pytest.importorskip("torch")


def _batch(B, seed):
    q = synth.splitmix64(seed, B) & np.uint64(0xFFFFFFFF)
    return q, synth.uniform01(seed + 1, B).astype(np.float32)


@pytest.mark.parametrize("B", [64, 128, 8128, 8192, 8256, 24640])
def test_gradient_over_batch_sizes(B):
    say("gradient: batch", B)
    p32 = _params(31)
    q, tgt = _batch(B, 40)
    g, loss = mbr.mlp_gradients(torch.from_numpy(p32).cuda(), dev_u32(q), torch.from_numpy(tgt).cuda())
    P = _split(_bf16(p32))
    G = OM.gradients(P, OM.features(q), tgt.astype(np.float64))
    want = OM.loss(P, OM.features(q), tgt.astype(np.float64))
    assert abs(float(loss.cpu()[0]) - want) <= 1e-5 * max(1.0, want)
    for a, b in zip(_split(g.cpu().numpy()), G):  # the gradient test's bar: fp32 sums over the batch
        a, b = np.atleast_1d(a), np.atleast_1d(b)
        assert np.abs(a - b).max() <= 1e-4 * max(1e-12, np.abs(b).max())


def test_gradients_from_several_threads():
    p = torch.from_numpy(_params(32)).cuda()
    work = [(B, dev_u32(_batch(B, 50 + i)[0]), torch.from_numpy(_batch(B, 50 + i)[1]).cuda()) for i, B in enumerate((4096, 8256, 512, 4096))]
    want = [mbr.mlp_gradients(p, q, t) for _, q, t in work]
    torch.cuda.synchronize()
    bad = []

    def loop(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(20):
                g, l = mbr.mlp_gradients(p, work[i][1], work[i][2])
                if not (torch.equal(g, want[i][0]) and torch.equal(l, want[i][1])):
                    bad.append(i)

    threads = [threading.Thread(target=loop, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
