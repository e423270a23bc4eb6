"""Calls split along time: each workgroup stores its chunk's sums and a second
kernel adds them up, with earlier samples of the integration.  Ring kernel
(whole and ragged N, one and several phases) and staging kernel (N = 255),
few channels so that every call is split; short and long calls of one
integration and snapshots.  Integer work: equal to the oracle's."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import first_mismatch, gpu_available

pytestmark = pytest.mark.gpu
if not gpu_available():
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


@pytest.mark.parametrize("N,F", [(16, 1), (32, 4), (48, 3), (100, 4), (101, 3), (176, 2), (200, 2), (250, 1), (255, 1)])
def test_split_calls_of_one_integration(N, F):
    import torch
    from paper_1904_07778_amd.xeng import Plan
    print(f"split N={N} F={F}", flush=True)
    rng = np.random.default_rng(N)
    blocks = [rng.integers(0, 256, size=(t, F, N), dtype=np.uint8) for t in (4000, 129, 4000, 2050)]
    dev = [torch.from_numpy(b).cuda() for b in blocks]
    with Plan([(N, F, 4000)]) as p:
        for _ in range(2):
            e = oracle.Engine(N, F)
            for b, d in zip(blocks[:-1], dev):
                e.correlate(b)
                p.correlate([d])
                snap, _ = p.dump(keep=True, to_host=True)
                want = e.dump(keep=True)[0]
                assert np.array_equal(snap[0].numpy(), want), first_mismatch(snap[0].numpy(), want)
            e.correlate(blocks[-1])
            out, n = p.correlate_dump([dev[-1]])
            torch.cuda.synchronize()
            want = e.dump()[0]
            got = out[0].cpu().numpy()
            assert n == [10179] and np.array_equal(got, want), first_mismatch(got, want)


def test_one_long_call():
    """One channel over 400,000 samples: the longest chunk a workgroup may
    integrate (32768) sets the split, after a short call on the same plan."""
    import torch
    from paper_1904_07778_amd.xeng import Plan
    N, F, T = 240, 1, 400000
    rng = np.random.default_rng(5)
    v = rng.integers(0, 256, size=(T, F, N), dtype=np.uint8)
    d = torch.from_numpy(v).cuda()
    e = oracle.Engine(N, F)
    e.correlate(v)
    want = e.dump()[0]
    with Plan([(N, F, T)]) as p:
        for _ in range(2):
            p.correlate([d[:100]])
            _, _ = p.dump(to_host=True)
            p.correlate([d])
            out, _ = p.dump(to_host=True)
            assert np.array_equal(out[0].numpy(), want), first_mismatch(out[0].numpy(), want)


@pytest.mark.parametrize("T", [200, 3000])
def test_last_block_of_an_integration_in_a_batch(T):
    """correlate, then correlate_dump into fresh buffers: the earlier sums are
    read from the accumulator (one chunk per item), or copied over first
    (items split along time), for arrays inside the persistent launch and on
    launches of their own; the next integration starts empty."""
    import torch
    from paper_1904_07778_amd.xeng import Plan
    shapes = [(192, 3, T), (32, 5, T), (40, 16, T), (255, 1, T)]
    rng = np.random.default_rng(T)
    vs = [rng.integers(0, 256, size=(t, f, n), dtype=np.uint8) for n, f, t in shapes]
    dev = [torch.from_numpy(v).cuda() for v in vs]
    print(f"last block T={T}", flush=True)
    with Plan(shapes) as p:
        for _ in range(2):
            p.correlate(dev)
            p.correlate([dev[0], None, dev[2], None])
            out = [torch.full_like(p.new_output(a), -1) for a in range(len(shapes))]
            _, n = p.correlate_dump(dev, out=out)
            torch.cuda.synchronize()
            assert n == [3 * T, 2 * T, 3 * T, 2 * T]
            for v, o, k in zip(vs, out, n):
                want = oracle.to_int32(oracle.accumulate(v) * (k // T))
                got = o.cpu().numpy()
                assert np.array_equal(got, want), first_mismatch(got, want)
