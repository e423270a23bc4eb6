"""Bit-exact parity of the 16-row ring kernel for N that is no multiple of 16.

Every tile count, both load units (16-byte chunks; 4-byte units where the
chunks would need a 17th tile), every shift of a channel's bytes within its
unit, rows whose stride is no multiple of the unit (phases), the last chunk
at the end of the block, groups short of channels, and the three epilogues.
Integer work: equal to the oracle's."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import first_mismatch, gpu_available, run_engine

pytestmark = pytest.mark.gpu
if not gpu_available():
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


def codes(rng, T, F, N):
    return rng.integers(0, 256, size=(T, F, N), dtype=np.uint8)   # -8 included


def expect(blocks, N, F):
    e = oracle.Engine(N, F)
    for b in blocks:
        e.correlate(b)
    return e.dump()[0]


# F = 16: whole chunks per row for every N (one phase), 5 or 11 channels: up
# to 16 phases; T = 64 k + remainder: partial stages
@pytest.mark.parametrize("N", [1, 2, 7, 8, 9, 15, 17, 20, 24, 30, 31, 40, 47, 50, 62, 72, 88, 95, 100, 104, 111,
                               113, 124, 126, 136, 143, 152, 158, 168, 175, 190, 200, 207, 216, 223, 232, 239,
                               241, 242, 243, 244, 245, 246, 247, 250, 252, 253, 254, 255])
@pytest.mark.parametrize("F,T", [(16, 203), (5, 333), (2, 1)])
def test_ragged_inputs(N, F, T):
    print(f"ragged N={N} F={F} T={T}", flush=True)
    v = codes(np.random.default_rng(N * 100 + F), T, F, N)
    got, n = run_engine([v], N, F)
    want = expect([v], N, F)
    assert n == T and np.array_equal(got, want), first_mismatch(got, want)


@pytest.mark.parametrize("N,F", [(3, 16), (40, 6), (100, 4), (190, 8), (200, 10), (250, 8), (251, 4), (253, 3)])
def test_ragged_accumulate_and_dump(N, F):
    """Store, read-modify-write and atomic epilogues over calls of one
    integration, the last straight into the destination; then a new one."""
    import torch
    from paper_1904_07778_amd.xeng import Plan
    print(f"ragged accumulate N={N} F={F}", flush=True)
    rng = np.random.default_rng(N)
    blocks = [codes(rng, t, F, N) for t in (65, 448, 3, 2100)]
    with Plan([(N, F, 2100)]) as p:
        for _ in range(2):
            for b in blocks[:-1]:
                p.correlate([torch.from_numpy(b).cuda()])
            out, n = p.correlate_dump([torch.from_numpy(blocks[-1]).cuda()])
            torch.cuda.synchronize()
            want = expect(blocks, N, F)
            got = out[0].cpu().numpy()
            assert n == [2616] and np.array_equal(got, want), first_mismatch(got, want)


def test_ragged_block_inside_a_larger_buffer():
    """The block's neighbours in memory (the chunks of the first and last
    channel reach into them) do not enter any sum."""
    import torch
    from paper_1904_07778_amd.xeng import Plan
    N, F, T = 37, 3, 130
    rng = np.random.default_rng(9)
    v = codes(rng, T, F, N)
    size = T * F * N
    big = torch.from_numpy(rng.integers(0, 256, size=size + 4096, dtype=np.uint8)).cuda()
    view = big[1024:1024 + size].view(T, F, N)
    view.copy_(torch.from_numpy(v))
    with Plan([(N, F, T)]) as p:
        out, _ = p.correlate_dump([view])
        torch.cuda.synchronize()
        got = out[0].cpu().numpy()
    want = expect([v], N, F)
    assert np.array_equal(got, want), first_mismatch(got, want)


def test_ragged_arrays_in_a_batch():
    import torch
    from paper_1904_07778_amd.xeng import Plan
    shapes = [(250, 4, 300), (40, 16, 900), (192, 3, 700), (37, 5, 260), (64, 8, 512)]
    rng = np.random.default_rng(12)
    vs = [codes(rng, t, f, n) for n, f, t in shapes]
    dev = [torch.from_numpy(v).cuda() for v in vs]
    with Plan(shapes) as p:
        for _ in range(3):
            p.correlate(dev)
            out, _ = p.correlate_dump(dev)
            torch.cuda.synchronize()
            for (n, f, t), v, o in zip(shapes, vs, out):
                want = expect([v, v], n, f)
                got = o.cpu().numpy()
                assert np.array_equal(got, want), (n, f, first_mismatch(got, want))
