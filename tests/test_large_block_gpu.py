"""Blocks above 4 GiB in one time range: a stage's byte count (rows times the
row stride, 32 bits) is that of its 64 rows at most, also while more than
2^32 bytes of the range are left.  At the lengths here the bytes left at ring
stage 1 or 3 are just above 2^32.  Integer work: equal to the oracle's."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import KIND_X16, first_mismatch, forced_kernel, gpu_available

pytestmark = pytest.mark.gpu
if not gpu_available():
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


# 4-byte loads (12 tiles, 9 tiles), 16-byte loads of whole rows (N = 64) and of ragged ones
@pytest.mark.parametrize("N,F,T", [(190, 1024, 22150), (132, 1024, 32000), (64, 2200, 30720), (60, 2352, 30650)])
def test_block_above_4_gib(N, F, T):
    import torch
    from paper_1904_07778_amd.xeng import Plan
    print(f"block of {T * F * N / 2**30:.3f} GiB, N={N} F={F} T={T}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(N)
    v = torch.randint(0, 256, (T, F, N), dtype=torch.uint8, device="cuda", generator=gen)
    with forced_kernel(N, F, T, KIND_X16, split=1):
        with Plan([(N, F, T)]) as p:
            out, n = p.correlate_dump([v])
            torch.cuda.synchronize()
    assert n == [T]
    for f in (0, F // 2 + 1, F - 1):
        want = oracle.correlate(v[:, f:f + 1].cpu().numpy())
        got = out[0][f:f + 1].cpu().numpy()
        assert np.array_equal(got, want), (f, first_mismatch(got, want))
