"""Rows per thread of the requantiser: one row, a number between, the most,
and a last group that is short, on both the paired and the general path.
Integer work: equal to the oracle's."""
import numpy as np
import pytest

from oracle import requant as R
from tests.gpu_util import gpu_available

pytestmark = pytest.mark.gpu
if not gpu_available():
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


# (T, F, N): 1024 pairs (or 256 samples) to a workgroup; 2048 workgroups of
# one row, then more rows each
@pytest.mark.parametrize("T,F,N", [(3, 1, 16), (2048, 1, 16), (4099, 1, 16), (13001, 1, 16), (33000, 1, 16), (2047, 1, 7),
                                   (6143, 1, 7), (40001, 1, 7), (515, 128, 32)])
def test_rows(T, F, N):
    import torch
    from paper_1904_07778_amd.xeng import requantize
    print(f"requant rows T={T} F={F} N={N}", flush=True)
    rng = np.random.default_rng(T + N)
    words = rng.integers(0, 2**64, size=(T, F, N), dtype=np.uint64)
    gains = rng.integers(0, 2**32, size=(F, N), dtype=np.uint64).astype(np.uint32)
    got = requantize(torch.from_numpy(words.view(np.int64)).cuda(), torch.from_numpy(gains.view(np.int32)).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), R.requantize(words, gains))
