"""The channeliser's launch shapes against the float64 oracle, every output:
each FFT length, narrow and wide workgroups, units (a pair over a run of
spectra) that do not fill the last workgroup, odd pair counts whose
workgroups span several runs, and last runs shorter than the others."""
import numpy as np
import pytest

from oracle import channelise as C
from tests.gpu_util import gpu_available

pytestmark = pytest.mark.gpu
if not gpu_available():
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]

TOL = 2e-5   # float32 over at most 11 radix-2 levels and 4 taps, of the largest magnitude

# per F: a single spectrum, one more than a run, and enough for the wide form
SHAPES = [(F, N, S) for F, wide in ((8, 9000), (16, 5000), (32, 3000), (64, 1200), (128, 700), (256, 600), (512, 300),
                                    (1024, 211))
          for N, S in ((2, 1), (6, 5), (10, wide), (34, 17))]


@pytest.mark.parametrize("F,N,S", SHAPES)
def test_every_output(F, N, S):
    import torch
    from paper_1904_07778_amd.xeng import channelise
    print(f"channelise F={F} N={N} S={S}", flush=True)
    rng = np.random.default_rng(F * 1000 + N * 10 + S)
    x = rng.integers(-128, 128, size=(N, 2 * F * (S + 3))).astype(np.int8)
    out = torch.full((S + 1, F, N), float("nan"), dtype=torch.complex64, device="cuda")
    channelise(torch.from_numpy(x).cuda(), F, out=out[:S])
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    want = C.channelise(x, F)
    assert np.abs(got[:S] - want).max() <= TOL * np.abs(want).max()
    assert np.isnan(got[S].real).all()                 # nothing past the last spectrum
