"""channelise() with an output of the caller's allocates nothing, and gives
what the form with a table workspace gives."""
import pytest

from tests.gpu_util import gpu_available

pytestmark = pytest.mark.gpu
if not gpu_available():
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


def test_no_table_allocation():
    import torch
    from paper_1904_07778_amd.xeng import _lib, channelise
    F, N, S = 64, 6, 5
    gen = torch.Generator(device="cuda").manual_seed(3)
    adc = torch.randint(-128, 128, (N, 2 * F * (S + 3)), dtype=torch.int8, device="cuda", generator=gen)
    tables = torch.empty(int(_lib.xeng_channelise_table_floats(F)), dtype=torch.float32, device="cuda")
    want = channelise(adc, F, tables=tables)
    out = torch.full_like(want, float("nan"))
    made = torch.cuda.memory_stats()["allocation.all.allocated"]
    channelise(adc, F, out=out)
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == made
    torch.cuda.synchronize()
    assert torch.equal(out, want)
