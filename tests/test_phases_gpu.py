"""Arrays whose time rows come in phases: calls of one integration that take
the staging and the ring kernel in turn, and phases added atomically (batched
plans keep no room for their sums), 4-byte and 16-byte loads.  Integer work:
equal to the oracle's."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import first_mismatch, gpu_available

pytestmark = pytest.mark.gpu
if not gpu_available():
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="no GPU")]


@pytest.mark.parametrize("shapes,lengths", [([(37, 301)], (100, 4096, 100)), ([(251, 5), (53, 3)], (3000, 7, 3000))])
def test_calls_of_one_integration(shapes, lengths):
    import torch
    from paper_1904_07778_amd.xeng import Plan
    print(f"phases {shapes} {lengths}", flush=True)
    rng = np.random.default_rng(len(lengths) + shapes[0][0])
    blocks = [[rng.integers(0, 256, size=(t, f, n), dtype=np.uint8) for n, f in shapes] for t in lengths]
    dev = [[torch.from_numpy(v).cuda() for v in b] for b in blocks]
    want = []
    for a, (n, f) in enumerate(shapes):
        e = oracle.Engine(n, f)
        for b in blocks:
            e.correlate(b[a])
        want.append(e.dump()[0])
    with Plan([(n, f, max(lengths)) for n, f in shapes]) as p:
        for _ in range(2):
            for b in dev[:-1]:
                p.correlate(b)
            out, n_int = p.correlate_dump(dev[-1])
            torch.cuda.synchronize()
            assert n_int == [sum(lengths)] * len(shapes)
            for o, w in zip(out, want):
                got = o.cpu().numpy()
                assert np.array_equal(got, w), first_mismatch(got, w)
