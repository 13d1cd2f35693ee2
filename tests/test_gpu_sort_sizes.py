"""The radix sort on both sides of the sizes where its passes change form
(65536 keys; 1024 blocks of its histogram, 16777216 keys), through the
interpolation, whose points it orders: every point must get its own value."""
import numpy as np
import pytest
import torch

import gen
from gpu_helpers import log
from paper_1606_02738_amd import sph as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sim():
    d = gen.lattice(12, jitter=0.2, seed=7711)
    s = S.SPH(d["box"], precision="fp64", workspace_bytes=2 << 30)
    t = S.to_device(d)
    s.bind(t)
    s.run()
    q = torch.from_numpy(np.random.default_rng(7712).normal(size=d["x"].size)).cuda()
    yield s, q
    s.close()


@pytest.mark.parametrize("n", [65535, 65537, 1 << 22, (1 << 24) - 1, 1 << 24, (1 << 24) + 1, (1 << 24) + 70001])
def test_every_point_gets_its_value(sim, n):
    s, q = sim
    log("case sort of %d points" % n)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    # points from a small set, in any order: the value of each is known
    few = [torch.rand(1000, generator=g, device="cuda", dtype=torch.float64) for _ in range(3)]
    want = s.interpolate(q, *few)
    i = torch.randint(0, 1000, (n,), generator=g, device="cuda")
    got = s.interpolate(q, *(a[i].contiguous() for a in few))
    # the same terms in another order: a few hundred roundings of 2^-53
    assert torch.max(torch.abs(got - want[i])).item() <= 1e-12 * torch.max(torch.abs(want)).item()
