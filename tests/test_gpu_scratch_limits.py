"""Builds near the limit of their scratch: workspaces as small as ever held a
box, and octree levels of more cells than the room set aside for one."""
import numpy as np
import pytest
import torch

import gen
from gpu_helpers import log, oracle_run
from paper_1606_02738_amd import sph as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_side,least", [(12, 1790000), (16, 2185000), (20, 2890000), (40, 13410000)])
def test_small_workspace_holds(n_side, least):
    """The least workspaces of an octree that worked level by level (measured
    for these boxes, and half a percent).  What a build only borrows is not
    reported as needed."""
    log("case lattice %d^3 in %d bytes" % (n_side, least))
    d = gen.lattice(n_side, vsigma=0.1, seed=71)
    high = []
    for size in (least, 1 << 28):
        sim = S.SPH(d["box"], precision="fp32c", workspace_bytes=size)
        # (bind() only makes a context's first workspace larger)
        sim.close()
        sim._create(size)
        t = S.to_device(d)
        sim.bind(t)
        sim.run()
        for _ in range(2):
            sim.step(1e-5)
        torch.cuda.synchronize()
        high.append(sim.stats()["workspace_high"])
        sim.close()
    log("high %d and %d" % tuple(high))
    assert high[1] < 1.1 * least


@pytest.mark.parametrize("n_side", [9, 27, 64])
def test_levels_of_more_cells_than_expected(n_side):
    """Smoothing lengths far below the spacing: in the FP32 modes every particle
    gets a cell of its own, where up to 64 would share one.  The first build borrows
    its room, the second has lists of one entry a leaf.  Beyond 65536 cells a
    workgroup writes the children of several sets of cells."""
    log("case one particle a leaf, %d^3" % n_side)
    d = gen.lattice(n_side, vsigma=0.1, seed=72)
    n = d["x"].size
    sim = S.SPH(d["box"], precision="fp32c")
    t = S.to_device(d)
    H = t["H"].clone()
    t["H"][1:] *= 1e-3  # (the first one keeps the top cells as they are)
    sim.bind(t)
    for _ in range(2):
        sim.build_cells()
        st = sim.stats()
        assert st["n_leaves"] == n and st["n_list"] >= n
        ids = t["id"].cpu().numpy()
        assert np.array_equal(np.sort(ids), np.arange(n))
        for k in ("x", "vz", "m"):
            assert np.array_equal(t[k].cpu().numpy(), d[k][ids]), k
        # another order for the next build
        mix = torch.randperm(n, generator=torch.Generator().manual_seed(n)).cuda()
        for v in t.values():
            v.copy_(v[mix])
    t["H"].copy_(H[t["id"]])
    sim.run()
    g = S.to_host(t)
    sim.close()
    if n < 20000:
        o = oracle_run(d)
        assert np.max(np.abs(g["rho"] - o["rho"]) / o["rho"]) < 1e-5
        assert np.max(np.abs(g["H"] - o["H"]) / o["H"]) < 1e-5
