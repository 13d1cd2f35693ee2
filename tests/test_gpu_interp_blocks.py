"""Interpolation in blocks of points: group sizes from 1 to 64 points a wave,
ragged ends, blocks that split (several boxes, jumps of the Morton order),
lists of leaves longer than a wave holds, repeated and invalid points.  The
value at a point must not depend on the points around it, and is checked
against the oracle's brute-force sum on a subset."""
import numpy as np
import pytest
import torch  # noqa: F401

import gen
import oracle
from gpu_helpers import log, oracle_run
from oracle import interp as OI
from test_gpu_interp import _gpu_interp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _dev():
    assert torch.cuda.is_available()
    from paper_1606_02738_amd import sph as S
    S.lib()
    oracle.build()


@pytest.fixture(scope="module")
def clustered():
    from paper_1606_02738_amd import sph as S
    d = gen.clustered(20, n_halos=6, seed=5511)
    Q = np.random.default_rng(5512).normal(size=d["x"].size)
    sim = S.SPH(d["box"], precision="fp64")
    t = S.to_device(d)
    sim.bind(t)
    sim.run()
    yield sim, t, d, Q, oracle_run(d)
    sim.close()


def _cloud(d, n, seed):
    """Points: uniform, around particles (dense regions), repeated, and NaN."""
    rng = np.random.default_rng(seed)
    P = rng.random((n, 3))
    near = rng.random(n) < 0.5
    i = rng.integers(0, d["x"].size, n)
    P[near] = np.stack([d["x"], d["y"], d["z"]], 1)[i[near]] + 1e-3 * rng.normal(size=(near.sum(), 3))
    P[n // 3:n // 3 + n // 50] = P[n // 3]
    P[n // 2] = np.nan
    return P


@pytest.mark.parametrize("n", [1, 7, 4095, 8192, 16385, 70001, 262144, 300007])
def test_values_do_not_depend_on_the_group(clustered, n):
    sim, t, d, Q, o = clustered
    log("case interp blocks n=%d" % n)
    P = _cloud(d, n, 5513)
    g = _gpu_interp(sim, t, Q, *(P[:, a].copy() for a in range(3)))
    assert np.array_equal(g, _gpu_interp(sim, t, Q, *(P[:, a].copy() for a in range(3))), equal_nan=True)
    bad = np.isnan(P[:, 0])
    assert np.isnan(g[bad]).all() and np.isfinite(g[~bad]).all()
    sub = np.random.default_rng(5514).choice(n, min(n, 300), replace=False)
    sub = sub[~bad[sub]]
    if sub.size == 0:
        return
    p = [P[sub, a].copy() for a in range(3)]
    args = (d["x"], d["y"], d["z"], d["m"], o["rho"], o["H"])
    sa = np.maximum(OI.interpolate(*p, *args, np.abs(Q), d["box"]), 1e-300)
    # the same terms in another order: a few hundred roundings of 2^-53
    assert np.max(np.abs(_gpu_interp(sim, t, Q, *p) - g[sub]) / sa) < 1e-12
    # against the oracle's own H and rho: the solver's tolerance
    assert np.max(np.abs(g[sub] - OI.interpolate(*p, *args, Q, d["box"])) / sa) < 1e-7


def test_long_leaf_lists():
    """Cells of one or two particles and 64-point blocks as wide as a top
    cell: a block's reach holds more leaves than a wave lists at a time."""
    from paper_1606_02738_amd import sph as S
    rng = np.random.default_rng(5521)
    d = gen.lattice(24, jitter=0.2, seed=5522)
    sim = S.SPH(d["box"], precision="fp64", n_split=2)
    t = S.to_device(d)
    sim.bind(t)
    sim.run()
    Q = rng.normal(size=d["x"].size)
    log("case interp long lists: %d leaves" % sim.stats()["n_leaves"])
    # most points in one spot, so that the groups are of 64 and the others'
    # blocks wide
    q = rng.random((3000, 3))
    P = np.concatenate([q, 0.9 + 1e-3 * rng.random((262144, 3))])
    P = [P[:, a].copy() for a in range(3)]
    p = [q[:, a].copy() for a in range(3)]
    g = _gpu_interp(sim, t, Q, *P)[:3000]
    one = _gpu_interp(sim, t, Q, *p)
    sim.close()
    o = oracle_run(d)
    args = (d["x"], d["y"], d["z"], d["m"], o["rho"], o["H"])
    sa = OI.interpolate(*p, *args, np.abs(Q), d["box"])
    assert np.max(np.abs(one - g) / sa) < 1e-12
    assert np.max(np.abs(one - OI.interpolate(*p, *args, Q, d["box"])) / sa) < 1e-7


@pytest.mark.parametrize("n", [500, 300000])
def test_blocks_of_several_boxes(n):
    from paper_1606_02738_amd import sph as S
    rng = np.random.default_rng(5531)
    d = gen.ensemble(3, (10, 14), seed=5532)
    sim = S.SPH(d["boxes"], precision="fp64")
    t = S.to_device(d)
    sim.bind(t)
    sim.run()
    Q = rng.normal(size=d["x"].size)
    pd = rng.integers(0, 4, n).astype(np.int32)  # 3: no such box
    P = rng.random((n, 3)) * np.concatenate([d["boxes"], [[1.0, 1.0, 1.0]]])[pd]
    log("case interp blocks of several boxes n=%d" % n)
    g = _gpu_interp(sim, t, Q, *(P[:, a].copy() for a in range(3)), pdom=pd)
    sim.close()
    assert np.isnan(g[pd == 3]).all()
    o = oracle_run(d)
    for k, b in enumerate(oracle.split_domains(d)):
        sub = np.nonzero(pd == k)[0][:100]
        ix = b["index"]
        p = [P[sub, a].copy() for a in range(3)]
        args = (b["x"], b["y"], b["z"], b["m"], o["rho"][ix], o["H"][ix])
        sa = np.maximum(OI.interpolate(*p, *args, np.abs(Q[ix]), b["box"]), 1e-300)
        assert np.max(np.abs(g[sub] - OI.interpolate(*p, *args, Q[ix], b["box"])) / sa) < 1e-7
