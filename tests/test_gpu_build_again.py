"""Builds after the first, which move the arrays in groups through the last
lists: every array must follow its particle from any order into the new one."""
import numpy as np
import pytest
import torch

from gpu_helpers import log
from paper_1606_02738_amd import sph as S
from test_gpu_build_sizes import particles

pytestmark = pytest.mark.gpu


def compare(t, d):
    g = {k: v.cpu().numpy() for k, v in t.items()}
    assert np.array_equal(np.sort(g["id"]), np.arange(g["id"].size))
    for k in S.FLOAT_FIELDS + ("domain",):
        assert np.array_equal(g[k], d[k][g["id"]]), k
    assert np.all(np.diff(g["domain"]) >= 0)
    return g["id"]


@pytest.mark.parametrize("n_boxes", [1, 3, 20])
@pytest.mark.parametrize("n", [131071, 131073, 200001, 400000])
@pytest.mark.parametrize("n_split", [8, 64])
def test_later_builds_permute_every_array(n, n_boxes, n_split):
    """(8 particles a leaf: more rows of the group fit the longer lists)"""
    log("case build again n=%d boxes=%d n_split=%d" % (n, n_boxes, n_split))
    d = particles(n, n_boxes, n + n_boxes)
    sim = S.SPH(np.ones((n_boxes, 3)), precision="fp32c", n_split=n_split, workspace_bytes=1 << 30)
    t = S.to_device(d)
    sim.bind(t)
    sim.build_cells()
    torch.cuda.synchronize()
    ids = compare(t, d)
    g = torch.Generator().manual_seed(n)
    for _ in range(3):
        mix = torch.randperm(n, generator=g).cuda()
        for v in t.values():
            v.copy_(v[mix])
        sim.build_cells()
        torch.cuda.synchronize()
        again = compare(t, d)
        assert sim.stats()["n_leaves"] >= n // 64
        # the order of the cells; within the finest ones it is that of the input
        assert np.array_equal(d["domain"][again], d["domain"][ids])
    sim.close()


def test_steps_permute_every_array():
    """The builds inside a step leave out what the step rewrites."""
    log("case steps with a build each")
    import gen
    d = gen.lattice(54, vsigma=0.1, seed=91)
    n = d["x"].size
    rng = np.random.default_rng(92)
    d["m"] = d["m"] * (1.0 + 0.01 * rng.random(n))
    mix = rng.permutation(n)
    e = {k: v[mix] if isinstance(v, np.ndarray) and v.shape == (n,) and k != "id" else v for k, v in d.items()}
    sim = S.SPH(d["box"], precision="fp32c")
    t = S.to_device(e)
    sim.bind(t)
    sim.run()
    dt = 1e-4
    for _ in range(3):
        sim.step(dt)
    torch.cuda.synchronize()
    assert sim.stats()["n_builds"] == 4
    g = S.to_host(t)
    assert np.array_equal(g["m"], e["m"])
    for a, v in zip("xyz", ("vx", "vy", "vz")):
        dx = g[a] - e[a] - 3 * dt * e[v]
        dx -= np.round(dx)
        assert np.max(np.abs(dx)) < 1e-5, a  # (dt^2 times the accelerations)
        assert np.max(np.abs(g[v] - e[v])) < 0.1, v
    # densities belong to their particles: the neighbours' masses around them
    sim2 = S.SPH(d["box"], precision="fp32c")
    f = {k: (g[k] if k in ("x", "y", "z", "vx", "vy", "vz", "u", "m", "H") else v) for k, v in e.items()}
    s = S.to_device(f)
    sim2.bind(s)
    sim2.run()
    h = S.to_host(s)
    for k in ("rho", "H", "omega", "P"):
        assert np.max(np.abs(g[k] - h[k]) / np.abs(h[k])) < 1e-4, k
    sim.close()
    sim2.close()
