"""Cell build at the sizes where its kernels change: tiles of the small radix
sort (1024 keys) and its limit (65536), the limit of the two-launch permutation
(131072), one and several boxes."""
import numpy as np
import pytest
import torch

from gpu_helpers import log
from paper_1606_02738_amd import sph as S

pytestmark = pytest.mark.gpu

SIZES = [300, 1023, 1024, 1025, 4097, 65535, 65536, 65537, 131072, 131073]


def particles(n, n_boxes, seed):
    rng = np.random.default_rng(seed)
    d = {k: rng.random(n) for k in ("x", "y", "z")}
    d.update({k: rng.normal(0.0, 0.1, n) for k in ("vx", "vy", "vz", "ax", "ay", "az", "dudt", "rho", "drho_dH",
                                                   "omega", "P")})
    d["u"] = 1.0 + rng.random(n)
    d["m"] = np.full(n, 1.0 / n) * (1.0 + rng.random(n))
    d["H"] = np.full(n, min(0.3, 2.3 * (n_boxes / n) ** (1 / 3))) * (1.0 + 0.05 * rng.random(n))
    d["id"] = np.arange(n, dtype=np.int64)
    d["domain"] = rng.integers(0, n_boxes, n).astype(np.int32)
    return d


@pytest.mark.parametrize("n_boxes", [1, 3, 20])
@pytest.mark.parametrize("n", SIZES)
def test_build_permutes_every_array_and_is_sorted(n, n_boxes):
    log("case build n=%d boxes=%d" % (n, n_boxes))
    if n < 300 * n_boxes:
        pytest.skip("boxes of too few particles")
    d = particles(n, n_boxes, n + n_boxes)
    sim = S.SPH(np.ones((n_boxes, 3)), precision="fp32c")
    t = S.to_device(d)
    sim.bind(t)
    sim.build_cells()
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in t.items()}
    assert np.array_equal(np.sort(g["id"]), np.arange(n))
    for k in S.FLOAT_FIELDS + ("domain",):
        assert np.array_equal(g[k], d[k][g["id"]]), k
    assert np.all(np.diff(g["domain"]) >= 0)
    # a stable sort leaves what is sorted as it is
    sim.build_cells()
    torch.cuda.synchronize()
    assert np.array_equal(t["id"].cpu().numpy(), g["id"])
    assert sim.stats()["n_leaves"] >= n // 64
    sim.close()


def test_build_order_is_the_morton_order():
    """Cells of a level-0 grid come in its order, and their octants in theirs."""
    n = 5000
    d = particles(n, 1, 7)
    d["H"][:] = 0.12
    sim = S.SPH(np.ones((1, 3)), precision="fp64")
    t = S.to_device(d)
    sim.bind(t)
    sim.build_cells()
    torch.cuda.synchronize()
    p = np.stack([t[k].cpu().numpy() for k in "xyz"], 1)
    nt = 8  # floor(1 / 0.12), halved where such cells hold under 64 particles on average
    nt = nt // 2 if n < 64 * nt ** 3 else nt
    c = np.minimum((p * nt).astype(int), nt - 1)
    top = (c[:, 0] * nt + c[:, 1]) * nt + c[:, 2]
    o = ((p * nt - c) * 2).astype(int)
    assert np.all(np.diff(top * 8 + (o[:, 0] * 2 + o[:, 1]) * 2 + o[:, 2]) >= 0)
    sim.close()
