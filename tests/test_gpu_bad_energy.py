"""The matrix-unit range tests let in pairs slightly out of range, which add
exact zeros.  A particle whose factor is no number (its internal energy is
not) must not reach particles through such a pair."""
import numpy as np
import pytest
import torch  # noqa: F401
from scipy.spatial import cKDTree

import gen
from gpu_helpers import gpu_run, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_split", [64, 8])
@pytest.mark.parametrize("prec", ["fp32c", "fp64"])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_bad_energy_stays_in_its_range(bad, prec, n_split):
    log("case energy %s %s n_split=%d" % (bad, prec, n_split))
    d = gen.lattice(40, vsigma=0.1, seed=61)
    k = np.random.default_rng(62).choice(d["x"].size, 400, replace=False)
    a, st = gpu_run(d, precision=prec, force="gather", n_split=n_split)
    # every leaf by several waves, or one wave a leaf
    assert (st["n_leaves"] > 2048) == (n_split == 8)
    e = dict(d, u=d["u"].copy())
    e["u"][k] = bad
    b, _ = gpu_run(e, precision=prec, force="gather", n_split=n_split)
    p = np.stack([d[f] for f in "xyz"], 1)
    H = a["H"]
    near = np.zeros(H.size, dtype=bool)
    tree = cKDTree(p, boxsize=1.0)
    for q, j in zip(k, tree.query_ball_point(p[k], float(H.max()) * 1.001)):
        j = np.asarray(j)
        dx = p[j] - p[q]
        dx -= np.round(dx)
        r = np.sqrt((dx ** 2).sum(1))
        near[j[r < np.maximum(H[j], H[q]) * (1 + 1e-5)]] = True
    assert H.size / 2 < np.sum(~near)
    for f in ("ax", "ay", "az", "dudt"):
        wrong = np.sum(a[f][~near] != b[f][~near])
        assert wrong == 0, (f, wrong)
