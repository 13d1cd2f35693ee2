"""Edges of the candidate tiles of the density and gather force kernels:
leaves that end inside, on and past a block of 16 particles, tiles with more
pairs than are listed at a time, coordinates far from order 1, and values that
must not spread from one particle to those out of its range."""
import numpy as np
import pytest
import torch  # noqa: F401

import gen
import oracle
from gpu_helpers import TOL_FP32, TOL_FP64, assert_close, gpu_run, log, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_split", [1, 15, 16, 17, 33, 49, 64])
@pytest.mark.parametrize("prec", ["fp64", "fp32c"])
def test_leaf_sizes(prec, n_split):
    log("case leaf sizes %s n_split=%d" % (prec, n_split))
    d = gen.lattice(14, vsigma=0.1, seed=31)
    g, st = gpu_run(d, precision=prec, n_split=n_split, force="gather")
    assert_close(g, oracle_run(d), TOL_FP64 if prec == "fp64" else TOL_FP32, counts_exact=prec == "fp64",
                 stats=st if prec == "fp64" else None)


@pytest.mark.parametrize("prec", ["fp64", "fp32c"])
def test_more_pairs_than_listed_at_once(prec):
    """About 450 neighbours a particle: most tiles hold several lists of pairs."""
    log("case many neighbours %s" % prec)
    d = gen.lattice(16, vsigma=0.1, seed=32)
    d["H"] = d["H"] * 2.1
    g, st = gpu_run(d, precision=prec, force="gather", eta=gen.ETA * 2.1)
    o = oracle.full(d, tree=True, eta=gen.ETA * 2.1)
    assert st["n_dens"] > 400 * g["x"].size
    assert_close(g, o, TOL_FP64 if prec == "fp64" else TOL_FP32, counts_exact=prec == "fp64",
                 stats=st if prec == "fp64" else None)


@pytest.mark.parametrize("k", [-20, 20])
def test_power_of_two_scale_is_exact(k):
    """Lengths times 2^k: every operation scales exactly, so the results are
    the unit box's bit for bit."""
    log("case scale 2^%d" % k)
    d = gen.clustered(24, n_halos=12, seed=33)
    s = 2.0 ** k
    e = dict(d, box=d["box"] * s, boxes=d["boxes"] * s)
    for f in ("x", "y", "z", "H"):
        e[f] = d[f] * s
    a, _ = gpu_run(d, force="gather")
    b, _ = gpu_run(e, force="gather")
    # v stays: du/dt scales like the inverse length
    for f, p in (("H", 1), ("rho", -3), ("drho_dH", -4), ("omega", 0), ("P", -3), ("ax", -1), ("ay", -1), ("az", -1),
                 ("dudt", -1)):
        assert np.array_equal(b[f], a[f] * s ** p), f
    assert np.array_equal(a["nngb"], b["nngb"])


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_bad_velocity_stays_in_its_range(bad):
    """A particle with a velocity that is no number changes du/dt only where
    r < max(H_i, H_j)."""
    log("case velocity %s" % bad)
    d = gen.lattice(12, vsigma=0.1, seed=34)
    k = 700
    a, _ = gpu_run(d, force="gather")
    e = dict(d, vx=d["vx"].copy())
    e["vx"][k] = bad
    b, _ = gpu_run(e, force="gather")
    dx = np.stack([d[f] - d[f][k] for f in "xyz"], 1)
    dx -= np.round(dx)
    r = np.sqrt((dx ** 2).sum(1))
    far = r >= np.maximum(a["H"], a["H"][k]) * (1 + 1e-5)
    assert 0 < np.sum(~far) < 100
    for f in ("ax", "ay", "az", "dudt", "rho"):
        assert np.array_equal(a[f][far], b[f][far]), f
    assert np.isfinite(b["ax"]).all()


@pytest.mark.parametrize("prec,mode", [("fp64", "grid"), ("fp64", "persistent"), ("fp32c", "persistent")])
def test_long_lists_are_shared_among_waves(prec, mode):
    """More than 2048 leaves, so that one wave takes a leaf and several waves
    the leaves with long lists (next to a halo); below that, in the other
    tests of this file, several waves take every leaf."""
    log("case long lists %s %s" % (prec, mode))
    d = gen.clustered(32, n_halos=4, seed=35, halo_frac=0.6)
    g, st = gpu_run(d, precision=prec, exec_mode=mode, n_split=8, force="gather")
    assert st["n_leaves"] > 2048
    assert_close(g, oracle_run(d), TOL_FP64 if prec == "fp64" else TOL_FP32, counts_exact=prec == "fp64",
                 stats=st if prec == "fp64" else None)
