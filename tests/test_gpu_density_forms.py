"""The density kernel's forms of one wave a leaf, which boxes of more than 2048
leaves run: every occupancy target gives the default's results bit for bit, and
the default's agree with the oracle."""
import numpy as np
import pytest
import torch  # noqa: F401

import gen
from gpu_helpers import TOL_FP32, assert_close, gpu_run, log, oracle_run

pytestmark = pytest.mark.gpu

KEYS = ("rho", "H", "omega", "P", "ax", "ay", "az", "dudt", "nngb")


@pytest.fixture(scope="module")
def box():
    d = gen.clustered(32, n_halos=4, seed=35, halo_frac=0.6)
    return d, {p: gpu_run(d, precision=p, n_split=8, force="gather") for p in ("fp32c", "fp32")}


@pytest.mark.parametrize("prec", ["fp32c", "fp32"])
def test_default_form(box, prec):
    log("case default form, %s" % prec)
    d, ref = box
    g, st = ref[prec]
    assert st["n_leaves"] > 2048
    assert_close(g, oracle_run(d), TOL_FP32, counts_exact=False)


@pytest.mark.parametrize("prec", ["fp32c", "fp32"])
@pytest.mark.parametrize("waves", [4, 5, 6, 8])
def test_form_is_bit_identical_to_default(box, waves, prec):
    log("case density at %d waves, %s" % (waves, prec))
    d, ref = box
    g, st = gpu_run(d, precision=prec, n_split=8, force="gather", waves_density=waves)
    assert st["n_leaves"] > 2048
    for k in KEYS:
        assert np.array_equal(g[k], ref[prec][0][k]), k
