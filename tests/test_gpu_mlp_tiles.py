"""Predictor network around the edges of its tiles: 16 particles a wave in
inference; 64 rows a workgroup in training (16 a wave), 256 workgroups that
then loop over tiles, the partial gradients summed 16 at a time."""
import numpy as np
import pytest
import torch  # noqa: F401

import oracle
from gpu_helpers import log
from oracle import mlp as M
from test_gpu_mlp import _pad, _params, _rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _dev():
    assert torch.cuda.is_available()
    from paper_1606_02738_amd import sph as S
    S.lib()
    oracle.build()


@pytest.mark.parametrize("n", [15, 17, 64, 65, 131073])
def test_forward_tile_edges(n):
    from paper_1606_02738_amd import sph as S
    log("case mlp forward n=%d" % n)
    p = _params(13)
    X, _ = _rows(n, 17)
    yg = S.mlp_forward(torch.from_numpy(p).cuda(), torch.from_numpy(X).cuda()).cpu().numpy()
    w = M.unpack(p.astype(np.float64))
    lay = M._layers(w, _pad(X.astype(np.float64)))
    yo = w["ymu"] + w["ysd"] * lay[-1]
    # three layers, each activation carried with a relative error of 2^-17
    # and summed in float32: bound by the magnitude of the output sum
    scale = np.abs(lay[-2]) @ np.abs(w["w4"]) + abs(w["b4"])
    assert (np.abs(yg - yo) / (w["ysd"] * scale)).max() < 2e-5


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 1025, 16384, 16385, 16448])
def test_loss_grad_tile_edges(n):
    from paper_1606_02738_amd import sph as S
    log("case mlp loss/grad n=%d" % n)
    p = _params(15)
    X, y = _rows(n, 19)
    t = [torch.from_numpy(a).cuda() for a in (p, X, y)]
    L, g = S.mlp_loss_grad(*t)
    L2, g2 = S.mlp_loss_grad(*t)
    assert L == L2 and torch.equal(g, g2)
    g = g.cpu().numpy().astype(np.float64)
    p64, X64 = p.astype(np.float64), _pad(X.astype(np.float64))
    Lo, go = M.loss_grad(p64, X64, y.astype(np.float64))
    # the residual is the output minus the target: its float32 error grows
    # with the output sum's magnitude over the residual's, and every entry of
    # the gradient carries the residual as a factor
    w = M.unpack(p64)
    lay = M._layers(w, X64)
    scale = (np.abs(lay[-2]) @ np.abs(w["w4"]) + abs(w["b4"])).max()
    tol = 1e-5 * (1.0 + scale / np.sqrt(2.0 * Lo))
    assert abs(L - Lo) <= 2 * tol * Lo
    for k in ("W1", "b1", "W2", "b2", "W3", "b3", "w4", "b4"):
        o, s = M.OFF[k]
        e = np.max(np.abs(g[o:o + s] - go[o:o + s])) / (np.max(np.abs(go[o:o + s])) + 1e-30)
        # entries of a block are sums of rows of both signs: ten times the
        # error of one row's factor
        assert e < 10 * tol, (k, e, tol)
