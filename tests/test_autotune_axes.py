"""The autotuner's second stage: candidates that launch the same kernels are
timed once, and the choice among them is the default (no GPU)."""
import numpy as np
import pytest
import torch

from paper_1606_02738_amd import autotune as AT

CELL = dict(n_split=64, exec_mode="grid", persistent_wgs=0, prune="box", use_graph=False, rebuild_steps=8,
            force="gather")


def tune(monkeypatch, base, leaves, fast=None):
    """autotune() over `base` alone with every timing a little below the one
    before, and that of `fast` a density value far below."""
    calls = []

    def time_config(boxes, t, state, cfg, precision, dt, steps, warmup):
        calls.append(cfg)
        ms = 10.0 - 0.01 * len(calls)
        return (5.0 if fast and cfg.get("waves_density") == fast else ms), leaves

    monkeypatch.setattr(AT, "_time_config", time_config)
    monkeypatch.setattr(AT, "_key", lambda *a: "k")
    best, table = AT.autotune(np.ones((1, 3)), {"H": torch.ones(4)}, "fp32c", 1e-3, cands=[base], cache=None)
    return best, table, calls


def test_axes_without_kernels_are_not_timed(monkeypatch):
    best, table, calls = tune(monkeypatch, CELL, 5000)
    assert [c.get("waves_density", 0) for c in calls] == [0, 4, 6]
    assert len(table) == 2 + len(AT.kernel_candidates(CELL))
    # (the later timing wins, and no value of the axes that do nothing with it)
    assert best["waves_density"] == 6 and best["waves_force"] == 0 and best["batch"] == 0


@pytest.mark.parametrize("fast", [4, 6])
def test_faster_density_form_is_chosen(monkeypatch, fast):
    best, _, _ = tune(monkeypatch, CELL, 5000, fast)
    assert best == dict(CELL, waves_density=fast, waves_force=0, batch=0)


@pytest.mark.parametrize("base,leaves", [(CELL, 2048), (dict(CELL, lists="particle"), 5000),
                                         (dict(CELL, prune="sorted", force="pairs"), 5000)])
def test_no_axis_has_kernels_here(monkeypatch, base, leaves):
    best, table, calls = tune(monkeypatch, base, leaves)
    assert len(calls) == 1
    assert best == dict(base, waves_density=0, waves_force=0, batch=0)
    assert len({ms for _, ms in table}) == 1


def test_wide_all_is_the_library_s():
    import os
    import re
    h = open(os.path.join(os.path.dirname(AT.__file__), "csrc", "sph_internal.h")).read()
    assert int(re.search(r"#define SPH_WIDE_ALL (\d+)", h).group(1)) == AT.WIDE_ALL
