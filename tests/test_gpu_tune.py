"""The per-layer tuning times what it names: the separate steps of every layer, also of
those that run as one kernel by default, and leaves the latter at their defaults."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2401_06145_amd import binding as B
from paper_2401_06145_amd import net, scenes, tune
from tests.gpu_helpers import DEV, say, to_dev

pytestmark = pytest.mark.gpu


def _row(K, c_in, c_out):
    coords = scenes.uniform_cells(3000, 20, 4000)
    km = B.KernelMap.build(to_dev(coords), K)
    op = net.Op("conv", "y", "x", 0, K, "subm", c_in, c_out)
    x = torch.randn(km.n_in, c_in, device=DEV).half()
    w = torch.randn(K ** 3, c_in, c_out, device=DEV).half()
    return tune.tune_layer(km, op, x, w, None, 2, rows_cands=(64, 512))


@pytest.mark.parametrize("K,c_in,c_out,one", [(3, 16, 32, True), (1, 64, 96, True), (3, 96, 64, False)])
def test_tune_layer(K, c_in, c_out, one):
    say(f"tune K={K} {c_in}->{c_out}")
    row = _row(K, c_in, c_out)
    assert row["one_kernel"] == one
    assert min(row["scatter_us"].values()) > 0 and min(row["gather_us"].values()) > 0
    assert K == 1 or (set(row["gemm_us"]) == {0, 64, 512} and min(row["gemm_us"].values()) > 0)
    opts = tune.tuned_options({"y": row})
    assert ("y" in opts) != one


def test_timed_refuses_a_kernel_that_does_not_run():
    say("timed kernel that does not run")
    coords = scenes.uniform_cells(500, 20, 4000)
    km = B.KernelMap.build(to_dev(coords), 3)
    x = to_dev(scenes.features(km.n_in, 16, "f16", 1))
    w = to_dev(scenes.weights(3, 16, 16, "f16", 2))
    f = B.Forward(km, 16, 16, torch.float16)
    with pytest.raises(RuntimeError):
        tune._timed(lambda: f(x, w), "k_gather", 1)
    assert np.isfinite(tune._timed(lambda: f(x, w), "k_conv_small", 1))
