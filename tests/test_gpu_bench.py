"""The layer benchmark times the form that a caller without options gets, and the separate
steps where an option names one of their forms."""
from __future__ import annotations

import pytest

import bench
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu

GMAS = ("k_gather", "k_gemm", "k_scatter", "k_scatter_centre", "k_conv_small")


@pytest.mark.parametrize("workload,opts,kernels", [
    (0, {}, {"k_conv_small"}),
    (2, {}, {"k_conv_small"}),
    (0, {"gather": "fused"}, {"k_gemm", "k_scatter"}),
    (0, {"gather": "buffer"}, {"k_gather", "k_gemm", "k_scatter"}),
    (2, {"partials": "f32"}, {"k_gemm", "k_scatter"}),
    (1, {}, {"k_gemm", "k_scatter_centre"}),
])
def test_layer_bench_form(workload, opts, kernels):
    say(f"layer bench {workload} {opts}")
    lb = bench.LayerBench(workload, None, **opts)
    try:
        kern = lb.kernels(R=1)
        assert {k for k in kern if k in GMAS} == kernels
        models = bench.kernel_models(lb.n, lb.n_out, lb.pairs, lb.L, lb.L.K ** 3, 1, fused=lb.fused, pelem=lb.pelem,
                                     centre=bool(lb.plan.centre))
        assert all(k in models or k == "k_gemm" for k in kernels)
    finally:
        lb.close()
