"""GPU parity of the one-kernel form of narrow layers (all K^3 weight matrices in LDS).

Features against the oracle at the sizes where the kernel's blocks, groups and pieces
end.  Sums are float32 throughout and rounded once, so 16-bit results are within one
rounding of the oracle's: 2^-11 (f16) or 2^-8 (bf16) of max |y|, doubled with a residual
whose own value takes part in the rounding; float32 within the common tolerance.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2401_06145_amd import binding as B
from paper_2401_06145_amd import scenes
from tests.gpu_helpers import TOL, forward_kernels, rel_err, say, to_dev, to_f64

pytestmark = pytest.mark.gpu

ROUNDING = {"f32": TOL["f32"], "f16": 2.0 ** -11 * 1.05, "bf16": 2.0 ** -8 * 1.05}


def _cloud(seed, n, side):
    rng = np.random.default_rng(seed)
    cells = rng.choice(side ** 3, n, replace=False)
    c = np.stack([np.zeros(n), cells // side ** 2, cells // side % side, cells % side], 1).astype(np.int32)
    return np.ascontiguousarray(c)


def _layer(K, c_in, c_out, dtype, coords, mode="subm", seed=1):
    stride = 1 if mode == "subm" else 2
    q = None if mode == "subm" else oracle.out_coords(coords, 2, 1)
    km = B.KernelMap.build(to_dev(coords), K, stride, 1, "subm" if mode == "subm" else "down")
    if mode == "up":
        km = km.transpose()
        okm = oracle.kernel_map(q, coords, K, 1, "up")
    else:
        okm = oracle.kernel_map(coords, q, K, 1, mode)
    x = scenes.features(km.n_in, c_in, dtype, seed)
    w = scenes.weights(K, c_in, c_out, dtype, seed + 1)
    ref = oracle.features(scenes.to_f64(x, dtype), scenes.to_f64(w, dtype), okm)
    return km, okm, x, w, ref


@pytest.mark.parametrize("dtype,K,c_in,c_out,mode,n", [
    ("f16", 3, 32, 32, "subm", 1),        # one row
    ("f16", 3, 32, 64, "subm", 16),       # one block
    ("f16", 3, 48, 32, "subm", 17),       # two k-steps, the second half empty; a block and a row
    ("bf16", 3, 16, 48, "subm", 127),     # two offsets per k-step; odd tiles; eight dies less one block
    ("bf16", 3, 8, 16, "subm", 2049),     # four offsets per k-step, one tile
    ("f16", 5, 8, 32, "subm", 3001),      # 125 offsets: five groups, the last of 13
    ("f16", 2, 24, 96, "subm", 3000),     # eight offsets: two entries per lane; a quarter k-step empty
    ("f16", 1, 64, 128, "subm", 3000),
    ("f16", 2, 96, 96, "up", 3000),       # three k-steps
    ("bf16", 2, 64, 128, "down", 3000),
    ("bf16", 3, 32, 64, "down", 3000),
    ("f32", 3, 16, 16, "subm", 3000),
    ("f32", 3, 4, 32, "subm", 3000),      # four offsets per k-step
    ("f32", 3, 8, 16, "up", 3000),
    ("f32", 3, 32, 32, "subm", 9000),
    ("f32", 1, 48, 96, "subm", 500),
])
def test_narrow_layer_matches_oracle(dtype, K, c_in, c_out, mode, n):
    say(f"one-kernel layer {dtype} K={K} {c_in}->{c_out} {mode} n={n}")
    coords = _cloud(900 + n + K, n, 40 if n > 5000 else 16)
    km, _, x, w, ref = _layer(K, c_in, c_out, dtype, coords, mode)
    f = B.Forward(km, c_in, c_out, B.TORCH_DTYPES[dtype])
    xd, wd = to_dev(x, dtype), to_dev(w, dtype)
    y = f(xd, wd)
    assert rel_err(to_f64(y), ref) <= ROUNDING[dtype]
    assert torch.equal(f(xd, wd), y)  # repeatable bit for bit
    # the separate steps (named by an option) stay within the common tolerance of it
    sep = B.Forward(km, c_in, c_out, B.TORCH_DTYPES[dtype], B.Options.make(gather=B.GATHER_FUSED))(xd, wd)
    assert rel_err(to_f64(sep), to_f64(y)) <= TOL[dtype]
    if dtype == "f32" and n >= 2000:
        # both sum an offset's channels first and then the offsets, so their errors differ
        # by chance only, over 32,000 outputs or more; one chain over both is 1.5 to 2 times
        # as far off
        assert np.linalg.norm(to_f64(y) - ref) <= 1.25 * np.linalg.norm(to_f64(sep) - ref)
    res = scenes.features(km.n_out, c_out, dtype, 7)
    ye = f(xd, wd, residual=to_dev(res, dtype), relu=True)
    assert rel_err(to_f64(ye), np.maximum(ref + scenes.to_f64(res, dtype), 0.0)) <= 2 * ROUNDING[dtype]


@pytest.mark.parametrize("dtype,c_in", [("f16", 32), ("bf16", 16), ("f32", 16)])
def test_weights_that_are_not_finite(dtype, c_in):
    """An infinite weight reaches the outputs that have a pair at its offset, and no
    others (rows without a pair are not multiplied by it)."""
    say(f"non-finite weight {dtype} c_in={c_in}")
    coords = _cloud(77, 1500, 16)
    km, okm, x, w, _ = _layer(3, c_in, 32, dtype, coords)
    xd, wd = to_dev(x, dtype), to_dev(w, dtype)
    wd[5, 0, 3] = float("inf")
    y = to_f64(B.Forward(km, c_in, 32, B.TORCH_DTYPES[dtype])(xd, wd))
    reached = np.zeros(len(coords), dtype=bool)
    a, b = okm.pairs(5)
    reached[b[scenes.to_f64(x, dtype)[a, 0] != 0]] = True
    assert 0 < reached.sum() < len(coords)
    assert not np.isfinite(y[reached, 3]).any() and np.isfinite(y[~reached, 3]).all()
    w0 = scenes.to_f64(w, dtype)
    w0[5, :, 3] = 0
    ref = oracle.features(scenes.to_f64(x, dtype), w0, okm)
    keep = np.ones(32, dtype=bool)
    keep[3] = False
    assert rel_err(y[:, keep], ref[:, keep]) <= ROUNDING[dtype]


def test_output_over_the_input():
    """A layer whose output buffer is its input keeps the separate steps, which read all
    inputs before the first output is written (float32, no centre in the scatter)."""
    say("output over the input")
    coords = _cloud(78, 3000, 16)
    km, _, x, w, ref = _layer(3, 16, 16, "f32", coords)
    xd, wd = to_dev(x), to_dev(w)
    f = B.Forward(km, 16, 16, torch.float32)
    assert f(xd, wd, y=xd) is xd
    assert rel_err(to_f64(xd), ref) <= TOL["f32"]


@pytest.mark.parametrize("dtype,c_in,c_out", [("f16", 16, 128), ("f32", 16, 64)])
def test_output_of_64_mib(dtype, c_in, c_out):
    """Outputs past the size from which the scatter streams its rows.  One offset, so that
    every output is one product: 2^-11 or float32 rounding of 16 terms."""
    say(f"output of 64 MiB {dtype}")
    coords = _cloud(79, 300_001, 70)
    km = B.KernelMap.build(to_dev(coords), 1)
    x = to_dev(scenes.features(km.n_in, c_in, dtype, 3), dtype)
    w = to_dev(scenes.weights(1, c_in, c_out, dtype, 4), dtype)
    y = B.Forward(km, c_in, c_out, B.TORCH_DTYPES[dtype])(x, w)
    assert y.numel() * y.element_size() >= 1 << 26
    ref = x.double() @ w[0].double()
    assert float((y.double() - ref).abs().max() / ref.abs().max()) <= ROUNDING[dtype]


@pytest.mark.parametrize("c_in", [4, 8, 16, 20])
def test_error_beside_a_weight_that_is_not_finite(c_in):
    """Columns without the infinite weight are as accurate as in separate steps, which sum an
    offset's channels first and then the offsets: the errors differ by chance only, over
    90,000 outputs of 19 pairs (one chain over both is 1.5 to 2.6 times as far off).  Four, two
    and one offsets per k-step, and two k-steps."""
    say(f"error beside a non-finite weight c_in={c_in}")
    c_out = 16 if c_in == 20 else 32
    coords = _cloud(80, 3000, 16)
    km, okm, x, w, _ = _layer(3, c_in, c_out, "f32", coords)
    w[5, 0, 3] = np.inf
    xd, wd = to_dev(x), to_dev(w)
    f = B.Forward(km, c_in, c_out, torch.float32)
    assert forward_kernels(lambda: f(xd, wd)) == {"k_conv_small": 1}
    w[5, 0, 3] = 0
    ref = oracle.features(x, w, okm)
    keep = np.arange(c_out) != 3
    err = [np.linalg.norm((to_f64(B.Forward(km, c_in, c_out, torch.float32, o)(xd, wd)) - ref)[:, keep])
           for o in (None, B.Options.make(gather=B.GATHER_FUSED))]
    assert err[0] <= 1.25 * err[1]
