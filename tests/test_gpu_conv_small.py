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
    return scenes.uniform_cells(n, side, seed)


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


def _check(dtype, K, c_in, c_out, mode, n, side, one):
    """Parity of the default form, which is one kernel or not, and of the separate steps."""
    coords = _cloud(900 + n + K, n, side)
    km, _, x, w, ref = _layer(K, c_in, c_out, dtype, coords, mode)
    f = B.Forward(km, c_in, c_out, B.TORCH_DTYPES[dtype])
    xd, wd = to_dev(x, dtype), to_dev(w, dtype)
    assert (forward_kernels(lambda: f(xd, wd)) == {"k_conv_small": 1}) == one
    y = f(xd, wd)
    assert rel_err(to_f64(y), ref) <= (ROUNDING if one else TOL)[dtype]
    assert torch.equal(f(xd, wd), y)  # repeatable bit for bit
    # the separate steps (named by an option) stay within the common tolerance of it
    fs = B.Forward(km, c_in, c_out, B.TORCH_DTYPES[dtype], B.Options.make(gather=B.GATHER_FUSED))
    assert "k_conv_small" not in forward_kernels(lambda: fs(xd, wd))
    sep = fs(xd, wd)
    assert rel_err(to_f64(sep), to_f64(y)) <= TOL[dtype]
    if dtype == "f32" and n >= 2000:
        # both sum an offset's channels first and then the offsets, so their errors differ
        # by chance only, over 32,000 outputs or more; one chain over both is 1.5 to 2 times
        # as far off
        assert np.linalg.norm(to_f64(y) - ref) <= 1.25 * np.linalg.norm(to_f64(sep) - ref)
    res = scenes.features(km.n_out, c_out, dtype, 7)
    ye = f(xd, wd, residual=to_dev(res, dtype), relu=True)
    assert rel_err(to_f64(ye), np.maximum(ref + scenes.to_f64(res, dtype), 0.0)) <= \
        2 * (ROUNDING if one else TOL)[dtype]


@pytest.mark.parametrize("dtype,K,c_in,c_out,mode,n,one", [
    ("f16", 3, 32, 32, "subm", 1, True),        # one row
    ("f16", 3, 32, 64, "subm", 16, False),      # few outputs, sparse, 108 KiB of weights
    ("f16", 3, 48, 32, "subm", 17, False),
    ("bf16", 3, 16, 48, "subm", 127, True),     # two offsets per k-step; odd tiles; eight dies less one block
    ("bf16", 3, 8, 16, "subm", 2049, True),     # four offsets per k-step, one tile
    ("f16", 5, 8, 32, "subm", 3001, True),      # 125 offsets: five groups, the last of 13
    ("f16", 2, 24, 96, "subm", 3000, True),     # eight offsets: two entries per lane; a quarter k-step empty
    ("f16", 1, 64, 128, "subm", 3000, True),
    ("f16", 2, 96, 96, "up", 3000, False),
    ("bf16", 2, 64, 128, "down", 3000, True),   # (dense: eight inputs per output)
    ("bf16", 3, 32, 64, "down", 3000, True),
    ("f32", 3, 16, 16, "subm", 3000, True),
    ("f32", 3, 4, 32, "subm", 3000, True),      # four offsets per k-step
    ("f32", 3, 8, 16, "up", 3000, True),
    ("f32", 3, 32, 32, "subm", 9000, True),
    ("f32", 1, 48, 96, "subm", 500, True),
])
def test_narrow_layer_matches_oracle(dtype, K, c_in, c_out, mode, n, one):
    say(f"narrow layer {dtype} K={K} {c_in}->{c_out} {mode} n={n}")
    _check(dtype, K, c_in, c_out, mode, n, 40 if n > 5000 else 16, one)


@pytest.mark.parametrize("dtype,K,c_in,c_out,mode,n,side,one", [
    ("f16", 3, 32, 64, "subm", 16, 3, True),       # one block
    ("f16", 3, 48, 32, "subm", 17, 3, True),       # two k-steps, the second half empty; a block and a row
    ("f16", 2, 96, 96, "up", 9000, 40, True),      # three k-steps
    ("bf16", 2, 64, 128, "down", 20000, 60, True),
    ("f16", 3, 48, 48, "subm", 9000, 40, False),   # the first width past the LDS
    ("f16", 4, 32, 16, "subm", 3000, 16, True),    # 64 offsets: three groups, the last of 8
    ("bf16", 4, 16, 48, "subm", 3000, 24, True),   # the same, two offsets per step
    ("f32", 4, 16, 16, "down", 3000, 16, True),
    ("f16", 5, 16, 32, "subm", 3000, 24, True),    # several groups, two offsets per step
    ("bf16", 5, 32, 16, "down", 3000, 24, True),   # one
    ("f32", 5, 4, 32, "subm", 3000, 16, True),     # four
    ("f32", 5, 8, 16, "subm", 3000, 24, True),
    ("f32", 2, 32, 32, "up", 9000, 40, True),
    ("f32", 3, 16, 64, "subm", 9000, 40, True),
])
def test_narrow_layer_groups_and_limits(dtype, K, c_in, c_out, mode, n, side, one):
    say(f"narrow layer {dtype} K={K} {c_in}->{c_out} {mode} n={n} in {side}^3")
    _check(dtype, K, c_in, c_out, mode, n, side, one)


@pytest.mark.parametrize("dtype,K,c_in", [("f16", 3, 24), ("bf16", 3, 48), ("f16", 3, 16), ("bf16", 3, 8), ("f16", 2, 96),
                                          ("f32", 3, 16), ("f32", 3, 8), ("f32", 3, 4), ("f32", 2, 12)])
def test_an_input_row_that_is_not_finite(dtype, K, c_in):
    """An infinite input row reaches the outputs that have a pair with it, and no others:
    they keep their bits.  One, two and four offsets per k-step, k-steps that are part empty."""
    say(f"non-finite input {dtype} K={K} c_in={c_in}")
    coords = _cloud(81, 3000, 16)
    km, okm, x, w, _ = _layer(K, c_in, 32, dtype, coords)
    f = B.Forward(km, c_in, 32, B.TORCH_DTYPES[dtype])
    xd, wd = to_dev(x, dtype), to_dev(w, dtype)
    y0 = f(xd, wd)
    xd[1234] = float("inf")
    assert forward_kernels(lambda: f(xd, wd)) == {"k_conv_small": 1}
    y = f(xd, wd)
    reached = np.zeros(len(coords), dtype=bool)
    for k in range(okm.K3):
        a, b = okm.pairs(k)
        reached[b[a == 1234]] = True
    assert 0 < reached.sum() < len(coords)
    r = torch.from_numpy(reached).to(y.device)
    assert torch.equal(y[~r], y0[~r])
    assert not torch.isfinite(y[r]).all(dim=1).any()


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
    xs = xd.clone()
    assert "k_conv_small" not in forward_kernels(lambda: f(xs, wd, y=xs))
    assert f(xd, wd, y=xd) is xd
    assert rel_err(to_f64(xd), ref) <= TOL["f32"]


@pytest.mark.parametrize("what,shift", [("x", 4), ("x", -1000), ("x", 47_996), ("w", 0), ("w", 6_908), ("w", -47_996)])
def test_output_over_part_of_an_operand(what, shift):
    """The same for an output that begins or ends inside the input or the weights; one that
    only touches them runs as one kernel."""
    say(f"output over part of {what}, {shift} elements on")
    n = 3000
    coords = _cloud(82, n, 16)
    km, _, x, w, ref = _layer(3, 16, 16, "f32", coords)
    f = B.Forward(km, 16, 16, torch.float32)
    buf = torch.empty(4 * 16 * n, device="cuda")
    at = 16 * n  # of the operand; the output lies `shift` elements on
    op = to_dev(x if what == "x" else w)
    held = buf[at:at + op.numel()].view(op.shape)
    y = buf[at + shift:at + shift + 16 * n].view(n, 16)
    other = to_dev(w if what == "x" else x)

    def run():
        held.copy_(op)
        return f(held, other, y=y) if what == "x" else f(other, held, y=y)

    assert "k_conv_small" not in forward_kernels(run)
    assert rel_err(to_f64(run()), ref) <= TOL["f32"]
    free = buf[at + op.numel():at + op.numel() + 16 * n].view(n, 16)  # touches the operand's end
    held.copy_(op)
    a, b = (held, other) if what == "x" else (other, held)
    assert forward_kernels(lambda: f(a, b, y=free)) == {"k_conv_small": 1}
    assert rel_err(to_f64(free), ref) <= TOL["f32"]


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
