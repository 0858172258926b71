"""GPU parity of the full-width matrix product in float32, and of small launches, whose
tiles and column slices are chosen by the rows there are.

float32 features against the oracle within the common tolerance.  Neither the rows of a
tile, nor the slices, nor the form of the gather changes the order of a sum, so those
agree bit for bit.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2401_06145_amd import binding as B
from paper_2401_06145_amd import scenes
from tests.gpu_helpers import TOL, rel_err, say, to_dev, to_f64

pytestmark = pytest.mark.gpu


def _cloud(seed, n, side):
    return scenes.uniform_cells(n, side, seed)


@pytest.mark.parametrize("dtype,K,c_in,c_out,n", [
    ("f32", 3, 64, 64, 1),         # one row
    ("f32", 3, 64, 128, 600),      # few rows: slices of two tiles
    ("f32", 3, 36, 48, 2000),      # a k-step of four channels; three tiles
    ("f32", 3, 260, 32, 700),      # wider than the full-width kernel takes
    ("f32", 3, 256, 256, 1500),    # the widest input it takes; two slices at the least
    ("f32", 1, 128, 192, 3000),    # one offset
    ("f32", 2, 20, 160, 3000),     # odd number of tiles
    ("f32", 3, 64, 64, 12000),     # tiles of 512 rows
    ("f16", 3, 128, 128, 400),     # few rows
    ("bf16", 2, 256, 256, 900),
    ("f16", 3, 64, 96, 4000),      # tiles of 256 rows
])
def test_tiles_and_slices(dtype, K, c_in, c_out, n):
    say(f"matrix product {dtype} K={K} {c_in}->{c_out} n={n}")
    coords = _cloud(500 + n, n, 28 if n > 5000 else 17)
    mode = "down" if K == 2 else "subm"
    q = oracle.out_coords(coords, 2, 1) if K == 2 else None
    km = B.KernelMap.build(to_dev(coords), K, 2 if K == 2 else 1, 1, mode)
    okm = oracle.kernel_map(coords, q, K, 1, mode)
    x, w = scenes.features(km.n_in, c_in, dtype, 3), scenes.weights(K, c_in, c_out, dtype, 4)
    ref = oracle.features(scenes.to_f64(x, dtype), scenes.to_f64(w, dtype), okm)
    xd, wd = to_dev(x, dtype), to_dev(w, dtype)

    def run(**opt):
        return B.Forward(km, c_in, c_out, B.TORCH_DTYPES[dtype], B.Options.make(centre=1, **opt))(xd, wd)

    y = run()
    assert rel_err(to_f64(y), ref) <= TOL[dtype]
    assert torch.equal(run(gemm_tile_rows=16), y)
    assert torch.equal(run(gemm_tile_rows=4096), y)
    assert torch.equal(run(gather=B.GATHER_BUFFER), y)
    assert torch.equal(run(gather=B.GATHER_FUSED), y)
