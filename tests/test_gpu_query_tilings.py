"""Which tiling of the query kernel runs is decided by the sizes of a plain problem: results on both sides of every
border against the fp64 oracle (sampled rows), and equal bits whatever block_size the caller names.

Tolerance: the bars of test_gpu_parity.py (bf16 rounding of weights, features and output, about 2e-3 r.m.s.)."""
import numpy as np
import pytest
import torch

from paper_2509_24899_amd import workloads as W
from test_gpu_parity import check

pytestmark = pytest.mark.gpu

# d, map width (0: rate 1, no maps), heads, N: 256-query workgroups are H ceil(N / 256), 128-query ones H ceil(N / 128)
CASES = [
    (64, 64, 12, 5376), (64, 64, 12, 5377),          # d = 64: 252 / 264 workgroups of 256 queries (border at 256)
    (64, 64, 1, 257),
    (128, 384, 12, 2688), (128, 384, 12, 2689),      # linear part precomputed: 252 / 264 workgroups of 128 queries
    (128, 0, 2, 16384), (128, 0, 2, 16385), (64, 0, 3, 230),   # no linear part: 256 / 258 workgroups of 128 queries
    (128, 0, 12, 6200), (128, 0, 12, 8000),                    # ... and a last round that is full / half empty
    (128, 128, 2, 129), (128, 128, 3, 1), (128, 128, 1, 256), (128, 256, 2, 385),
]


@pytest.mark.parametrize("d,width,H,N", CASES)
@pytest.mark.parametrize("dtype", ("bf16", "f32"))
def test_both_sides_of_the_tiling_rules(d, width, H, N, dtype):
    R = 1 if width == 0 else 4 if N > 1 else 0
    width = width or d
    P = 3 if width == 384 else 2
    w = W.Workload(f"tiling_d{d}_F{width}_H{H}_N{N}_{dtype}", 1, H, N, d, dtype, 64, R, width, width, poly_degree=P, seed=N)
    inp = W.make_inputs(w)
    rows = W.sample_rows(w, n_random=32) if N > 600 else None
    y64, _ = check(w.name + "_bs64", inp, block_size=64, rows=rows)
    y128, _ = check(w.name + "_bs128", inp, block_size=128, rows=rows)
    assert np.array_equal(y64, y128)
