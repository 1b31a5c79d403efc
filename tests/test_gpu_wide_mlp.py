"""The streaming layer kernel of the wide feature maps, through the forward (the gradient suites cover the images it keeps
for the backward pass): widths with and
without a block of four output tiles, shortest and longest contraction, two and three layers, token counts around the
256-token tile and the last idle waves, more heads than a workgroup's run, both dtypes.

Tolerance: the bars of test_gpu_parity.py."""
import numpy as np
import pytest
import torch

from paper_2509_24899_amd import workloads as W
from test_gpu_parity import check

pytestmark = pytest.mark.gpu


def work(N, hid, feat, mid=0, P=2, H=2, B=1, R=3, dtype="bf16", seed=0):
    return W.Workload(f"wm_{hid}_{mid}_{feat}_N{N}_H{H}_{dtype}", B, H, N, 128, dtype, 128, R, hid, feat, poly_degree=P, d_mid=mid, seed=seed)


@pytest.mark.parametrize("dtype", ("bf16", "f32"))
@pytest.mark.parametrize("hid,feat,mid,P", ((128, 384, 0, 3), (768, 128, 0, 2), (384, 640, 0, 4), (256, 512, 0, 4),
                                            (128, 128, 128, 2), (640, 768, 384, 6), (768, 768, 768, 6)))
def test_widths(hid, feat, mid, P, dtype):
    check("wm", W.make_inputs(work(333, hid, feat, mid, P, dtype=dtype, seed=hid + feat)))


@pytest.mark.parametrize("N", (1, 32, 255, 256, 257, 289, 2049))
@pytest.mark.parametrize("mid", (0, 256))
def test_token_counts(N, mid):
    w = work(N, 384, 384, mid, 3, R=0 if N == 1 else 4 if N > 4 else 2, seed=N)
    check(w.name, W.make_inputs(w), rows=W.sample_rows(w, n_random=16) if N > 600 else None)


def test_many_heads():
    w = work(300, 384, 512, 256, 4, H=60, B=3, R=2, seed=9)
    check(w.name, W.make_inputs(w), rows=np.arange(0, 300, 7))
